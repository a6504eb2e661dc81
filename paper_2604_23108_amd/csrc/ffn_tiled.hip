// Expert feed-forward networks for prefill-sized token counts on gfx950: a ragged
// grouped GEMM on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16, fp32 accumulate).
//
// Two launches: "up" computes H = SiLU(X W_gate^T) * (X W_up^T) for every expert's
// rows, "down" computes Y = H W_down^T.  Both have the form C[rows of expert e] =
// A_rows . B_e^T with A and B contiguous along the reduction dimension.  What makes it
// ragged: the row count n_e comes from the router (device memory `offsets`), the width
// F_g differs from group to group (it is N of the up and K of the down projection).
//
// Schedule (device side, no host synchronisation).  A one-workgroup kernel turns
// `offsets` into a list of tiles: up to 256 token rows x 256 weight rows (up: 128 W_gate +
// the matching 128 W_up rows).  It picks the tile height (128, 192 or 256 rows) that needs
// the fewest rounds over the compute units, orders tiles so that tiles sharing operands are
// neighbours and every stretch of the list mixes all group widths, and cuts the list into 8 ranges of
// equal cost, one per XCD (each XCD has its own L2).  The GEMM kernel is persistent: one
// workgroup per compute unit, workgroup b serves XCD b%8 (the hardware hands workgroups
// to XCDs round-robin) and draws tiles of that XCD's range from an atomic counter.
//
// Tile kernel.  8 waves as 2 (token) x 4 (weight) with wave tiles of 128 x 64; a wave owns
// the 32-row token fragments {wm, wm+2, wm+4, wm+6}, so a tile with fewer rows keeps both
// wave rows equally busy and simply runs fewer MFMAs (the inner loop is instantiated for
// 1..4 active fragments).  Operands go global -> LDS with global_load_lds_dwordx4 (no
// staging registers) in 128-byte row segments (BK = 64): the texture path handles about one
// 128-byte line per two clocks however little of it is used, so 64-byte segments halve the
// feed rate (measured 24 vs 57 B/clk per CU).  16-byte chunks are XOR-swizzled inside the
// tile rows so that ds_read_b128 fragment reads are conflict free.  All 160 KB of LDS are
// used, asymmetrically: two stages for the token operand (its rows are shared by all column
// tiles of an expert and mostly hit in L2) and three for the weight operand (streamed from
// HBM), whose requests so start half a stage earlier.  The token gather is fused: a tile
// row's global address is taken through `perm`.
// Which instruction: power bounds these launches (the clock falls to 1.7 to 2.0 GHz), and on operands with full mantissas
// 16x16x32 draws less of it than 32x32x16, whose accumulators are read and written twice as often per product: alone 2060
// against 1750 TFLOP/s, with the operand reads from LDS 1870 against 1650.
// The inner loop is ordered by hand (pinned with sched_barrier): between the MFMAs of a 32-deep k-step stand the LDS reads of
// the fragments it will need next, a token fragment's register being refilled right after its last use, and the global -> LDS
// requests, spread over the whole stage; one barrier per stage, placed three token fragments into its second k-step, so
// that the first fragments of the next stage are read under MFMAs as well (run_tile has the figures).  16384 tokens, d = 4096,
// skewed: launch 2029 -> 1820 us (1.07 -> 1.19 PFLOP/s), main loop 2400 -> 2260 clocks a stage at 1.72 -> 1.82 GHz.
// The MFMA takes the weight fragment as first operand: a lane then holds 4 consecutive
// output features of one token; the epilogue packs them to bf16 (hardware conversion),
// transposes through a wave-private LDS patch and stores whole row segments.
//
// Backward products (modes of the same kernel).  Their second operand, and for the weight
// gradients both operands, are stored with the reduction index as the row: dH = dY W_down
// reduces over the rows of W_down[e] ([d, F]), dX = [dA|dB] W13 over the rows of W13[e]
// ([2F, d]), dW_e = A_e^T B_e over the routed rows of expert e.  Such an operand is staged as
// 64 reduction rows x 256 features (512-byte row segments, again through global_load_lds,
// chunks swizzled by the row), and its MFMA fragments are read with ds_read_b64_tr_b16, which
// hands every lane four consecutive reduction indices of one feature.  No operand is
// transposed in memory.  The ragged reduction of the weight gradients needs no padding
// either: rows past the expert's last token are fetched from a row of zeros.
#include <type_traits>

#include "common.h"
#include "tiled.h"

namespace mohge {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBM = 256, kBN = 256, kBK = 64;
constexpr int kStagesA = 2, kStagesB = 3;   // 32 KB parts: 2 token + 3 weight = all 160 KB of LDS
constexpr int kWGM = 2, kWGN = 4;
// LDS words for the hand-over between the tiles of a persistent workgroup: beyond the epilogue patches
// (one per wave, at most 32 rows x 144 bytes), inside a stage buffer that is dead between two tiles
constexpr int kHandoverOffset = (kWGM * kWGN * 32 * 144 / 4096 + 1) * 4096;
static_assert(kHandoverOffset == 40960 && kHandoverOffset + 8 <= 2 * kBM * kBK * 2, "inside the second token part");
// Cost model of the schedule: fixed part of a tile's stage, in 64-row units.  (Now a stage of 64, 128, 192, 256 rows takes 930,
// 1410, 1808, 2270 clocks and the rest of such a tile 5.7, 7.1, 7.9, 10.8 k.  Ranges cut and heights chosen by that, (1 + units) x
// (stages + 4): 0.985 to 1.02 of the time over 14 layers, mean 1.00, so that these lines stay where they were measured.)
constexpr int kTileCost = 18;

// gate and up rows share a tile in the two up-projection modes
constexpr bool is_up(int mode) { return mode == kUp || mode == kUpSave; }
// operand stored reduction-index major (features contiguous): read through the transposing LDS read
constexpr bool tr_a(int mode) { return mode == kWgrad; }
constexpr bool tr_b(int mode) { return mode == kWgrad || mode == kDgradH || mode == kDgradX; }
// reduction over d, F_g output columns
constexpr bool red_d(int mode) { return is_up(mode) || mode == kDgradH; }

// Tile geometry.  Big: 256 x 256 tiles, 8 waves, all 160 KB of LDS, one persistent workgroup per
// compute unit.  Small: 128 x 128 tiles, 4 waves, half the LDS, two workgroups per compute unit (the
// launches that would leave compute units idle with big tiles, see use_small_tiles).
struct BigTile { static constexpr int BM = kBM, BN = kBN, WGM = kWGM, WGN = kWGN; static constexpr bool LONG = false; };
// Long: big tiles of weights whose rows are so long (kLongRow) that a 32-bit offset does not reach from a tile's first row to its last.
// With its addresses everywhere 16384 tokens of d = 4096 took 1.4 % longer (2031 -> 2062 us).
struct LongTile : BigTile { static constexpr bool LONG = true; };
constexpr int kLongRow = 1 << 23;       // 256 rows of 2 bytes times this: 2^32 bytes
struct SmallTile { static constexpr int BM = 128, BN = 128, WGM = 2, WGN = 2; static constexpr bool LONG = false; };
// Tall: the small form's token modes, up to 192 rows of one expert (see small_token_tile)
struct TallTile : SmallTile { static constexpr int BM = 192; };

template <int MODE>
struct Shape {
  static constexpr int NCOLS_PER_TILE = is_up(MODE) ? kBN / 2 : kBN;
  // wave grid of the workgroup: 2 x 4 waves with 128 x 64 wave tiles (2 x 2 waves with
  // 128 x 128 wave tiles read a third fewer fragments per MFMA but measured slower in every
  // mode, the weight gradients with their transposing reads included; 4 x 4 waves with 64 x 64
  // wave tiles leave 128 registers a lane, spill, and measured 10 % slower)
  static constexpr int WGM = kWGM, WGN = kWGN;
  static constexpr int THREADS = 64 * WGM * WGN;
};

// ---------------------------------------------------------------------------------------
// schedule: one workgroup of 256 threads per projection; thread v <-> expert at visiting
// position v for the per-expert quantities, then threads stride over the tiles
// ---------------------------------------------------------------------------------------
// wave_incl_scan for 64-bit values (not negative): three parts of 24 bits, each summed by itself (64 x 2^24 fits an int)
__device__ __forceinline__ long long wave_incl_scan64(long long v) {
  const int lo = wave_incl_scan((int)(v & 0xffffff)), mid = wave_incl_scan((int)((v >> 24) & 0xffffff));
  const int hi = wave_incl_scan((int)(v >> 48));
  return ((long long)hi << 48) + ((long long)mid << 24) + lo;
}

struct SchedShared {
  long long tp[kMaxExperts + 1];   // tiles before expert v
  long long cp[kMaxExperts + 1];   // cost before expert v
  int e[kMaxExperts], cnt[kMaxExperts], nt[kMaxExperts], kc[kMaxExperts], row0[kMaxExperts];
  int fp[kMaxExperts + 1];         // row blocks before expert v
  int sp[kMaxExperts + 1];         // tiles of the shortest reduction before expert v (see build_schedule)
  long long wsum[4][4];
  int rows;
  int xb[kXcds + 1];               // tile ranges per XCD (copy of the header's)
  int xs[kXcds + 1];               // tiles of the shortest reduction before each range
};

// Per-expert quantities of a mode: rows (`cnt`, starting at `row0`), output columns, and
// reduction length in 64-deep stages.
// Expert at visiting position v.  group_major: all experts of a group are neighbours, groups by
// decreasing width (tiles of one reduction length run together and the shortest come last);
// otherwise expert index major, group minor ("all-size sets": every stretch mixes all widths).
__device__ __forceinline__ void visit(const TileArgs& a, int v, int& e, int& g) {
  if (a.group_major) { g = a.order[v / a.N]; e = g * a.N + v % a.N; }
  else { g = a.order[v % a.Ng]; e = g * a.N + v / a.Ng; }
}

template <int MODE>
__device__ __forceinline__ void expert_dims(const TileArgs& a, int e, int g, int& row0, int& cnt,
                                            int& ncols, int& kc) {
  if constexpr (MODE == kWgrad) {
    row0 = 0;
    cnt = a.Mrows[g];
    ncols = a.Ncols[g];
    kc = (a.offsets[e + 1] - a.offsets[e] + 63) / 64;
    if (kc < 1) kc = 1;          // an expert without tokens still gets its zero gradient written
  } else {
    row0 = a.offsets[e];
    cnt = a.offsets[e + 1] - row0;
    ncols = red_d(MODE) ? a.F[g] : a.d;
    kc = (red_d(MODE) ? a.d : a.F[g]) / 64;
  }
}

// Tile height for a launch of MODE: the candidate with the lowest estimated time.  Called by all
// 256 threads; uses sh.wsum and sh.rows.
template <int MODE>
__device__ __forceinline__ int choose_tile_rows(const TileArgs& a, SchedShared& sh, bool fused = false) {
  constexpr int NCPT = Shape<MODE>::NCOLS_PER_TILE;
  const int v = threadIdx.x, lane = v & 63, w = v >> 6;
  int cnt = 0, nt = 0, kc = 0;
  if (v < a.Ne) {
    int e, g;
    visit(a, v, e, g);
    int ncols, row0;
    expert_dims<MODE>(a, e, g, row0, cnt, ncols, kc);
    nt = (ncols + NCPT - 1) / NCPT;
  }
  long long cand[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int h = 256 - 64 * c;
    cand[c] = wave_incl_scan64((long long)((cnt + h - 1) / h) * nt * kc);      // lane 63: the wave's sum
  }
  __syncthreads();
  if (lane == 63) { sh.wsum[w][0] = cand[0]; sh.wsum[w][1] = cand[1]; sh.wsum[w][2] = cand[2]; }
  __syncthreads();
  if (v == 0) {
    long long kmax = 1;
    for (int g = 0; g < a.Ng; ++g)
      kmax = max(kmax, (long long)((red_d(MODE) ? a.d : a.F[g]) / 64));
    float best = 0.f;
    int best_rows = 256;
    for (int c = 0; c < 3; ++c) {
      const long long tot = sh.wsum[0][c] + sh.wsum[1][c] + sh.wsum[2][c] + sh.wsum[3][c];
      // rounds count more than height (the constants are those of the loop before this one; heights chosen by the present
      // clocks gain nothing, see kTileCost)
      // (fused launch: the down tiles fill the last round of up tiles, so the up tiles are
      // costed by their total work rather than by whole rounds)
      const float units = fused ? (float)tot / (float)((long long)a.ncu * kmax)
                                : (float)((tot + (long long)a.ncu * kmax - 1) / ((long long)a.ncu * kmax));
      const float est = units * ((float)(4 - c) + 18.5f);
      if (c == 0 || est < best) { best = est; best_rows = 256 - 64 * c; }
    }
    sh.rows = a.force_rows ? a.force_rows : best_rows;
  }
  __syncthreads();
  const int h = sh.rows;
  __syncthreads();
  return h;
}

// Tile list of a launch of MODE with tile height h.  FUSED: the list belongs to a launch that
// runs up and down tiles together; down tiles then carry the number of up tiles they wait for.
// part / nparts: several workgroups may build one list together: each derives the (cheap) per-expert
// prefix sums itself and writes every nparts-th stretch of 256 records; part 0 writes the header.
template <int MODE>
__device__ __forceinline__ void build_schedule(const TileArgs& a, SchedShared& sh, int h, bool fused,
                                               int part = 0, int nparts = 1) {
  constexpr int NCPT = Shape<MODE>::NCOLS_PER_TILE;
  const int v = threadIdx.x, lane = v & 63, w = v >> 6;
  int e = 0, cnt = 0, nt = 0, kc = 0, row0 = 0;
  if (v < a.Ne) {
    int g;
    visit(a, v, e, g);
    int ncols;
    expert_dims<MODE>(a, e, g, row0, cnt, ncols, kc);
    nt = (ncols + NCPT - 1) / NCPT;
  }
  sh.e[v] = e; sh.cnt[v] = cnt; sh.nt[v] = nt; sh.kc[v] = kc; sh.row0[v] = row0;
  // exclusive prefix sums of tiles, cost and row blocks over the experts
  const int my_t = (cnt + h - 1) / h * nt;
  // cost of a tile = reduction stages x (kTileCost + its 64-row units)
  const long long my_c = ((long long)kTileCost * ((cnt + h - 1) / h) + (cnt + 63) / 64) * nt * kc;
  const int my_f = MODE == kWgrad ? 0 : (cnt + h - 1) / h;
  // Second list of a fused launch (its tiles wait for tiles of the first): inside every XCD range
  // the tiles of the groups with the shortest reduction go last, everything else keeps its order.
  // The end of a range is then handed out in its smallest pieces (the launch ends when the slowest
  // workgroup does), and a tile only ever moves to a LATER position, so none meets its row block
  // earlier than before.
  int kmin = 1 << 30, kmax = 0;
  for (int g = 0; g < a.Ng; ++g) {
    const int k = (red_d(MODE) ? a.d : a.F[g]) / 64;
    kmin = min(kmin, k);
    kmax = max(kmax, k);
  }
  const bool short_last = fused && a.short_last && (MODE == kDown || MODE == kDgradX) && kmin < kmax;
  const int my_s = (short_last && v < a.Ne && kc == kmin) ? my_t : 0;
  const int it = wave_incl_scan(my_t), jf = wave_incl_scan(my_f), is = wave_incl_scan(my_s);
  const long long ic = wave_incl_scan64(my_c);
  if (lane == 63) { sh.wsum[w][0] = it; sh.wsum[w][1] = ic; sh.wsum[w][2] = jf; sh.wsum[w][3] = is; }
  __syncthreads();
  long long bt = 0, bc = 0, bf = 0, bs = 0;
  for (int ww = 0; ww < w; ++ww) { bt += sh.wsum[ww][0]; bc += sh.wsum[ww][1]; bf += sh.wsum[ww][2]; bs += sh.wsum[ww][3]; }
  sh.tp[v] = bt + it - my_t;
  sh.cp[v] = bc + ic - my_c;
  sh.fp[v] = (int)(bf + jf - my_f);
  sh.sp[v] = (int)(bs + is - my_s);
  if (v == 255) { sh.tp[256] = bt + it; sh.cp[256] = bc + ic; sh.fp[256] = (int)(bf + jf); sh.sp[256] = (int)(bs + is); }
  __syncthreads();
  const int total = (int)sh.tp[256];
  const long long ctot = sh.cp[256];
  // expert (visiting position) of tile t: last v with tp[v] <= t
  auto expert_of = [&](int t) {
    int lo = 0, hi = a.Ne - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (sh.tp[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  // Inside an expert the tiles run in bands of `band` row blocks: band after band, inside a band
  // column tile major, row block minor.  The workgroups of an XCD draw consecutive tiles, so at any
  // moment they work on a few row blocks x a few column tiles of one expert and share both operand
  // panels through that XCD's L2 (an expert's whole column of row blocks per column tile would
  // share the weight panel only).
  const int RB = a.band > 0 ? a.band : 1;
  // XCD x starts at the first tile whose preceding cost is >= x/8 of the total.  The cost before
  // the tile at position rel of an expert follows from the band order in closed form, so the tile
  // is found by bisection once the expert is known.
  // (a wave takes two of the eight ranges and its lanes look at 64 positions at once: one thread per range, bisecting
  // over 256 experts: 13.7 us for the launch at 24 experts x 683 rows, now 11.9)
  for (int x = w; x < kXcds; x += 4) {
    const long long target = (ctot * x + kXcds - 1) / kXcds;
    int lo = 0, hi = a.Ne - 1;               // last expert with cp[ve] <= target
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (sh.cp[mid] <= target) lo = mid; else hi = mid - 1;
    }
    const int ve = lo;
    const int c = sh.cnt[ve], kcv = sh.kc[ve], ntv = sh.nt[ve];
    const long long rem = target - sh.cp[ve];
    int tile;
    if (rem <= 0 || c == 0 || kcv == 0 || ntv == 0) {
      tile = (int)sh.tp[ve];                 // (cp[ve] == target: the expert's first tile)
      if (rem > 0) tile = (int)sh.tp[ve + 1];
    } else {
      const int mt = (c + h - 1) / h, units = (c + 63) / 64, hu = h / 64;
      auto cost_before = [&](int rel) -> long long {
        if (rel >= mt * ntv) return ((long long)kTileCost * mt + units) * ntv * kcv;
        const int bnd = rel / (RB * ntv), rel2 = rel - bnd * RB * ntv;
        const int rb = min(RB, mt - bnd * RB);
        const int ni = rel2 / rb, mi2 = rel2 % rb;
        const int ub = min(units - bnd * RB * hu, RB * hu);         // 64-row units of this band
        return ((long long)kTileCost * rel + (long long)bnd * RB * hu * ntv + (long long)ni * ub +
                min(mi2 * hu, ub)) * kcv;
      };
      // smallest rel in [0, mt * ntv] with cost_before(rel) >= rem (the last one has it): lane l looks at the end of
      // the l-th of 64 stretches, and the first that qualifies holds it
      int rl = 0, len = mt * ntv + 1;
      while (len > 1) {
        const int step = (len + 63) / 64, at = min((lane + 1) * step, len) - 1;
        const unsigned long long ok = __ballot(cost_before(rl + at) >= rem);
        const int first = ok ? (int)__builtin_ctzll(ok) : 63;
        rl += first * step;
        len = min(step, len - first * step);
      }
      tile = min((int)sh.tp[ve] + rl, (int)sh.tp[ve + 1]);
    }
    if (lane == 0) {
      if (part == 0) a.hdr->xcd_begin[x] = tile;
      sh.xb[x] = tile;
    }
  }
  if (v == kXcds) {
    if (part == 0) a.hdr->xcd_begin[v] = total;
    sh.xb[v] = total;
  }
  __syncthreads();
  // tiles of the shortest reduction before tile t (t may be `total`)
  auto short_before = [&](int t, int ve) {         // ve: the tile's expert
    return sh.sp[ve] + ((sh.sp[ve + 1] > sh.sp[ve]) ? t - (int)sh.tp[ve] : 0);
  };
  if (v <= kXcds) {
    const int t = sh.xb[v];
    sh.xs[v] = !short_last ? 0 : t >= total ? sh.sp[256] : short_before(t, expert_of(t));
  }
  __syncthreads();
  for (int t = v + 256 * part; t < total; t += 256 * nparts) {
    const int ve = expert_of(t);
    const int c = sh.cnt[ve], mt = (c + h - 1) / h, ntv = sh.nt[ve];
    const int rel = t - (int)sh.tp[ve];
    const int bnd = rel / (RB * ntv), rel2 = rel - bnd * RB * ntv;
    const int rb = min(RB, mt - bnd * RB);
    const int ni = rel2 / rb, mi = bnd * RB + rel2 % rb;
    TileRec r;
    r.e = sh.e[ve];
    r.row_start = sh.row0[ve] + mi * h;
    r.rows = min(h, c - mi * h);
    r.n0 = ni * NCPT;
    r.fam = sh.fp[ve] + mi;
    // a down tile of the fused forward waits for the up tiles of its row block: one per 128
    // hidden units of the expert's group (F holds the group's width in kDown)
    // (kDown: the reduction is the group's width, the up tiles are 128 hidden units wide; kDgradX:
    // twice the width, the dH tiles are 256 hidden units wide)
    r.need = !fused ? 0
             : MODE == kDown ? (sh.kc[ve] * kBK + kBN / 2 - 1) / (kBN / 2)
             : MODE == kDgradX ? (sh.kc[ve] * kBK / 2 + kBN - 1) / kBN : 0;
    int pos = t;
    if (short_last) {
      int x = 0;                                   // the tile's XCD range
      while (x + 1 < kXcds && t >= sh.xb[x + 1]) ++x;
      const int sb = short_before(t, ve) - sh.xs[x];   // short tiles of the range before t
      const int nlong = (sh.xb[x + 1] - sh.xb[x]) - (sh.xs[x + 1] - sh.xs[x]);
      const bool is_short = sh.sp[ve + 1] > sh.sp[ve];
      pos = is_short ? sh.xb[x] + nlong + sb : sh.xb[x] + (t - sh.xb[x]) - sb;
    }
    a.recs[pos] = r;
  }
  if (part != 0) return;                     // (workgroup-uniform: everything below is part 0's)
  // tail[x]: the tiles at the end of range x that belong to an expert whose tiles continue in
  // range x+1.  The fused launch computes them first (see fused_phase).
  if (v < kXcds) {
    const int cut = sh.xb[v + 1];
    int n = 0;
    if (cut > 0 && cut < total) {
      const int ve = expert_of(cut);                 // expert of the first tile of range x+1
      n = cut - (int)sh.tp[ve];                      // its tiles before the cut ...
      n = min(n, cut - sh.xb[v]);                    // ... that lie inside range x
      if (n < 0) n = 0;
    }
    a.hdr->tail[v] = n;
  }
  // the first ncu/8 tiles of a range are taken statically, one per workgroup (fused launch:
  // every tile is handed out by the counter, so that the tiles a waiting workgroup depends on
  // never sit with a workgroup that has not started yet)
  if (v < kXcds) a.hdr->counters[v] = fused ? 0 : a.ncu / kXcds;
  if (v == 0) { a.hdr->tile_rows = h; a.hdr->total = total; a.hdr->pad[0] = 0; }
  // fused forward: the row-block counters start at zero (the up list's workgroup clears them)
  if (fused && (is_up(MODE) || MODE == kDgradH))
    for (int i = v; i < sh.fp[256]; i += 256) a.fam_done[i] = 0;
}

template <int MODE>
__device__ __forceinline__ void build_schedule(const TileArgs& a, SchedShared& sh) {
  const int h = choose_tile_rows<MODE>(a, sh);
  build_schedule<MODE>(a, sh, h, false);
}

// workgroup 0 schedules the up projection, workgroup 1 the down projection (mask bits 0 / 1).
// mask 7: both lists for the fused launch, which needs one tile height for both (the up
// projection's choice, it is the larger part) so that row blocks coincide.
__global__ void __launch_bounds__(256) ffn_schedule_kernel(const TileArgs up, const TileArgs dn, int mask) {
  __shared__ SchedShared sh;
  if (mask == 7) {
    // several workgroups per list (blockIdx.x = list + 2 * part)
    const int h = choose_tile_rows<kUp>(up, sh, true);
    const int part = blockIdx.x >> 1, nparts = gridDim.x >> 1;
    if ((blockIdx.x & 1) == 0) build_schedule<kUp>(up, sh, h, true, part, nparts);
    else build_schedule<kDown>(dn, sh, h, true, part, nparts);
    return;
  }
  const int which = (mask == 3) ? (int)blockIdx.x : (mask == 2 ? 1 : 0);
  if (which == 0) build_schedule<kUp>(up, sh);
  else build_schedule<kDown>(dn, sh);
}

// the four schedules of the expert backward pass in one launch: workgroup i <-> launch i
// fused: the lists are for two fused launches (dH then dX, which waits for dH's row blocks and
// so shares its tile height; the two weight gradients one after the other)
__global__ void __launch_bounds__(256) bwd_schedule_kernel(const TileArgs dh, const TileArgs dx,
                                                           const TileArgs w2, const TileArgs w13, int fused,
                                                           const GatherArgs ga) {
  if (blockIdx.x >= 4) {
    // rows of x in sorted order, one wave per row; the first of these workgroups also clears the
    // row of zeros the weight-gradient tiles read past an expert's last row
    const int b = blockIdx.x - 4;
    if (b == 0 && threadIdx.x < 32) ga.zero_row[threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
    const int p = b * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (p >= ga.P || ga.perm == nullptr) return;
    const long long row = ga.perm[p] / ga.Ke;
    for (int c = lane; c < ga.chunks; c += 64) ga.xs[(long long)p * ga.chunks + c] = ga.x[row * ga.chunks + c];
    return;
  }
  __shared__ SchedShared sh;
  if (fused) {
    if (blockIdx.x < 2) {
      const int h = choose_tile_rows<kDgradH>(dh, sh, true);
      if (blockIdx.x == 0) build_schedule<kDgradH>(dh, sh, h, true);
      else build_schedule<kDgradX>(dx, sh, h, true);
    } else if (blockIdx.x == 2) {
      const int h = choose_tile_rows<kWgrad>(w2, sh);
      build_schedule<kWgrad>(w2, sh, h, true);
    } else {
      const int h = choose_tile_rows<kWgrad>(w13, sh);
      build_schedule<kWgrad>(w13, sh, h, true);
    }
    return;
  }
  if (blockIdx.x == 0) build_schedule<kDgradH>(dh, sh);
  else if (blockIdx.x == 1) build_schedule<kDgradX>(dx, sh);
  else if (blockIdx.x == 2) build_schedule<kWgrad>(w2, sh);
  else build_schedule<kWgrad>(w13, sh);
}

// schedule of one launch
template <int MODE>
__global__ void __launch_bounds__(256) tile_schedule_kernel(const TileArgs a) {
  __shared__ SchedShared sh;
  build_schedule<MODE>(a, sh);
}

// ---------------------------------------------------------------------------------------
// tile kernel
// ---------------------------------------------------------------------------------------
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Copy to LDS, 16 bytes per lane, as an instruction the compiler does not model.  The builtin counts as an access to both
// memories: until a wait for every one of them, which this kernel never makes in its main loop, each wait for an LDS read is
// for all of them, and in front of a transposing read (an intrinsic) it waits for every copy on its way.  M0 holds the LDS
// destination; the compiler puts it there (an operand bound to the register, so it knows what M0 holds before and after).
// One wait state, which the hardware asks for after a scalar write of M0; a vector instruction that wrote it or the base would
// need five: the build looks for one in the code the compiler made and takes five everywhere if it finds it (602 -> 608 us for
// 8192 rows, d = 4096).  Both address forms write no register; completion is awaited by the explicit vmcnt waits of the stages.
#ifndef MOHGE_LDS_COPY_NOP
#define MOHGE_LDS_COPY_NOP "0"
#endif
// lds_addr: address in the workgroup's LDS (lds_address() of the buffer plus an offset), wave-uniform.
__device__ __forceinline__ int lds_address(const unsigned char* lds) {
  return (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)lds;
}
__device__ __forceinline__ void async_copy16(const void* gptr, int lds_addr) {
  asm volatile("s_nop " MOHGE_LDS_COPY_NOP "\n\tglobal_load_lds_dwordx4 %0, off"
               ::"v"(gptr), "{m0}"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory");
}
// wave-uniform base, 32-bit byte offset per lane (half the registers)
__device__ __forceinline__ void async_copy16(const void* uniform_base, uint32_t offset, int lds_addr) {
  asm volatile("s_nop " MOHGE_LDS_COPY_NOP "\n\tglobal_load_lds_dwordx4 %0, %1"
               ::"v"(offset), "s"(uniform_base), "{m0}"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory");
}

#define MOHGE_PIN() __builtin_amdgcn_sched_barrier(0)

// 16-byte store performed at device scope (the sc1 cache policy of a vector store): written
// through the XCD's L2, so that once the store has completed (vmcnt) a workgroup on any XCD
// that has not cached the line before reads the new data.
__device__ __forceinline__ void store16_device_scope(void* p, const uint4 v) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 q = {v.x, v.y, v.z, v.w};
  asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(p), "v"(q) : "memory");
}

// SwiGLU backward for 8 packed bf16 values.  The training forward stored, per hidden unit,
//   p = b * SiLU'(a) = b * s * (1 + a*(1-s))   and   q = SiLU(a) = a * s,   s = sigmoid(a),
// so that  dA = dh * p,  dB = dh * q.
__device__ __forceinline__ void swiglu_bwd8(const uint4 dh, const uint4 pv, const uint4 qv, uint4& da,
                                            uint4& db) {
  const uint32_t hw[4] = {dh.x, dh.y, dh.z, dh.w};
  const uint32_t pw[4] = {pv.x, pv.y, pv.z, pv.w};
  const uint32_t qw[4] = {qv.x, qv.y, qv.z, qv.w};
  uint32_t oa[4], ob[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float ra[2], rb[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float g = __uint_as_float(h ? (hw[i] & 0xffff0000u) : (hw[i] << 16));
      ra[h] = g * __uint_as_float(h ? (pw[i] & 0xffff0000u) : (pw[i] << 16));
      rb[h] = g * __uint_as_float(h ? (qw[i] & 0xffff0000u) : (qw[i] << 16));
    }
    oa[i] = pack_bf16x2(ra[0], ra[1]);
    ob[i] = pack_bf16x2(rb[0], rb[1]);
  }
  da = make_uint4(oa[0], oa[1], oa[2], oa[3]);
  db = make_uint4(ob[0], ob[1], ob[2], ob[3]);
}

// Short tiles.  A tile of fewer rows has less to multiply per stage and waits for its weights.  Its token parts are short, so the
// same LDS holds more stages of both operands: four up to 64 rows of a 256-row tile, three up to 128.  Measured on the loop of
// 32x32x16 MFMAs before this one, where every expert has a few rows and its weights are the work, d = 4096, 64 experts: 40 tokens
// 406 -> 373 us, 100 tokens 417 -> 381, 600 tokens 435 -> 401; unchanged where full tiles dominate.  (The backward products, bound by
// their transposing reads, gained nothing: 0.99 to 1.04 of the time.  Three stages up to 64 rows of a 128-row tile, ten layers, 33 to
// 400 tokens: 0.94 to 1.065 of the time, slower at d = 2048 with 24 experts and d = 4096 with 8.)
// Tall tiles of more than 128 rows: two stages of both operands (2 x 24 KB of tokens and 2 x 16 KB of weights).
template <typename GEO>
constexpr int short_depth(int mode, int nact) {
  if (GEO::BM == TallTile::BM && nact == 3) return 2;
  if (tr_b(mode)) return 0;
  if (GEO::BM == kBM) return nact == 1 ? 4 : nact == 2 ? 3 : 0;
  return 0;
}

// One tile with NACT active 32-row token fragments per wave (tile rows <= 64*NACT).
// phase clocks for the optional counters of the benchmark library (a.cycles)
#define PROBE_T(i) do { if (a.cycles) ts[i] = __builtin_amdgcn_s_memtime(); } while (0)

template <int MODE, int NACT, typename GEO>
__device__ __forceinline__ void run_tile(const TileArgs& a, const TileRec rec, unsigned char* lds,
                                         int lane, int w, int* signal = nullptr) {
  constexpr bool UP = is_up(MODE);
  constexpr bool TRA = tr_a(MODE), TRB = tr_b(MODE);   // operand read by transposing LDS reads
  constexpr bool WG = MODE == kWgrad;
  constexpr bool DH = MODE == kDgradH;
  // Operands as a wave-uniform base and 32-bit offsets per lane (64-bit pointers cost twice the registers): the weights of
  // the token modes, and their tokens where they are neighbouring rows (the up modes gather theirs through perm)
  constexpr bool OFFA = !WG && !UP;
  // (a value the compiler cannot trace, here and before the epilogue: what depends on the lane would be computed once before
  // the first tile and kept through every main loop, in registers that those do not have.  Its range is told again: divisions of
  // a number that may be negative are three times as long)
  asm volatile("" : "+v"(lane));
  lane &= 63;
  long long ts[6] = {0, 0, 0, 0, 0, 0};
  PROBE_T(0);
  constexpr int BM = GEO::BM, BN = GEO::BN, BK = kBK;
  static_assert(BM == BN || !TRA, "one part size for both operands");
  constexpr int WGM = GEO::WGM, WGN = GEO::WGN, NWAVES = WGM * WGN, NT = 64 * NWAVES;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int MF = WTM / 32;             // 32-row token blocks of a wave
  constexpr int CH = BK / 8, ROWB = BK * 2, RPL = 64 / CH, SH = 1;   // 8 chunks, 128-byte rows
  constexpr int KK = BK / 32;                                        // MFMA k-steps per stage
  constexpr int B_LOADS = BN * CH / NT;
  // wave-wide load j of the token part fills tile rows [64j, 64j+64): only NACT of them matter
  // (token-major operands: a part is 64 tokens x BM features, all of it is loaded)
  // (NACT active fragments per wave cover the tile rows [0, NACT * 32 * WGM))
  constexpr int A_LOADS = TRA ? BM * CH / NT : NACT * (32 * WGM / (NWAVES * RPL));
  static_assert((32 * WGM) % (NWAVES * RPL) == 0 && B_LOADS * NWAVES * RPL == BN, "whole wave-wide loads");
  constexpr int PART = BN * ROWB;                 // 32 (16) KB: one weight part, or a token part of as many rows
  // 16-row fragments: MT of the tokens (two per active block), NW of the weights
  constexpr int MT = 2 * NACT, NW = WTN / 16;
  static_assert(NACT >= 1 && NACT <= MF, "active token blocks");
  static_assert(KK == 2 && (!UP || NW % 2 == 0), "two k-steps a stage; gate and up halves per wave");
  // LDS map: token parts A0, A1 (two stages), then weight parts B0, B1, B2 (three stages).
  // Short tiles (see short_depth): DEPTH stages of both, the token parts only as long as the tile.
  constexpr int DEPTH = short_depth<GEO>(MODE, NACT);
  constexpr bool DEEP = DEPTH > 0;
  // Small tiles of the forward, whose few rows wait for weights from HBM: stage kt requests the weights of stage kt+3 instead of
  // kt+2.  128 experts, d = 1024, call of 34 tokens 145.9 -> 145.1 us, of 190 186.0 -> 184.8, of 1016 211.4 -> 209.2; the input
  // gradients do not gain (dH of 777 tokens, 32 experts, 21.9 -> 22.5).
  constexpr bool FAR = !DEEP && !TRB && BN < kBN;
  constexpr int APART = DEEP ? NACT * 32 * WGM * ROWB : PART, SLOTS = DEEP ? DEPTH : kStagesB;
  constexpr int BBASE = DEEP ? DEPTH * APART : kStagesA * PART;
  static_assert(BBASE + SLOTS * PART <= (kStagesA + kStagesB) * PART, "LDS of a workgroup");
  static_assert(DEEP || NACT * 32 * WGM * ROWB <= PART, "a stage's tokens fit their part");
  // (token part of stage kt, whose weights are in `slot`)
  auto a_part = [&](int stage, int slot) { return lds + (DEEP ? slot : stage & 1) * APART; };
  auto b_part = [&](int slot) { return lds + BBASE + slot * PART; };

  const int g = rec.e / a.N, e_i = rec.e % a.N, F = a.F[g];
  int K;
  int tok0 = 0, ntok = 0;       // kWgrad: the expert's routed rows [tok0, tok0 + ntok)
  if constexpr (WG) {
    tok0 = a.offsets[rec.e];
    ntok = a.offsets[rec.e + 1] - tok0;
    K = (ntok + BK - 1) / BK * BK;
    if (K < BK) K = BK;
  } else {
    K = red_d(MODE) ? a.d : F;
  }
  const int wm = w / WGN, wn = w % WGN;

  // ---- global source pointers of this thread's 16-byte chunks -------------------------
  // wave-wide load j fills tile rows (j*NWAVES + w)*RPL .. +RPL-1; lane l fills row l/CH,
  // physical chunk l%CH, which holds logical chunk (l%CH) ^ ((row >> SH) & (CH-1)).
  const int lrow = lane / CH, lpos = lane % CH;
  const uint16_t* src_a[TRA || OFFA ? 1 : A_LOADS];
  uint32_t off_a[OFFA ? A_LOADS : 1];             // (WG: the lane's part, the same for every load; so off_b)
  uint32_t off_b[TRB ? 1 : B_LOADS];
  const uint16_t* base_b = nullptr;               // not WG
  // OFFA: first row of wave-wide load j, and from there the lane's row (at most 7 further: offsets stay small)
  auto first_row = [&](int j) { return min((j * NWAVES + w) * RPL, rec.rows - 1); };
  // Operands stored reduction-index major (rows = reduction index, features contiguous): a part
  // holds 64 reduction rows x BN features, TRB_ROW = 512 (256) bytes a row.  Wave-wide load j fills
  // the TPL = 2 (4) rows from TPL*(j*NWAVES + w); lane l fills physical chunk l%TCH of row t = that +
  // l/TCH, which holds logical chunk (l%TCH) ^ (4*(t&3)) ^ (2*((t>>3)&1)): the eight rows that 32 lanes of a
  // transposing read touch at once (k0..k0+3 and k0+8..k0+11) then sit in different banks.
  constexpr int TRB_ROW = BN * 2, TCH = BN / 8, TPL = 1024 / TRB_ROW;
  static_assert(!(TRA || TRB) || (NWAVES * TPL % 16 == 0 && B_LOADS == BN * CH / NT), "part layout");
  // (trow0 <= 15: from there the offset of a row has 32 bits up to rows of 2^27 elements; the list of a backward call with rows of
  // 2^24 would fill the memory of the GPU)
  const int trow0 = TPL * w + lane / TCH;         // row of load 0; load j: + TPL*NWAVES*j
  const int tr_lc = (lane % TCH) ^ (4 * (trow0 & 3)) ^ (2 * ((trow0 >> 3) & 1));
  const uint16_t* zsrc = nullptr;
  unsigned tr_ldb = 0;                            // row pitch of the transposed weights in elements (input gradients)
  if constexpr (TRA) {
    int ma = rec.row_start + tr_lc * 8;
    // feature chunks past the matrix edge: any chunk inside the row (never stored)
    if (ma > a.Mrows[g] - 8) ma = a.Mrows[g] - 8;
    off_a[0] = ((uint32_t)trow0 * (uint32_t)a.lda + (uint32_t)ma) * 2u;
  }
  if constexpr (TRB) {
    int nb = rec.n0 + tr_lc * 8;
    if constexpr (WG) {
      if (nb > a.Ncols[g] - 8) nb = a.Ncols[g] - 8;
      zsrc = a.zero_row + (lane % TCH) * 8;
      off_b[0] = ((uint32_t)trow0 * (uint32_t)a.ldb + (uint32_t)nb) * 2u;
    } else if constexpr (DH) {
      if (nb > F - 8) nb = F - 8;                 // W_down[e]: [d, F]
      tr_ldb = a.ldw[g];
      base_b = a.W[g] + (long long)e_i * a.d * a.ldw[g];
      off_b[0] = (uint32_t)(trow0 * a.ldw[g] + nb) * 2u;
    } else {
      if (nb > a.d - 8) nb = a.d - 8;             // W13[e]: [2F, d]; F holds 2 F_g here
      tr_ldb = a.ldw[g];
      base_b = a.W[g] + (long long)e_i * F * a.ldw[g];
      off_b[0] = (uint32_t)(trow0 * a.ldw[g] + nb) * 2u;
    }
  }
#pragma unroll
  for (int j = 0; j < (TRA ? 0 : A_LOADS); ++j) {
    const int row = (j * NWAVES + w) * RPL + lrow;
    const int rr = row < rec.rows ? row : rec.rows - 1;     // rows past the end: any valid row
    const int pos = rec.row_start + rr;
    long long src_row;
    if constexpr (UP) src_row = a.perm ? (long long)(a.perm[pos] / a.Ke) : (long long)pos;
    else src_row = pos;
    const int chunk = lpos ^ ((row >> SH) & (CH - 1));
    if constexpr (OFFA) off_a[j] = ((uint32_t)(rr - first_row(j)) * (uint32_t)a.lda + chunk * 8) * 2u;
    else src_a[j] = a.A + src_row * a.lda + chunk * 8;
  }
  // plain weights: row n0 of the tile's matrix; up modes: W_up is F rows further, and a wave-wide load holds rows of one of them
  static_assert(!UP || (BN / 2) % (NWAVES * RPL) == 0, "loads of one half");
  const int ncols_b = UP ? F : a.d;
  // LONG: first row of wave-wide load j in its half, and from there the lane's row (at most 7 further)
  auto first_row_b = [&](int j) { return min((j * NWAVES + w) * RPL % (UP ? BN / 2 : BN), ncols_b - 1 - rec.n0); };
  if constexpr (!TRB) base_b = a.W[g] + ((long long)e_i * (UP ? 2 : 1) * ncols_b + rec.n0) * a.ldw[g];
#pragma unroll
  for (int j = 0; j < (TRB ? 0 : B_LOADS); ++j) {
    const int row = (j * NWAVES + w) * RPL + lrow;
    const int chunk = lpos ^ ((row >> SH) & (CH - 1));
    // the row of the tile's weights, from the first one of its half (up modes: [0, BN/2) W_gate rows n0.., the rest W_up rows)
    int r = UP ? row % (BN / 2) : row;
    if (rec.n0 + r > ncols_b - 1) r = ncols_b - 1 - rec.n0;
    if constexpr (GEO::LONG) r -= first_row_b(j);
    off_b[j] = ((uint32_t)r * (uint32_t)a.ldw[g] + chunk * 8) * 2u;
  }
  const int ld_off = w * 1024;      // + j * NWAVES * 1024: wave-uniform destination inside a part

  f32x4 acc[NW][MT];
#pragma unroll
  for (int fi = 0; fi < NW; ++fi)
#pragma unroll
    for (int ti = 0; ti < MT; ++ti)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[fi][ti][r] = 0.f;

  const int KT = K / BK;
  // reduction-major operands: load j of a stage starts TPL*NWAVES*j rows further down.  In kWgrad the rows are routed tokens;
  // in the expert's last stage those at or past its count read the zero row instead (ENDS: the stage may be that one; without,
  // every lane's row is there, and what the choice costs per load, a branch among the MFMAs, is saved)
  auto wg_copy = [&](const uint16_t* base, unsigned ld, uint32_t off, int stage, int j, int to, auto ENDS) {
    const int t = stage * BK + TPL * NWAVES * j;    // row of this load, less trow0
    // wave-uniform 32 x 32 -> 64 bit product: stays in scalar registers
    const uint16_t* p = base + (unsigned long long)(unsigned)(tok0 + t) * ld;
    if constexpr (decltype(ENDS)::value) {
      const uint16_t* row = reinterpret_cast<const uint16_t*>(reinterpret_cast<const unsigned char*>(p) + off);
      asm("" : "+v"(row));          // (computed in every lane: as a branch per load it waits for its scalar operands each time)
      async_copy16(t + trow0 < ntok ? row : zsrc, to);
    } else {
      async_copy16(p, off, to);
    }
  };
  const int lds0 = lds_address(lds);
  auto issue_a = [&](int stage, int slot, int j, auto ENDS) {
    const int to = lds0 + (int)(a_part(stage, slot) - lds) + j * NWAVES * 1024 + ld_off;
    if constexpr (OFFA) {
      const uint16_t* base = a.A + (unsigned long long)(unsigned)(rec.row_start + first_row(j)) * (unsigned)a.lda;
      async_copy16(base + stage * BK, off_a[j], to);
    } else if constexpr (TRA) {
      wg_copy(a.A, a.lda, off_a[0], stage, j, to, ENDS);
    } else {
      async_copy16(src_a[j] + stage * BK, to);
    }
  };
  auto issue_b = [&](int stage, int slot, int j, auto ENDS) {
    const int to = lds0 + (int)(b_part(slot) - lds) + j * NWAVES * 1024 + ld_off;
    if constexpr (WG) {
      wg_copy(a.B2, a.ldb, off_b[0], stage, j, to, ENDS);
    } else if constexpr (TRB) {
      const unsigned t = stage * BK + TPL * NWAVES * j;           // row of this load, less trow0
      async_copy16(base_b + (unsigned long long)t * tr_ldb, off_b[0], to);
    } else {
      long long first = UP && j * NWAVES * RPL >= BN / 2 ? (long long)F * a.ldw[g] : 0;
      if constexpr (GEO::LONG) first += (long long)first_row_b(j) * a.ldw[g];
      async_copy16(base_b + first + stage * BK, off_b[j], to);
    }
  };

  // prologue: request the first two stages (DEEP: DEPTH of them, as far as they exist; FAR: the weights of a third), wait for
  // the first, read its first fragments
  using Ends = std::true_type;
  constexpr int AHEAD = DEEP ? DEPTH : 2;
  PROBE_T(1);
  __syncthreads();                  // the previous tile's epilogue has left the LDS
#pragma unroll
  for (int st = 0; st < AHEAD; ++st)
    if (st < KT) {
#pragma unroll
      for (int j = 0; j < B_LOADS; ++j) issue_b(st, st, j, Ends{});
#pragma unroll
      for (int j = 0; j < A_LOADS; ++j) issue_a(st, st, j, Ends{});
    }
  if (FAR && KT > 2) {
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) issue_b(2, 2, j, Ends{});
  }

  // ---- LDS offsets of the MFMA operand fragments ---------------------------------------
  // fragment row = base + lane%16, logical chunk = 4*kk + lane/16
  // Reduction-major parts: the transposing read works on groups of 16 lanes.  Lane 4*a + b of a
  // group passes the address of 4 features (8 bytes) of row k0 + a at feature m0 + 4*b and
  // gets back rows k0..k0+3 of feature m0 + (its index in the group).  Group q of the wave
  // covers the fragment's 16 features and rows 8*q.. of the k-step, so two
  // reads (k0, k0 + 4) give a lane its 8 consecutive reduction indices of one fragment row.
  const int frow = lane & 15, fh = lane >> 4;
  const int ta = (lane & 15) >> 2, tb = lane & 3;
  int foff[KK], foff_t[KK];       // plain parts / reduction-major parts (only one is live
                                  // unless the two operands differ)
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    foff_t[kk] = (32 * kk + 8 * fh + ta) * TRB_ROW + (tb >> 1) * 16 + (tb & 1) * 8;
    foff[kk] = frow * ROWB + (((4 * kk + fh) ^ ((frow >> SH) & (CH - 1))) << 4);
  }
  // first feature of a fragment -> its 16-byte chunk, swizzled like the loads wrote it
  auto tr_base = [&](int feat) { return (((feat >> 3) ^ (4 * ta) ^ (2 * (fh & 1))) << 4); };
  int fbase_a[MT], fbase_b[NW];   // token fragments (32-row blocks interleaved over the wave rows), weight fragments
#pragma unroll
  for (int ti = 0; ti < MT; ++ti) {
    const int row = ((ti >> 1) * WGM + wm) * 32 + (ti & 1) * 16;
    fbase_a[ti] = TRA ? tr_base(row) : row * ROWB;
  }
#pragma unroll
  for (int fi = 0; fi < NW; ++fi) {
    int row;
    if constexpr (UP) {
      constexpr int NWh = NW / 2;
      row = (fi < NWh) ? wn * (WTN / 2) + fi * 16 : BN / 2 + wn * (WTN / 2) + (fi - NWh) * 16;
    } else {
      row = wn * WTN + fi * 16;
    }
    fbase_b[fi] = TRB ? tr_base(row) : row * ROWB;
  }
  // (They are worked out here, under the wait for the first stage.  Placed by the compiler, they stood between its arrival and the
  // first products: a weight-gradient tile of one stage took 2400 clocks for those, now 2130.)
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    if constexpr (TRA || TRB) asm volatile("" : "+v"(foff_t[kk]));
    if constexpr (!TRA || !TRB) asm volatile("" : "+v"(foff[kk]));
  }
  if constexpr (TRA)
#pragma unroll
    for (int ti = 0; ti < MT; ++ti) asm volatile("" : "+v"(fbase_a[ti]));
  if constexpr (TRB)
#pragma unroll
    for (int fi = 0; fi < NW; ++fi) asm volatile("" : "+v"(fbase_b[fi]));
  // a fragment at p: plain, or two transposing reads
  auto read_frag = [&](const unsigned char* p, auto TR) {
    if constexpr (decltype(TR)::value) {
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * TRB_ROW));
      const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8, v);
    } else {
      return *reinterpret_cast<const bf16x8*>(p);
    }
  };
  auto read_a = [&](const unsigned char* pa, int kk, int ti) {
    return read_frag(pa + fbase_a[ti] + (TRA ? foff_t[kk] : foff[kk]), std::integral_constant<bool, TRA>{});
  };
  auto read_b = [&](const unsigned char* pb, int kk, int fi) {
    return read_frag(pb + fbase_b[fi] + (TRB ? foff_t[kk] : foff[kk]), std::integral_constant<bool, TRB>{});
  };
  if (FAR && KT > 2) wait_vmcnt<A_LOADS + 2 * B_LOADS>();
  else if (KT >= AHEAD) wait_vmcnt<(AHEAD - 1) * (A_LOADS + B_LOADS)>();
  else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  MOHGE_PIN();
  // Fused launches: the counter of the row block that this workgroup's PREVIOUS tile completed.
  // Vector memory operations of a wave complete in issue order, so a wave whose first-stage loads
  // have landed has seen all its earlier stores complete, and the barrier above makes that true
  // of every wave: the previous tile's rows are in memory.  (Waiting for those stores at the end of
  // the previous tile instead cost a memory round trip with nothing to overlap it.)
  if (signal != nullptr && threadIdx.x == 0)
    __hip_atomic_fetch_add(signal, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  PROBE_T(2);
  // Registers of the main loop: the weight fragments of a k-step and those of the next one, and a ring of RA token
  // fragments.  A group is one token fragment times all weight fragments, MT groups a k-step, 2 MT a stage; after
  // group G its register takes the token fragment of group G + RA.
  constexpr int RA = MT < 4 ? 4 : MT, NG = KK * MT;
  static_assert(NG % RA == 0, "a ring position per group of a stage");
  bf16x8 fa[RA], fb[KK][NW];
  __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0): with scalar loads among the LDS reads they could not be counted below
#pragma unroll
  for (int fi = 0; fi < NW; ++fi) fb[0][fi] = read_b(b_part(0), 0, fi);
#pragma unroll
  for (int i = 0; i < RA; ++i) fa[i] = read_a(a_part(0, 0), i / MT, i % MT);

  // Stage kt: token part kt&1, weight slot `slot` = kt%3.  Its groups [0, GB) run before the one barrier of the stage,
  // and under them everything that is still to be read of the stage: the second k-step's weight fragments and the token
  // fragments of groups RA and up.  The reads end GB - (NG - RA) groups ahead of the barrier, which they need to arrive.
  // From the barrier on nobody reads the stage's LDS parts again.  Stage kt requests stage kt+2: the weights under the groups
  // before the barrier, into the slot that stage kt-1 left (so all but the newest B_LOADS requests having landed certifies
  // stage kt+1 at the barrier), the tokens under the groups after it, into the stage's own part.  The requests are spread
  // over the MFMAs: a compute unit takes about 57 bytes a clock of them, a stage's 64 KB in 1150 clocks, and a wave
  // whose request finds the queue full issues nothing else (all of them behind the barrier, with the first fragments of stage
  // kt+1, which are read there as well: 2520 clocks a stage of 256 x 256 at d = 4096, 2080 without LDS reads or
  // requests, 2220 with the reads, 2400 with the requests alone).
  constexpr int GB = NG - RA + (MT == 8 ? (WG ? 2 : 3) : MT == 6 ? 2 : MT == 4 ? 1 : 2);
  static_assert(GB > NG - RA && 2 * GB >= NW, "a stage's reads are issued before its barrier");
  int slot = 0;
  // DEEP: both parts of stage kt+DEPTH are requested after the barrier, LATER stages past kt+1 may be in flight at the
  // barrier.
  // FAR: after the barrier the tokens of stage kt+2, then (FARB: it exists) the weights of stage kt+3 into the stage's own slot;
  // at the barrier those of stage kt+2, requested a stage earlier, may be in flight.
  auto stage = [&](int kt, auto REQ, auto LAST, auto LATER, auto ENDS, auto FARB) {
    // req: stage kt+AHEAD exists and is requested (ENDS: it may be the last); last: no stage kt+1
    constexpr bool req = decltype(REQ)::value, last = decltype(LAST)::value;
    constexpr bool farb = FAR && decltype(FARB)::value;
    const unsigned char* pa = a_part(kt, slot);
    const unsigned char* pb = b_part(slot);
    const int slot1 = slot == SLOTS - 1 ? 0 : slot + 1;        // stage kt+1
    const int slot2 = slot1 == SLOTS - 1 ? 0 : slot1 + 1;      // stage kt+2
    const unsigned char* pa1 = a_part(kt + 1, slot1);
    const unsigned char* pb1 = b_part(slot1);
    constexpr int NPRE = req && !DEEP && !FAR ? B_LOADS : 0;                          // requests before the barrier
    constexpr int NPOST = req ? (DEEP || farb ? A_LOADS + B_LOADS : A_LOADS) : 0;     // and after it
    constexpr int NP = (NG - GB) * NW;                 // MFMAs after the barrier
    constexpr int NOLD = GB - (NG - RA);               // token fragments of stage kt+1 whose register is free at the barrier
    static_assert(NW + NOLD <= NP, "a read per MFMA");
    // x-th read after the barrier: weight fragment 0, those token fragments and the other weight fragments of stage kt+1
    auto ahead = [&](int x) {
      if (x == 0) fb[0][0] = read_b(pb1, 0, 0);
      else if (x == 1) fa[(NG - RA) % RA] = read_a(pa1, 0, 0);
      else if (x <= NW) fb[0][x - 1] = read_b(pb1, 0, x - 1);
      else fa[(NG - RA + x - NW) % RA] = read_a(pa1, (x - NW) / MT, (x - NW) % MT);
    };
    // the register of group G takes the token fragment of group G + RA
    auto refill = [&](int G) {
      const int nx = G + RA;
      if (nx < NG) fa[G % RA] = read_a(pa, nx / MT, nx % MT);
      else if (!last && G >= GB) fa[G % RA] = read_a(pa1, (nx - NG) / MT, (nx - NG) % MT);
      MOHGE_PIN();
    };
#pragma unroll
    for (int G = 0; G < NG; ++G) {
      const int kk = G / MT, ti = G % MT;
      if (!last && G == GB) {
        // my reads of this stage are complete; my requests for stage kt+1 have landed
        if constexpr (DEEP)
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(decltype(LATER)::value * (A_LOADS + B_LOADS)) : "memory");
        else
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(FAR && req ? B_LOADS : NPRE) : "memory");
        __builtin_amdgcn_s_barrier();
        MOHGE_PIN();
      }
#pragma unroll
      for (int fi = 0; fi < NW; ++fi) {
        // to and fro over the weight fragments: every MFMA shares an operand with the one before it, which saves power (all of
        // them the same way 1860 TFLOP/s with the operand reads from LDS and nothing else, to and fro 1897)
        const int fw = G & 1 ? NW - 1 - fi : fi;
        acc[fw][ti] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[kk][fw], fa[G % RA], acc[fw][ti], 0, 0, 0);
        MOHGE_PIN();
        // (one MFMA later: the register is the third operand's of the last one as often as not, and that is still being read)
        if (fi == 0 && G > 0) refill(G - 1);
        // second k-step's weight fragments, two under each of the first groups
        if (G < (NW + 1) / 2 && fi < 2 && 2 * G + fi < NW) {
          fb[1][2 * G + fi] = read_b(pb, 1, 2 * G + fi);
          MOHGE_PIN();
        }
        if (G < GB) {
          const int m = G * NW + fi;                   // this MFMA among the GB * NW before the barrier
#pragma unroll
          for (int j = 0; j < NPRE; ++j)
            if (m == (2 * j + 1) * GB * NW / (2 * (NPRE > 0 ? NPRE : 1))) {
              issue_b(kt + 2, slot2, j, ENDS);
              MOHGE_PIN();
            }
        } else if (!last) {
          const int m = (G - GB) * NW + fi;
          if (m < NW + NOLD) {
            ahead(m);
            MOHGE_PIN();
          }
#pragma unroll
          for (int j = 0; j < NPOST; ++j)
            if (m == (2 * j + 1) * NP / (2 * (NPOST > 0 ? NPOST : 1))) {
              if (j < A_LOADS) issue_a(kt + AHEAD, slot, j, ENDS);
              else issue_b(kt + (FAR ? 3 : AHEAD), slot, j - A_LOADS, ENDS);
              MOHGE_PIN();
            }
        }
      }
    }
    refill(NG - 1);
    slot = slot1;
  };

  {
    using T = std::true_type;
    using Fa = std::false_type;
    using I0 = std::integral_constant<int, 0>;
    int kt = 0;
    if constexpr (DEEP) {
      for (; kt + DEPTH < KT; ++kt) stage(kt, T{}, Fa{}, std::integral_constant<int, DEPTH - 2>{}, Fa{}, Fa{});
      if constexpr (DEPTH == 4)
        if (kt + 3 < KT) { stage(kt, Fa{}, Fa{}, std::integral_constant<int, 2>{}, Fa{}, Fa{}); ++kt; }
      if constexpr (DEPTH >= 3)
        if (kt + 2 < KT) { stage(kt, Fa{}, Fa{}, std::integral_constant<int, 1>{}, Fa{}, Fa{}); ++kt; }
    } else if constexpr (FAR) {
      for (; kt + 3 < KT; ++kt) stage(kt, T{}, Fa{}, I0{}, Fa{}, T{});
      if (kt + 2 < KT) { stage(kt, T{}, Fa{}, I0{}, Fa{}, Fa{}); ++kt; }
    } else {
      for (; kt + 2 + WG < KT; ++kt) stage(kt, T{}, Fa{}, I0{}, Fa{}, Fa{});
      if constexpr (WG)
        if (kt + 2 < KT) { stage(kt, T{}, Fa{}, I0{}, T{}, Fa{}); ++kt; }
    }
    if (kt + 1 < KT) { stage(kt, Fa{}, Fa{}, I0{}, Fa{}, Fa{}); ++kt; }
    stage(kt, Fa{}, T{}, I0{}, Fa{}, Fa{});
  }
  PROBE_T(3);

  // ---- epilogue: accumulators -> bf16 -> a wave-private LDS patch -> 16-byte stores ------
  // A lane holds, per 16x16 block, token lane%16 and weight rows 4*(lane/16) + r:
  // 4 consecutive output features.  Every wave transposes its part through
  // LDS (row stride padded by 16 bytes against bank conflicts) and stores row segments.
  __syncthreads();                     // all waves are done reading the stages
  {
    constexpr int OC = UP ? WTN / 2 : WTN;           // output features of this wave
    constexpr int RS = OC * 2 + 16;                  // LDS row stride in bytes
    constexpr int EPI_BYTES = 32 * RS;               // one 32-token fragment at a time
    constexpr int CPR = OC * 2 / 16;                 // 16-byte chunks per row
    constexpr int NFo = UP ? NW / 2 : NW;
    static_assert(NWAVES * EPI_BYTES <= (kStagesA + kStagesB) * PART, "epilogue patch must fit the stage buffers");
    static_assert(32 * CPR % 64 == 0, "whole wave-wide copies");
    unsigned char* my = lds + w * EPI_BYTES;
    asm volatile("" : "+v"(lane));
    lane &= 63;
    const int tok_l = lane & 15, fsub = (lane >> 4) * 4;
    const int ncols = red_d(MODE) ? F : (WG ? a.Ncols[g] : a.d);
    const int col0 = rec.n0 + wn * OC;
    // kWgrad: first row of the tile in the expert's gradient
    uint16_t* wout = nullptr;
    if constexpr (WG) wout = a.Wout[g] + ((long long)e_i * a.Mrows[g] + rec.row_start) * ncols;
    // kUpSave makes three passes over the patch: h, then the backward factors p and q
    constexpr int NPASS = MODE == kUpSave ? 3 : 1;
    constexpr int NIT = 32 * CPR / 64;     // row-segment copies per lane and fragment
    // kDgradH: the stored factor chunks a lane will meet in the copy loop are requested before
    // the transposition through LDS (rows / columns past the tile edge: any valid chunk)
    auto load_pre = [&](int ti, uint4 (&pa)[NIT], uint4 (&pb)[NIT]) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int idx = it * 64 + lane;
        int trow = (ti * WGM + wm) * 32 + idx / CPR, col = col0 + (idx % CPR) * 8;
        if (trow > rec.rows - 1) trow = rec.rows - 1;
        if (col > ncols - 8) col = ncols - 8;
        const long long at = (long long)(rec.row_start + trow) * a.ldpre + col;
        pa[it] = *reinterpret_cast<const uint4*>(a.pre + at);
        pb[it] = *reinterpret_cast<const uint4*>(a.pre + at + F);
      }
    };
#pragma unroll
    for (int ti = 0; ti < NACT; ++ti) {
      uint4 pre_a[DH ? NIT : 1], pre_b[DH ? NIT : 1];
      if constexpr (DH) load_pre(ti, pre_a, pre_b);
      // kUpSave: the two factors the backward pass multiplies dh with, computed along with h
      // (one sigmoid per element) and kept packed until their pass
      uint2 keep_p[MODE == kUpSave ? NFo * 2 : 1], keep_q[MODE == kUpSave ? NFo * 2 : 1];
#pragma unroll
      for (int pass = 0; pass < NPASS; ++pass) {
#pragma unroll
        for (int fi = 0; fi < NFo; ++fi)
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const int t16 = 2 * ti + hh;
            uint2 o;
            if (MODE == kUpSave && pass > 0) {
              o = pass == 1 ? keep_p[fi * 2 + hh] : keep_q[fi * 2 + hh];
            } else {
              float v[4], vp[4], vq[4];
#pragma unroll
              for (int b = 0; b < 4; ++b) {
                if constexpr (MODE == kUpSave) {
                  const float ga = acc[fi][t16][b], ub = acc[fi + NW / 2][t16][b];
                  const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-ga));
                  vq[b] = ga * sg;                                   // SiLU(a)
                  v[b] = ga * ub * sg;                               // h, rounded as in kUp
                  vp[b] = ub * sg * (1.f + ga * (1.f - sg));         // b * SiLU'(a)
                } else if constexpr (UP) {
                  v[b] = swiglu(acc[fi][t16][b], acc[fi + NW / 2][t16][b]);
                } else {
                  v[b] = acc[fi][t16][b];
                }
              }
              o.x = pack_bf16x2(v[0], v[1]);
              o.y = pack_bf16x2(v[2], v[3]);
              if constexpr (MODE == kUpSave) {
                keep_p[fi * 2 + hh] = make_uint2(pack_bf16x2(vp[0], vp[1]), pack_bf16x2(vp[2], vp[3]));
                keep_q[fi * 2 + hh] = make_uint2(pack_bf16x2(vq[0], vq[1]), pack_bf16x2(vq[2], vq[3]));
              }
            }
            *reinterpret_cast<uint2*>(my + (hh * 16 + tok_l) * RS + (fi * 16 + fsub) * 2) = o;
          }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int idx = it * 64 + lane;
          const int row = idx / CPR, c = idx % CPR;
          const uint4 v = *reinterpret_cast<const uint4*>(my + row * RS + c * 16);
          const int trow = (ti * WGM + wm) * 32 + row;
          const int col = col0 + c * 8;
          if (trow < rec.rows && col < ncols) {
            if constexpr (WG) {
              *reinterpret_cast<uint4*>(wout + (unsigned long long)(unsigned)trow * (unsigned)ncols + col) = v;
            } else if constexpr (DH) {
              // v holds dh; the stored factors turn it into the gradients of the pre-activations
              const long long at = (long long)(rec.row_start + trow) * a.ldpre + col;
              uint4 da, db;
              swiglu_bwd8(v, pre_a[it], pre_b[it], da, db);
              if (a.coherent_out) {
                store16_device_scope(a.C2 + at, da);
                store16_device_scope(a.C2 + at + F, db);
              } else {
                *reinterpret_cast<uint4*>(a.C2 + at) = da;
                *reinterpret_cast<uint4*>(a.C2 + at + F) = db;
              }
            } else if (pass == 0) {
              uint16_t* dst = a.C + (long long)(rec.row_start + trow) * a.ldc + col;
              if (UP && a.coherent_out) store16_device_scope(dst, v);
              else *reinterpret_cast<uint4*>(dst) = v;
            } else {
              const long long at = (long long)(rec.row_start + trow) * a.ldpre + (pass == 2 ? F : 0) + col;
              *reinterpret_cast<uint4*>(a.pre + at) = v;
            }
          }
        }
      }
    }
  }
  PROBE_T(4);
  if (a.cycles && threadIdx.x == 0) {
    // setup, wait for the first stages, main loop, epilogue; tiles; stages
    long long* d = a.cycles + (size_t)blockIdx.x * 8;
    for (int i = 0; i < 4; ++i) d[i] += ts[i + 1] - ts[i];
    d[4] += 1;
    d[5] += KT;
  }
}

// The instantiation of run_tile for the tile's row count: a wave's k-th fragment serves the tile
// rows [32 * WGM * k, 32 * WGM * (k + 1)) together with the other wave rows.
template <int MODE, typename GEO = BigTile>
__device__ __forceinline__ void run_tile_rows(const TileArgs& a, const TileRec& rec, unsigned char* lds, int lane,
                                              int w, int* signal) {
  constexpr int UNIT = 32 * GEO::WGM, MF = GEO::BM / UNIT;
  static_assert(MF >= 2 && MF <= 4, "two to four token fragments per wave");
  const int nact = (rec.rows + UNIT - 1) / UNIT;
  if constexpr (MF == 4)
    if (nact == 4) { run_tile<MODE, 4, GEO>(a, rec, lds, lane, w, signal); return; }
  if constexpr (MF >= 3)
    if (nact == 3) { run_tile<MODE, 3, GEO>(a, rec, lds, lane, w, signal); return; }
  if (nact >= 2) run_tile<MODE, 2, GEO>(a, rec, lds, lane, w, signal);
  else run_tile<MODE, 1, GEO>(a, rec, lds, lane, w, signal);
}

// Persistent tile kernel: workgroup b serves XCD b % 8.  Its first tile is fixed (range start
// + b / 8); further tiles are handed out by an atomic counter per range, so a workgroup that
// drew cheap tiles simply takes more of them.  The counter is read one tile ahead (the
// atomic's latency hides behind the tile) and the result is passed to the other waves
// through one LDS word between the tiles.  Which workgroup computes a tile has no influence
// on the tile's result, so the output stays bit-identical from run to run.
template <int MODE, typename GEO = BigTile>
__global__ void __launch_bounds__(Shape<MODE>::THREADS) ffn_tile_kernel(const TileArgs a) {
  extern __shared__ __align__(1024) unsigned char lds[];
  // LDS word for the hand-over: beyond the epilogue patches, inside a stage buffer that is
  // dead between a tile's last barrier and the first barrier of the next tile
  constexpr int kBcastOffset = kHandoverOffset;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  int tbeg = a.hdr->xcd_begin[xcd], tend = a.hdr->xcd_begin[xcd + 1];
  const int total = a.hdr->total;
  if (tbeg < 0) tbeg = 0;
  if (tend > total) tend = total;
  int t = tbeg + slot;
  while (t < tend) {
    int t_next = 0;
    if (threadIdx.x == 0) t_next = tbeg + atomicAdd(&a.hdr->counters[xcd], 1);
    TileRec rec = a.recs[t];
    rec.e = __builtin_amdgcn_readfirstlane(rec.e);
    rec.row_start = __builtin_amdgcn_readfirstlane(rec.row_start);
    rec.rows = __builtin_amdgcn_readfirstlane(rec.rows);
    rec.n0 = __builtin_amdgcn_readfirstlane(rec.n0);
    // a record that does not describe rows of this call would mean a corrupted schedule:
    // skip it rather than touch memory through it
    bool ok = !(rec.e < 0 || rec.e >= a.Ne || rec.rows < 1 || rec.rows > kBM ||
                rec.row_start < 0 || rec.n0 < 0);
    if (ok) {
      if constexpr (MODE == kWgrad) {
        ok = rec.row_start + rec.rows <= a.Mrows[rec.e / a.N] && rec.n0 < a.Ncols[rec.e / a.N] &&
             a.zero_row != nullptr && a.offsets[rec.e] >= 0 && a.offsets[rec.e + 1] <= a.P &&
             a.offsets[rec.e] <= a.offsets[rec.e + 1];
      } else {
        ok = rec.row_start + rec.rows <= a.P;
      }
    }
    if (ok) {
      run_tile_rows<MODE, GEO>(a, rec, lds, lane, w, nullptr);
    }
    __syncthreads();       // every wave is past its epilogue (and past reading the old word)
    if (threadIdx.x == 0) *reinterpret_cast<volatile int*>(lds + kBcastOffset) = t_next;
    __syncthreads();
    t = __builtin_amdgcn_readfirstlane(*reinterpret_cast<volatile int*>(lds + kBcastOffset));
  }
}

// Fused forward: the up tiles and the down tiles of a layer call in one persistent launch.
// Workgroup b serves XCD b % 8: first the up tiles of that XCD's range of the up list, then the
// down tiles of its range of the down list, each range with its own hand-out counter as in
// ffn_tile_kernel.  A down tile reads the H rows of one (expert, row block), which the up tiles
// of that row block write: every finished up tile adds one to the row block's counter
// (fam_done), a down tile waits until the counter has reached the number of up tiles of the
// block.  What makes the hand-over sound on any XCD:
//  * H is stored at device scope (coherent_out), and every wave waits for its stores (vmcnt)
//    before the workgroup barrier that precedes the counter increment;
//  * the consumer reads the counter at device scope and reads H only after that; no cache on
//    its path can hold an older copy of these lines, since nothing reads H rows of a row block
//    in this launch before the block's counter is complete, and launch boundaries invalidate
//    the caches.
// Waiting cannot deadlock: tiles are handed out in list order, all up tiles of an XCD come
// before its down tiles, and an up tile never waits for anything; a down tile whose row block
// belongs to another XCD's range waits for tiles that were handed out there before any of
// that XCD's down tiles.  The wait is bounded all the same (kSpinLimit polls, about a second);
// if it ever expires the tile is computed regardless and a flag is left in the header of the
// waiting list, which mohge_fused_status reports.  A negative limit (test hook: mohge_ffn_options.spin_limit) makes every dependent tile give up without looking.
constexpr int kSpinLimit = 1 << 22;

// Output region of a tile of a token mode (rows x 256 columns of C) filled with bf16 NaNs.
__device__ __forceinline__ void poison_tile(const TileArgs& a, const TileRec& rec) {
  if (a.C == nullptr) return;
  const int ncols = min(kBN, a.ldc - rec.n0);
  for (int i = threadIdx.x; i < rec.rows * (kBN / 2); i += blockDim.x) {
    const int r = i / (kBN / 2), c = (i % (kBN / 2)) * 2;
    if (c < ncols)
      *reinterpret_cast<uint32_t*>(a.C + (long long)(rec.row_start + r) * a.ldc + rec.n0 + c) = 0x7FC07FC0u;
  }
}

// One phase of a fused launch: the tiles of one list in MODE.  ROLE 1: producer (every finished
// tile adds one to its row block's counter; the range's straddling tail goes first), ROLE 2:
// consumer (a tile waits until its row block's counter has reached rec.need), ROLE 0: neither.
template <int MODE, int ROLE>
__device__ __forceinline__ void fused_phase(const TileArgs& a, unsigned char* lds, int lane, int w) {
  constexpr int PHASE = ROLE == 1 ? 0 : 1;
  constexpr int kBcastOffset = kHandoverOffset;
  const int home = blockIdx.x % kXcds;
  const int total = a.hdr->total;
  // The counter of a range hands out positions 0, 1, 2, ...  Up phase: the positions map to the
  // range's tail first (tiles of an expert that continues in the next XCD's range: down tiles of
  // both ranges wait for them), then to the rest in list order.  Down phase: list order, the order
  // in which the up tiles they depend on were handed out.
  // A workgroup serves its own XCD's range until the counter runs past its end and then (steal)
  // whichever other range still has tiles, so the launch ends when all tiles are done rather than
  // when the slowest range is.  (The number of rounds is bounded for form's sake: every round but
  // the last exhausts a range, and counters only grow.)  A stolen tile is an ordinary draw from that range's counter, so the
  // argument about waiting below holds for it as well.
  int* pending = nullptr;      // ROLE 1: counter of the row block of the tile just finished, not yet added to
  int cur = home;
  for (int round = 0; round <= 4 * kXcds; ++round) {
    if (round > 0) {
      // Own range exhausted: look at the counters of all other ranges at once (one memory round
      // trip: looking at them one after the other cost a round trip each at the moment when the
      // workgroup has nothing to do, 15-30 us where the whole launch takes 230) and go to the first
      // one, in ring order, that still has tiles.  (A counter is looked at before it is drawn
      // from, so that an exhausted one is left alone.)
      // (only where a compute unit sees several tiles of this list: with fewer, what a stolen tile
      // saves at the end does not pay for fetching its operands into another XCD's L2)
      if (!(a.steal & (PHASE == 0 ? 1 : 2)) || total < 4 * a.ncu) break;
      __syncthreads();
      if (threadIdx.x == 0) {
        int c[kXcds];
#pragma unroll
        for (int x = 0; x < kXcds; ++x)
          c[x] = __hip_atomic_load(&a.hdr->counters[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int pick = -1;
#pragma unroll
        for (int k = kXcds - 1; k >= 1; --k) {
          const int x = (home + k) % kXcds;
          int b = a.hdr->xcd_begin[x], e = a.hdr->xcd_begin[x + 1];
          if (b < 0) b = 0;
          if (e > total) e = total;
          int cx = 0;
#pragma unroll
          for (int y = 0; y < kXcds; ++y) cx = y == x ? c[y] : cx;
          if (cx < e - b) pick = x;
        }
        *reinterpret_cast<volatile int*>(lds + kBcastOffset) = pick;
      }
      __syncthreads();
      cur = __builtin_amdgcn_readfirstlane(*reinterpret_cast<volatile int*>(lds + kBcastOffset));
      if (cur < 0 || cur >= kXcds) break;
    }
    int tbeg = a.hdr->xcd_begin[cur], tend = a.hdr->xcd_begin[cur + 1];
    if (tbeg < 0) tbeg = 0;
    if (tend > total) tend = total;
    const int n = tend - tbeg;
    int ntail = PHASE == 0 ? a.hdr->tail[cur] : 0;
    ntail = ntail < 0 ? 0 : (ntail > n ? n : ntail);
    __syncthreads();         // everybody has read the last hand-over word
    if (threadIdx.x == 0) *reinterpret_cast<volatile int*>(lds + kBcastOffset) = atomicAdd(&a.hdr->counters[cur], 1);
    __syncthreads();
    int pos = __builtin_amdgcn_readfirstlane(*reinterpret_cast<volatile int*>(lds + kBcastOffset));
    while (pos >= 0 && pos < n) {
      const int t = pos < ntail ? tend - ntail + pos : tbeg + (pos - ntail);
      int t_next = 0;
      if (threadIdx.x == 0) t_next = atomicAdd(&a.hdr->counters[cur], 1);
      TileRec rec = a.recs[t];
      rec.e = __builtin_amdgcn_readfirstlane(rec.e);
      rec.row_start = __builtin_amdgcn_readfirstlane(rec.row_start);
      rec.rows = __builtin_amdgcn_readfirstlane(rec.rows);
      rec.n0 = __builtin_amdgcn_readfirstlane(rec.n0);
      rec.fam = __builtin_amdgcn_readfirstlane(rec.fam);
      rec.need = __builtin_amdgcn_readfirstlane(rec.need);
      bool ok = !(rec.e < 0 || rec.e >= a.Ne || rec.rows < 1 || rec.rows > kBM || rec.row_start < 0 ||
                  rec.n0 < 0 || rec.fam < 0);
      if (ok) {
        if constexpr (MODE == kWgrad) {
          ok = rec.row_start + rec.rows <= a.Mrows[rec.e / a.N] && rec.n0 < a.Ncols[rec.e / a.N] &&
               a.zero_row != nullptr && a.offsets[rec.e] >= 0 && a.offsets[rec.e + 1] <= a.P &&
               a.offsets[rec.e] <= a.offsets[rec.e + 1];
        } else {
          ok = rec.row_start + rec.rows <= a.P && rec.fam <= a.P;
        }
      }
      if (ok) {
        bool gave_up = false;
        if constexpr (ROLE == 2) {
          if (threadIdx.x == 0) {
            const long long w0 = a.cycles ? __builtin_amdgcn_s_memtime() : 0;
            int polls = 0, bad = 0;
            if (a.spin_limit < 0) bad = 1;
            else
              while (__hip_atomic_load(&a.fam_done[rec.fam], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < rec.need) {
                if (++polls > a.spin_limit) { bad = 1; break; }
                __builtin_amdgcn_s_sleep(8);
              }
            if (bad) a.hdr->pad[0] = 1;
            *reinterpret_cast<volatile int*>(lds + kBcastOffset + 4) = bad;
            if (a.cycles) {
              a.cycles[(size_t)blockIdx.x * 8 + 6] += __builtin_amdgcn_s_memtime() - w0;
              a.cycles[(size_t)blockIdx.x * 8 + 7] += polls > 0;
            }
          }
          __syncthreads();
          gave_up = __builtin_amdgcn_readfirstlane(*reinterpret_cast<volatile int*>(lds + kBcastOffset + 4)) != 0;
        }
        if (gave_up) {
          // the rows this tile depends on never became complete: its output is written as NaN, so
          // that nothing downstream can take it for a result (the header flag says why)
          poison_tile(a, rec);
        } else {
          run_tile_rows<MODE>(a, rec, lds, lane, w, pending);
        }
        // ROLE 1: this tile's row-block counter is added to by the workgroup's next tile once its
        // first stage has landed, or after the loop (a tile of ROLE 1 is never one that gave up);
        // without `defer_signal` at once, after a wait for this tile's stores
        if constexpr (ROLE == 1) {
          pending = &a.fam_done[rec.fam];
          if (!a.defer_signal) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
      }
      __syncthreads();       // every wave is past its epilogue
      if (threadIdx.x == 0) {
        if (ROLE == 1 && !a.defer_signal && pending != nullptr)
          __hip_atomic_fetch_add(pending, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *reinterpret_cast<volatile int*>(lds + kBcastOffset) = t_next;
      }
      if (ROLE == 1 && !a.defer_signal) pending = nullptr;
      __syncthreads();
      pos = __builtin_amdgcn_readfirstlane(*reinterpret_cast<volatile int*>(lds + kBcastOffset));
    }
  }
  if constexpr (ROLE == 1) {
    // the last tile of this workgroup in this list: wait for its stores, then add to its counter
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (pending != nullptr && threadIdx.x == 0)
      __hip_atomic_fetch_add(pending, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// first: the tiles of list `p` in mode M0, then those of list `q` in mode M1; DEP: the second
// list's tiles wait for row blocks of the first
template <int M0, int M1, bool DEP>
__global__ void __launch_bounds__(Shape<M0>::THREADS) ffn_fused_kernel(const TileArgs p, const TileArgs q) {
  static_assert(Shape<M0>::THREADS == Shape<M1>::THREADS, "one workgroup shape");
  extern __shared__ __align__(1024) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  long long k0 = 0, r0 = 0, k1 = 0, r1 = 0;
  if (p.cycles) { k0 = __builtin_amdgcn_s_memtime(); r0 = __builtin_amdgcn_s_memrealtime(); }
  fused_phase<M0, DEP ? 1 : 0>(p, lds, lane, w);
  if (p.cycles) { k1 = __builtin_amdgcn_s_memtime(); r1 = __builtin_amdgcn_s_memrealtime(); }
  fused_phase<M1, DEP ? 2 : 0>(q, lds, lane, w);
  if (p.cycles && threadIdx.x == 0) {
    // second half of the buffer: [workgroup][8] = core clocks and 100 MHz ticks of the two
    // lists, then the 100 MHz time stamps of the workgroup's start and end
    long long* d = p.cycles + (size_t)(gridDim.x + blockIdx.x) * 8;
    const long long k2 = __builtin_amdgcn_s_memtime(), r2 = __builtin_amdgcn_s_memrealtime();
    d[0] = k1 - k0; d[1] = r1 - r0; d[2] = k2 - k1; d[3] = r2 - r1; d[4] = r0; d[5] = r2;
  }
}

// ---------------------------------------------------------------------------------------
// small tiles: launches that would leave compute units idle with 256 x 256 tiles
// ---------------------------------------------------------------------------------------
// Bound by what the compute units draw from L2 and the last-level cache, twice the bytes per FLOP of a big tile:
// a stage of both workgroups of a unit takes about 1.1 us for its 64 KB, by the launch times 15 TB/s over the chip.  More stages on the way do not
// help (operands through registers, three stages ahead: 50 -> 65 us for 777 tokens of a 1024-wide layer, 107 ->
// 140 for 64 experts x 144 rows; one 256 x 128 tile per unit with all of the LDS: 107 -> 135); what helps is
// that one workgroup's prologue and epilogue run under the other's stages.
// Same tile code, 128 x 128, two workgroups per compute unit, one tile per workgroup; no schedule:
// a workgroup finds its tile from `offsets` with wave-wide scans, the grid covers the largest possible number
// of tiles and the workgroups past the last one exit.  The two projections are two launches (the
// second has nothing to wait for tile by tile, and no counters have to be cleared first); so are the
// two steps of the backward pass, each with everything that is independent in it.
// Consecutive workgroups go to the 8 XCDs in turn; eight neighbouring tiles of the list (a few row
// tiles x a few column tiles of one expert) go to one XCD, where they meet in its L2 (stretches of 32
// measured the same on many tiles and up to 10 % slower on few).
constexpr int kSmallChunk = 8;
__device__ __forceinline__ int small_tile_index(int b) {
  const int xcd = b % kXcds, q = b / kXcds;
  return ((q / kSmallChunk) * kXcds + xcd) * kSmallChunk + q % kSmallChunk;
}

// Tall tiles.  An expert of 129 to 192 rows as two row tiles has every weight fetched twice, the second time for a few
// rows.  Where at least three quarters of the experts are of that size they can be one tile of 192 rows each (two stages of both
// operands instead of two and three, the same 80 KB).  With few such experts, or a remainder of up to 64 rows joined to the last of
// several tiles, the longer tiles end later than what they save: 64 x 112 121 -> 125, 24 x 183 skewed 140 -> 145.
__device__ __forceinline__ bool small_tall(int cnt) { return cnt > SmallTile::BM && cnt <= TallTile::BM; }
__device__ __forceinline__ int small_row_tiles(int cnt, bool tall) {
  return tall && small_tall(cnt) ? 1 : (cnt + SmallTile::BM - 1) / SmallTile::BM;
}

// Whether a launch takes them.  A unit runs two workgroups at a time, and a tall tile is about as long as two of the others, so
// what counts is how both lists fill whole rounds.  Time of the launch tall / plain (on the loop of 32x32x16 MFMAs before this one),
// 23 layers of d = 1024 to 4096 with 12 to 80 experts, 145 to 178 rows each (256 units), by tall tiles:
//   up: up to 512 0.73 to 1.03, mean 0.88 (saving the pre-activations 0.81 to 1.06, 0.94); 513 to 800 0.90 to 1.17, mean 1.06 (1.00
//     to 1.27, 1.13): they begin a third tile per unit; from 832 on 0.88 to 1.09, mean 0.96 (0.97 to 1.06, 1.01), with a fifth of the
//     experts past 192 rows 1.02 (call 145 -> 148 us)
//   down, with nothing else in the launch to fill its units: from 512 on with at most a twentieth of the
//     experts past 192 rows 0.79 to 0.99, mean 0.92, with more 0.84 to 1.09, 1.00; 448 to 511 0.80 to 1.00, 0.94, but
//     1.01 to 1.14 where the last tile of every expert is half a one (d = 1344) and 0.87 to 1.10 with more past 192; below 0.84 to
//     1.30, mean 1.08
//   dH: below 180 0.95 to 1.34, mean 1.09; 180 to 512 0.69 to 0.97, mean 0.83
//   dX (the weight gradients fill what it leaves idle): from 192 on 0.90 to 1.03, mean 0.94
// With less than three quarters of a tile per unit a launch lasts as long as its longest tile: up and dX, 10 layers of two or three
// experts per group and two shared experts of 145 to 180 rows, 16 to 168 up tiles, call 0.96 to 1.15, step 0.98 to 1.17.
// (The launch after one of the same form finds its operands nearer: down 44 us behind tall up tiles, 46 behind plain ones, tall itself.
// Whole calls with these lines against no tall tiles: forward 0.81 to 1.02, mean 0.96 (98 sizes), training step 0.92 to 1.00, 0.97
// (74); tall wherever three quarters of the experts are of their size 0.83 to 1.16, 1.01, and 0.92 to 1.14, 1.01.)
// Here, what only the counts tell: n_tall experts of that size, n_past above it, `tiles` in the launch with tall ones; the rest is
// in may_be_tall.
template <int MODE>
__device__ __forceinline__ bool tall_pays(const TileArgs& a, int n_tall, int n_past, int tiles) {
  if (4 * n_tall < 3 * a.Ne) return false;
  if constexpr (is_up(MODE)) return tiles <= 2 * a.ncu || (20 * n_past <= a.Ne && 4 * tiles >= 13 * a.ncu);
  if constexpr (MODE == kDown) return 20 * n_past <= a.Ne;
  if constexpr (MODE == kDgradH) return tiles <= 2 * a.ncu;
  return true;
}

// tile t of the list of a token mode; false if there is none.  The same in every lane; called by whole waves.
template <int MODE, bool TALL>
__device__ __forceinline__ bool small_token_tile(const TileArgs& a, int t, int lane, TileRec& rec) {
  constexpr int NCPT = is_up(MODE) ? TallTile::BN / 2 : TallTile::BN;
  auto columns = [&](int g) { return ((red_d(MODE) ? a.F[g] : a.d) + NCPT - 1) / NCPT; };
  int before = 0;
  bool tall = false;
  if (TALL && a.Ne > 64) {                         // (up to 64 experts: in the only round below)
    int n_tall = 0, n_past = 0, tiles = 0;
    for (int v0 = 0; v0 < a.Ne; v0 += 64) {
      const int v = min(v0 + lane, a.Ne - 1), cnt = v0 + lane < a.Ne ? a.offsets[v + 1] - a.offsets[v] : 0;
      n_tall += __popcll(__ballot(small_tall(cnt)));
      n_past += __popcll(__ballot(cnt > TallTile::BM));
      tiles += small_row_tiles(cnt, true) * columns(v / a.N);
    }
    tall = tall_pays<MODE>(a, n_tall, n_past, __builtin_amdgcn_readlane(wave_incl_scan(tiles), 63));
  }
  for (int v0 = 0; v0 < a.Ne; v0 += 64) {
    const int v = v0 + lane;                       // groups by decreasing width: the longest tiles start first
    const int g = a.order[(v < a.Ne ? v : 0) / a.N], e = g * a.N + (v < a.Ne ? v : 0) % a.N;
    const int lo = a.offsets[e], cnt = v < a.Ne ? a.offsets[e + 1] - lo : 0;
    const int nt = columns(g);
    int n = small_row_tiles(cnt, TALL && (a.Ne <= 64 || tall)) * nt;
    int incl = wave_incl_scan(n);
    if (TALL && a.Ne <= 64) {
      tall = tall_pays<MODE>(a, __popcll(__ballot(small_tall(cnt))), __popcll(__ballot(cnt > TallTile::BM)),
                             __builtin_amdgcn_readlane(incl, 63));
      if (!tall) {
        n = small_row_tiles(cnt, false) * nt;
        incl = wave_incl_scan(n);
      }
    }
    const int first = before + incl - n;
    const unsigned long long hit = __ballot(t >= first && t < first + n);
    if (hit) {
      const int l = (int)__builtin_ctzll(hit);
      const int rel = t - __builtin_amdgcn_readlane(first, l), ntv = __builtin_amdgcn_readlane(nt, l);
      const int c = __builtin_amdgcn_readlane(cnt, l), mt = small_row_tiles(c, tall);
      // bands of four row tiles; inside a band column tile major, row tile minor
      constexpr int RB = 4;
      const int bnd = rel / (RB * ntv), rel2 = rel - bnd * RB * ntv, rb = min(RB, mt - bnd * RB);
      const int ni = rel2 / rb, mi = bnd * RB + rel2 % rb;
      rec.e = __builtin_amdgcn_readlane(e, l);
      rec.row_start = __builtin_amdgcn_readlane(lo, l) + mi * SmallTile::BM;
      rec.rows = mt == 1 ? c : min(SmallTile::BM, c - mi * SmallTile::BM);
      rec.n0 = ni * NCPT;
      rec.fam = 0;
      rec.need = 0;
      return rec.row_start >= 0 && rec.rows >= 1 && rec.row_start + rec.rows <= a.P;
    }
    before += __builtin_amdgcn_readlane(incl, 63);
  }
  return false;
}

// tile t of a weight gradient (the list depends on the layer's shape only)
__device__ __forceinline__ bool small_wgrad_tile(const TileArgs& a, int t, TileRec& rec) {
  for (int gi = 0; gi < a.Ng; ++gi) {
    const int g = a.order[gi];
    const int mt = (a.Mrows[g] + SmallTile::BM - 1) / SmallTile::BM, nt = (a.Ncols[g] + SmallTile::BN - 1) / SmallTile::BN;
    if (t < a.N * mt * nt) {
      const int i = t / (mt * nt), rel = t - i * mt * nt;
      rec.e = g * a.N + i;
      rec.row_start = rel / nt * SmallTile::BM;
      rec.rows = min(SmallTile::BM, a.Mrows[g] - rec.row_start);
      rec.n0 = rel % nt * SmallTile::BN;
      rec.fam = 0;
      rec.need = 0;
      return a.offsets[rec.e] >= 0 && a.offsets[rec.e + 1] <= a.P && a.offsets[rec.e] <= a.offsets[rec.e + 1];
    }
    t -= a.N * mt * nt;
  }
  return false;
}

constexpr int kSmallThreads = 64 * SmallTile::WGM * SmallTile::WGN;
constexpr int kSmallLds = (kStagesA * SmallTile::BM + kStagesB * SmallTile::BN) * kBK * 2;

template <int MODE, bool TALL = false>
__device__ __forceinline__ void small_tile(const TileArgs& a, int b, unsigned char* lds) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  TileRec rec;
  bool ok;
  if constexpr (MODE == kWgrad) ok = small_wgrad_tile(a, small_tile_index(b), rec);
  else ok = small_token_tile<MODE, TALL>(a, small_tile_index(b), lane, rec);
  if (ok) run_tile_rows<MODE, typename std::conditional<TALL, TallTile, SmallTile>::type>(a, rec, lds, lane, w, nullptr);
}

template <int MODE, bool TALL>
__global__ void __launch_bounds__(kSmallThreads, 2) ffn_small_kernel(const TileArgs a) {
  extern __shared__ __align__(1024) unsigned char lds[];
  // (nothing waits here: the flag that mohge_fused_status reads stays clear)
  if (MODE == kDown && blockIdx.x == 0 && threadIdx.x == 0) a.hdr->pad[0] = 0;
  small_tile<MODE, TALL>(a, blockIdx.x, lds);
}

// Backward, first launch: dH, and on the workgroups past its n_dh the rows of x in sorted order and the
// row of zeros (kSmallGatherRows rows per workgroup, four per wave: their loads are issued together, and the compiler keeps
// three of the four pieces in private memory until their store, 80 bytes per lane).
constexpr int kSmallGatherRows = 16;

template <bool TALL>
__global__ void __launch_bounds__(kSmallThreads, 2) ffn_small_bwd1_kernel(const TileArgs dh, const GatherArgs ga, int n_dh) {
  extern __shared__ __align__(1024) unsigned char lds[];
  if ((int)blockIdx.x < n_dh) {
    small_tile<kDgradH, TALL>(dh, blockIdx.x, lds);
    return;
  }
  const int b = blockIdx.x - n_dh, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (b == 0 && threadIdx.x < 32) ga.zero_row[threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
  if (ga.perm == nullptr || ga.P <= 0) return;
  constexpr int R = kSmallGatherRows / 4;
  const int p0 = b * kSmallGatherRows + w * R;
  long long src[R];
#pragma unroll
  for (int i = 0; i < R; ++i) src[i] = (long long)(ga.perm[min(p0 + i, ga.P - 1)] / ga.Ke) * ga.chunks;
  for (int c = lane; c < ga.chunks; c += 64) {
    uint4 v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = ga.x[src[i] + c];
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (p0 + i < ga.P) ga.xs[(long long)(p0 + i) * ga.chunks + c] = v[i];
  }
}

// Backward, second launch: dX (the longest reductions first), then both weight gradients
template <bool TALL>
__global__ void __launch_bounds__(kSmallThreads, 2) ffn_small_bwd2_kernel(const TileArgs dx, const TileArgs w2,
                                                                          const TileArgs w13, int n_dx, int n_w2) {
  extern __shared__ __align__(1024) unsigned char lds[];
  const int b = blockIdx.x;
  if (b == 0 && threadIdx.x == 0) dx.hdr->pad[0] = 0;
  if (b < n_dx) small_tile<kDgradX, TALL>(dx, b, lds);
  else if (b < n_dx + n_w2) small_tile<kWgrad>(w2, b - n_dx, lds);
  else small_tile<kWgrad>(w13, b - n_dx - n_w2, lds);
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
// Workgroups of a small-tile list, a multiple of 64 (small_tile_index).  Token modes: the counts are not
// known here; full row tiles of the widest group plus a partial one per expert that can have rows.
static long long small_column_tiles(const LayerDesc& L, int mode, int g) {
  const int cp = is_up(mode) ? SmallTile::BN / 2 : SmallTile::BN;
  return ((red_d(mode) ? L.F[g] : L.d) + cp - 1) / cp;
}

static long long small_grid(const LayerDesc& L, int mode) {
  long long n = 0, widest = 0;
  for (int g = 0; g < L.Ng; ++g) {
    const long long nt = small_column_tiles(L, mode, g);
    n += nt * L.N;
    widest = nt > widest ? nt : widest;
  }
  if (L.P * widest < n) n = L.P * widest;
  n += (long long)(L.P / SmallTile::BM) * widest;
  return (n + kXcds * kSmallChunk - 1) / (kXcds * kSmallChunk) * (kXcds * kSmallChunk);
}

// Launches in which tall tiles are looked for (tall_pays: why these lines).  Outside of 140 to 184 rows per expert an even spread
// leaves fewer than three quarters of the experts with 129 to 192 rows (135 and 187: 1.01 to 1.02 of the time); the
// instantiation without them is up to 1 % faster where it finds none (3 % with more than 64 experts, whose lists take two rounds of
// counting, and 5 to 12 % of an up launch whose tiles turn out to begin a third one per unit).
static bool may_be_tall(const LayerDesc& L, int mode) {
  if (L.P < 140ll * L.Ne || L.P > 184ll * L.Ne) return false;
  const long long cus = tile_num_cus();
  long long n = 0;                                        // tiles with one row tile per expert
  for (int g = 0; g < L.Ng; ++g) n += L.N * small_column_tiles(L, mode, g);
  if (is_up(mode)) return 4 * n >= 3 * cus && (n <= 2 * cus || n >= 3 * cus);
  if (mode == kDown) return n >= 2 * cus || (4 * n >= 7 * cus && L.d % SmallTile::BN == 0);
  if (mode == kDgradH) return 10 * n >= 7 * cus && n <= 2 * cus;
  return 4 * n >= 3 * cus;
}

static long long small_wgrad_grid(const TileArgs& a) {
  long long n = 0;
  for (int g = 0; g < a.Ng; ++g)
    n += (long long)a.N * ((a.Mrows[g] + SmallTile::BM - 1) / SmallTile::BM) * ((a.Ncols[g] + SmallTile::BN - 1) / SmallTile::BN);
  return (n + kXcds * kSmallChunk - 1) / (kXcds * kSmallChunk) * (kXcds * kSmallChunk);
}

template <auto KERN, typename... Args>
static hipError_t launch_small(long long grid, hipStream_t s, const Args&... args) {
  static std::atomic<unsigned long long> allowed{0};
  if (grid * kSmallThreads >= 1ll << 32) return hipErrorInvalidConfiguration;      // (only if asked for beyond the rule below)
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(KERN), kSmallLds, allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(KERN, dim3((unsigned)grid), dim3(kSmallThreads), kSmallLds, s, args...);
  return hipGetLastError();
}

// Which geometry a bf16 call past decode size takes.  Small tiles fill the chip, need no schedule launch and overlap one
// workgroup's ends with the other's stages; big ones move half the operand bytes per FLOP.  The measure is the work
// per compute unit in stages of a big tile, both projections, for evenly spread rows.  Time small / big over 17 layer
// shapes (d = 768 to 8192, 8 to 128 experts, 4 to 1024 rows per expert), even and skewed routing, on the present loop:
//   one row tile per expert in either form (up to 112 rows; at 128 half of the experts need two small ones), weights to
//     move and little else:      forward up to 180 stages 0.46 to 1.03, mean 0.76, above 1.06 to 1.13, mean 1.10;
//     backward up to 130 stages 0.40 to 1.10, mean 0.73, above 1.00 to 1.15, mean 1.08
//   more rows, up to 80 stages:  forward 0.46 to 1.21, mean 0.81, backward 0.41 to 1.19, mean 0.82
//              above:            forward 0.81 to 1.37, mean 1.11, backward 0.82 to 1.28, mean 1.13
//     but above 48 where several big row tiles are nine tenths full (d = 2048, 24 experts x 500 rows, on the loop before this one:
//     188 -> 205 us)
// The mean cost of a wrong choice is 0.8 % forward, 0.7 % backward (the largest 1.40 and 1.34: d = 2048, 8 experts x 500 rows, 1.5 big
// up tiles per unit, where full row tiles take the big form).  From 1.7 big up tiles per compute unit on the big form has no
// idle units to lose to; forward, where the big row tiles are not nearly full, from 2.0.  These two limits and the exception for full
// row tiles were drawn on the loop before this one: d = 1024, 32 experts, 768 rows 122 -> 127 us; that limit alone, whatever the length
// of the reduction, cost 1.7 and 2.2 %, up to 1.29; forward 26 layers and token counts with 1.69 to 1.76 tiles per unit 0.58 to 0.99,
// mean 0.87 (rows spread evenly 0.70 to 1.03, 0.92), 13 with 1.83 to 2.0, d = 768 to 1856, 137 to 1375 rows, 0.77 to 1.05, mean 0.91
// (0.75 to 1.07, 0.93).
bool use_small_tiles(const LayerDesc& L, const FfnOptions& o, bool backward) {
  if (o.small >= 0) return o.small != 0;
  const long long rows = L.P > L.Ne ? L.P / L.Ne : 1;     // per expert if they were spread evenly
  long long big = 0, stages = 0;                          // big up tiles; stages of all big tiles
  for (int g = 0; g < L.Ng; ++g) {
    const long long blocks = L.N * ((rows + kBM - 1) / kBM), ut = (L.F[g] + kBN / 2 - 1) / (kBN / 2);
    big += blocks * ut;
    stages += blocks * (ut * (L.d / kBK) + (L.d + kBN - 1) / kBN * (long long)(L.F[g] / kBK));
  }
  const long long cus = tile_num_cus();
  if (!backward && rows <= 112) return stages <= 180 * cus;
  const bool full = rows > kBM && 10 * rows >= 9 * kBM * ((rows + kBM - 1) / kBM);
  return 10 * big < (full || backward ? 17 : 20) * cus && stages <= (rows <= 112 ? 130 : full ? 48 : 80) * cus;
}

hipError_t launch_small_bwd(const LayerDesc& L, const TileArgs& dh, const TileArgs& dx, const TileArgs& w2,
                            const TileArgs& w13, const GatherArgs& ga, hipStream_t s) {
  const long long n_dh = small_grid(L, kDgradH);
  // at least one gather workgroup: it writes the row of zeros (a call without tokens still clears the weight gradients)
  const int gather = ga.perm && ga.P > 0 ? (ga.P + kSmallGatherRows - 1) / kSmallGatherRows : 1;
  hipError_t e = may_be_tall(L, kDgradH) ? launch_small<ffn_small_bwd1_kernel<true>>(n_dh + gather, s, dh, ga, (int)n_dh)
                                         : launch_small<ffn_small_bwd1_kernel<false>>(n_dh + gather, s, dh, ga, (int)n_dh);
  if (e != hipSuccess) return e;
  const long long n_dx = small_grid(L, kDgradX), n_w2 = small_wgrad_grid(w2), n_w13 = small_wgrad_grid(w13);
  return may_be_tall(L, kDgradX) ? launch_small<ffn_small_bwd2_kernel<true>>(n_dx + n_w2 + n_w13, s, dx, w2, w13, (int)n_dx, (int)n_w2)
                                 : launch_small<ffn_small_bwd2_kernel<false>>(n_dx + n_w2 + n_w13, s, dx, w2, w13, (int)n_dx, (int)n_w2);
}

void apply_options(TileArgs& t, const FfnOptions& o) {
  t.band = o.band > 0 ? o.band : 1;
  t.group_major = o.group_major != 0;
  t.steal = o.steal;
  t.short_last = o.short_last != 0;
  t.defer_signal = o.defer_signal != 0;
  t.spin_limit = o.spin_limit == 0 ? kSpinLimit : o.spin_limit;
}

static long long max_tiles(const LayerDesc& L, bool up) {
  // smallest tile height 64 (forced) / 128 (chosen): every expert adds at most one partial tile
  const long long mt = (long long)L.P / 64 + L.Ne;
  const int ncols = up ? L.Fmax : L.d;
  const int ncpt = up ? kBN / 2 : kBN;
  return mt * ((ncols + ncpt - 1) / ncpt);
}

// row-block counters of the fused launch: at most one row block per 64 routed rows plus a
// partial one per expert
static size_t fam_bytes(const LayerDesc& L) {
  return ((size_t)(L.P / 64 + L.Ne + 1) * sizeof(int) + 255) / 256 * 256;
}

// bytes at the start of the workspace reserved for the two schedules and the row-block counters
size_t tiled_sched_bytes(const LayerDesc& L) {
  size_t b = 0;
  for (int up = 0; up < 2; ++up) {
    const size_t n = (size_t)max_tiles(L, up);
    b += 256 + (n * sizeof(TileRec) + 255) / 256 * 256;
  }
  return b + fam_bytes(L);
}

long long tile_capacity(const LayerDesc& L, int mode) {
  if (mode == kUp || mode == kUpSave) return max_tiles(L, true);
  if (mode == kDown || mode == kDgradX) return max_tiles(L, false);
  if (mode == kDgradH) return ((long long)L.P / 64 + L.Ne) * ((L.Fmax + kBN - 1) / kBN);
  const int m = L.d > 2 * L.Fmax ? L.d : 2 * L.Fmax, n = L.d > L.Fmax ? L.d : L.Fmax;
  return (long long)L.Ne * ((m + 63) / 64) * ((n + kBN - 1) / kBN);
}

int tile_num_cus() {
  static std::atomic<int> known{0};       // (GPUs of one kind: any thread's answer serves)
  int n = known.load(std::memory_order_relaxed);
  if (!n) {
    int dev = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess)
      n = p.multiProcessorCount;
    if (n < kXcds) n = 256;
    n = n / kXcds * kXcds;
    known.store(n, std::memory_order_relaxed);
  }
  return n;
}

template <int MODE, typename GEO = BigTile>
static hipError_t launch_stage(const TileArgs& a, hipStream_t s) {
  constexpr size_t smem = (size_t)(kStagesA * kBM + kStagesB * kBN) * kBK * 2;
  auto kern = ffn_tile_kernel<MODE, GEO>;
  static std::atomic<unsigned long long> allowed{0};
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), (int)smem, allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.ncu), dim3(Shape<MODE>::THREADS), smem, s, a);
  return hipGetLastError();
}

template <int M0, int M1, bool DEP>
static hipError_t launch_fused(const TileArgs& up, const TileArgs& dn_in, hipStream_t s) {
  const TileArgs& dn = dn_in;
  constexpr size_t smem = (size_t)(kStagesA * kBM + kStagesB * kBN) * kBK * 2;
  auto kern = ffn_fused_kernel<M0, M1, DEP>;
  static std::atomic<unsigned long long> allowed{0};
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), (int)smem, allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(up.ncu), dim3(Shape<M0>::THREADS), smem, s, up, dn);
  return hipGetLastError();
}

template <int MODE>
static hipError_t sched_and_run(const TileArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((tile_schedule_kernel<MODE>), dim3(1), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_stage<MODE>(a, s);
}

hipError_t launch_bwd_schedules(const TileArgs& dh, const TileArgs& dx, const TileArgs& w2,
                                const TileArgs& w13, const GatherArgs& ga, bool fused, hipStream_t s) {
  // at least one gather workgroup, so that the row of zeros gets written
  const unsigned gather_blocks = ga.P > 0 && ga.perm ? (unsigned)((ga.P + 3) / 4) : 1u;
  hipLaunchKernelGGL(bwd_schedule_kernel, dim3(4 + gather_blocks), dim3(256), 0, s, dh, dx, w2, w13,
                     fused ? 1 : 0, ga);
  return hipGetLastError();
}


// byte offset, inside the workspace of the forward, of the header of the list whose tiles wait
size_t tiled_waiting_header_offset(const LayerDesc& L) {
  return 256 + ((size_t)max_tiles(L, true) * sizeof(TileRec) + 255) / 256 * 256;
}

// dH and dX in one launch (dX tiles wait for the dH tiles of their row block)
hipError_t launch_dgrad_pair(const TileArgs& dh, const TileArgs& dx, hipStream_t s) {
  return launch_fused<kDgradH, kDgradX, true>(dh, dx, s);
}

// the two weight-gradient products in one launch
hipError_t launch_wgrad_pair(const TileArgs& w2, const TileArgs& w13, hipStream_t s) {
  return launch_fused<kWgrad, kWgrad, false>(w2, w13, s);
}

hipError_t launch_tiles(int mode, const TileArgs& a, hipStream_t s) {
  switch (mode) {
    case kDgradH: return launch_stage<kDgradH>(a, s);
    case kDgradX: return launch_stage<kDgradX>(a, s);
    case kWgrad: return launch_stage<kWgrad>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_tile_gemm(int mode, const TileArgs& a, hipStream_t s) {
  switch (mode) {
    case kUpSave: return sched_and_run<kUpSave>(a, s);
    case kDgradH: return sched_and_run<kDgradH>(a, s);
    case kDgradX: return sched_and_run<kDgradX>(a, s);
    case kWgrad: return sched_and_run<kWgrad>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// `pre` != NULL (training): the up projection also stores the backward factors b SiLU'(a) and
// SiLU(a) as rows of [P, 2*Fmax] for the backward pass.
hipError_t launch_ffn_tiled(const LayerDesc& L, const void* x, const int32_t* perm,
                            const int32_t* offsets, const GroupPtrs& W, void* y_perm, void* ws,
                            hipStream_t s, int stages, void* pre, int parts, const FfnOptions& o) {
  unsigned char* base = static_cast<unsigned char*>(ws);
  uint16_t* H = reinterpret_cast<uint16_t*>(base + tiled_sched_bytes(L));
  TileArgs up{};
  up.pre = static_cast<uint16_t*>(pre);
  up.ldpre = 2 * L.Fmax;
  up.A = static_cast<const uint16_t*>(x);
  up.perm = perm;
  up.offsets = offsets;
  up.C = H;
  up.lda = L.d; up.ldc = L.Fmax;
  up.Ke = L.Ke; up.Ng = L.Ng; up.N = L.N; up.Ne = L.Ne; up.d = L.d; up.P = L.P;
  up.ncu = tile_num_cus();
  apply_options(up, o);
  up.cycles = o.cycles;
  // visit groups by decreasing width: the down projection's longest reductions come first
  int order[kMaxGroups];
  for (int g = 0; g < kMaxGroups; ++g) order[g] = g;
  for (int i = 1; i < L.Ng; ++i)
    for (int j = i; j > 0 && L.F[order[j]] > L.F[order[j - 1]]; --j) {
      int t = order[j]; order[j] = order[j - 1]; order[j - 1] = t;
    }
  for (int g = 0; g < kMaxGroups; ++g) {
    up.F[g] = L.F[g];
    up.order[g] = order[g];
    up.W[g] = static_cast<const uint16_t*>(W.w13[g]);
    up.ldw[g] = L.d;
  }
  TileArgs dn = up;
  dn.A = H;
  dn.perm = nullptr;
  dn.C = static_cast<uint16_t*>(y_perm);
  dn.lda = L.Fmax; dn.ldc = L.d;
  for (int g = 0; g < kMaxGroups; ++g) {
    dn.W[g] = static_cast<const uint16_t*>(W.w2[g]);
    dn.ldw[g] = L.F[g];
  }
  // schedule areas: [header 256 B][records][cost prefix] for up, then the same for down
  unsigned char* p = base;
  for (int st = 0; st < 2; ++st) {
    TileArgs& t = st == 0 ? up : dn;
    const size_t n = (size_t)max_tiles(L, st == 0);
    t.hdr = reinterpret_cast<SchedHeader*>(p);
    p += 256;
    t.recs = reinterpret_cast<TileRec*>(p);
    p += (n * sizeof(TileRec) + 255) / 256 * 256;
    t.force_rows = o.tile_rows[st];
  }
  up.fam_done = dn.fam_done = reinterpret_cast<int*>(p);
  // weight rows of kLongRow elements: the two lists one after the other, in the form that has 64-bit addresses
  if (L.d >= kLongRow || L.Fmax >= kLongRow) {
    if (parts & 1) {
      hipLaunchKernelGGL(ffn_schedule_kernel, dim3(stages == 3 ? 2 : 1), dim3(256), 0, s, up, dn, stages);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    if (!(parts & 2)) return hipSuccess;
    hipError_t e = hipSuccess;
    if (stages & 1) e = pre ? launch_stage<kUpSave, LongTile>(up, s) : launch_stage<kUp, LongTile>(up, s);
    if (e == hipSuccess && (stages & 2)) e = launch_stage<kDown, LongTile>(dn, s);
    return e;
  }
  if (parts == 3 && use_small_tiles(L, o, false)) {
    up.cycles = dn.cycles = nullptr;           // (the counters have room for a workgroup per compute unit)
    hipError_t e = hipSuccess;
    if (stages & 1) {
      const long long n = small_grid(L, kUp);
      const bool tall = may_be_tall(L, pre ? kUpSave : kUp);
      if (pre) e = tall ? launch_small<ffn_small_kernel<kUpSave, true>>(n, s, up) : launch_small<ffn_small_kernel<kUpSave, false>>(n, s, up);
      else e = tall ? launch_small<ffn_small_kernel<kUp, true>>(n, s, up) : launch_small<ffn_small_kernel<kUp, false>>(n, s, up);
    }
    if (e == hipSuccess && (stages & 2)) {
      const long long n = small_grid(L, kDown);
      e = may_be_tall(L, kDown) ? launch_small<ffn_small_kernel<kDown, true>>(n, s, dn) : launch_small<ffn_small_kernel<kDown, false>>(n, s, dn);
    }
    return e;
  }
  // the whole forward in one launch: up and down tiles share the persistent workgroups
  if (stages == 3 && o.fused) {
    up.coherent_out = 1;
    // parts: 1 = the tile schedule only, 2 = the product launch only (on a schedule that no
    // launch has consumed yet), 3 = both
    if (parts & 1) {
      // a workgroup per list writes 256 records at a time: about two rounds each (four workgroups took 22 us
      // for the 8000 tiles of a 16384-token call)
      long long parts_per_list = max_tiles(L, false) / 512;
      parts_per_list = parts_per_list < 4 ? 4 : parts_per_list > 32 ? 32 : parts_per_list;
      hipLaunchKernelGGL(ffn_schedule_kernel, dim3((unsigned)(2 * parts_per_list)), dim3(256), 0, s, up, dn, 7);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    if (!(parts & 2)) return hipSuccess;
    return pre ? launch_fused<kUpSave, kDown, true>(up, dn, s) : launch_fused<kUp, kDown, true>(up, dn, s);
  }
  if (parts != 3) return hipErrorInvalidValue;       // (the API checks this before it gets here)
  // both schedules depend only on `offsets`: one launch builds whichever are needed
  hipLaunchKernelGGL(ffn_schedule_kernel, dim3(stages == 3 ? 2 : 1), dim3(256), 0, s, up, dn, stages);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (stages & 1) e = pre ? launch_stage<kUpSave>(up, s) : launch_stage<kUp>(up, s);
  if (e != hipSuccess) return e;
  if (stages & 2) e = launch_stage<kDown>(dn, s);
  return e;
}

}  // namespace mohge
