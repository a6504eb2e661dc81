// Two-level router (section 3.2 of the paper) for gfx950.
//
// One workgroup owns 16*TM tokens.  Phase 1 computes the N_g + N_e logits of its
// tokens with the fp32 matrix cores (v_mfma_f32_16x16x4_f32): tokens are the M
// rows, router rows (group embeddings first, then expert embeddings) the N columns.
// Each lane loads 8 consecutive hidden elements of "its" token / router row straight
// from global memory -- this is already the operand layout the instruction wants, so
// no LDS staging is needed.  The hidden dimension is split over the waves of the
// workgroup; every wave folds its fp32 accumulators into fp64 totals after each 64
// hidden elements, and the per-wave totals are added in fp64 in a fixed order.  This
// keeps the logit error near 1e-7, which bit-exact top-k agreement with an fp64
// reference needs.
// With few tokens (decode) one workgroup per 16 tokens leaves most of the chip idle while two
// compute units grind through the whole reduction: then the hidden dimension is split over
// grid.y workgroups as well, each leaves its fp64 sums in a workspace, and a second small kernel
// adds them in a fixed order and runs phase 2.
// Phase 2 runs one wavefront per token with lane <-> expert: group top-K_g by rank
// counting, softmax inside kept groups, scaling by the group score, expert top-k by
// rank counting, a ballot + popcount to assign ascending output slots, and a
// cross-lane sum for the gate normalisation.
#include <type_traits>

#include "common.h"
#include "route_select.h"

namespace mohge {

template <bool BF16, int TM, int TN>
__global__ void __launch_bounds__(512) route_kernel(const RouteArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int BT = 16 * TM, NC = 16 * TN;
  const int NW = blockDim.x >> 6;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, q = lane >> 4;
  const int t0 = blockIdx.x * BT;
  double* part = reinterpret_cast<double*>(smem);                 // [NW][BT][NC]
  float* lg = reinterpret_cast<float*>(smem + a.region0);         // [BT][NOpad]

  // ---- phase 1: logits ----------------------------------------------------
  size_t xrow[TM];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    int t = t0 + 16 * tm + r;
    xrow[tm] = (size_t)(t < a.T ? t : a.T - 1) * a.d;
  }
  // passes over the router rows: one workgroup after the other, or (split form) side by side
  for (int nc = blockIdx.z * NC; nc < a.NO; nc += NC * gridDim.z) {
    const float* wrow[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      int o = nc + 16 * tn + r;
      if (o > a.NO - 1) o = a.NO - 1;
      wrow[tn] = (o < a.Ng) ? a.wg + (size_t)o * a.d : a.we + (size_t)(o - a.Ng) * a.d;
    }
    f32x4 acc[TM][TN];
    double tot[TM][TN][4];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        acc[tm][tn] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) tot[tm][tn][i] = 0.0;
      }
    // (the last slices may be short or empty: d need not be a multiple of the slices together)
    const int kbeg = ((int)blockIdx.y * NW + w) * a.kslice, kend = min(kbeg + a.kslice, a.d);
    // The token rows are read exactly once from HBM in small pieces (16 rows x 64 bytes per
    // wave-wide load), so the loop is bound by memory latency unless many loads are in
    // flight: all token loads of a chunk of 32-element steps are requested up
    // front and kept packed in registers; the router rows (L2 resident) are requested one
    // step ahead.  The fp32 accumulators are folded into the fp64 totals after every pair of
    // steps (64 elements).
    if constexpr (!BF16) {
      // fp32 tokens: four steps at a time, each with a check.  (Whole runs of steps without one, as below, take more
      // registers here, with two token tiles one workgroup per compute unit instead of two: d = 512, 15 rows,
      // 32768 tokens 28.2 us, without checks 41.1; d = 4096, 68 rows, 4096 tokens 51.4 and 58.9.)
      constexpr int XS = 4;
      for (int kc = kbeg; kc < kend; kc += 32 * XS) {
        float4 xraw[TM][XS][2];
#pragma unroll
        for (int st = 0; st < XS; ++st)
          if (kc + 32 * st < kend) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
              const float4* p = reinterpret_cast<const float4*>(static_cast<const char*>(a.x) +
                                                                (xrow[tm] + kc + 32 * st + 8 * q) * 4);
              xraw[tm][st][0] = p[0];
              xraw[tm][st][1] = p[1];
            }
          }
        float wb[2][TN][8];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) load8<false>(wrow[tn], (size_t)(kc + 8 * q), wb[0][tn]);
#pragma unroll
        for (int st = 0; st < XS; ++st) {
          const int k = kc + 32 * st;
          if (k < kend) {
            if (st + 1 < XS && k + 32 < kend) {
#pragma unroll
              for (int tn = 0; tn < TN; ++tn) load8<false>(wrow[tn], (size_t)(k + 32 + 8 * q), wb[(st + 1) & 1][tn]);
            }
            float xa[TM][8];
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
              const float4 lo = xraw[tm][st][0], hi = xraw[tm][st][1];
              xa[tm][0] = lo.x; xa[tm][1] = lo.y; xa[tm][2] = lo.z; xa[tm][3] = lo.w;
              xa[tm][4] = hi.x; xa[tm][5] = hi.y; xa[tm][6] = hi.z; xa[tm][7] = hi.w;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
              for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                  acc[tm][tn] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[tm][j], wb[st & 1][tn][j], acc[tm][tn], 0, 0, 0);
            if ((st & 1) || k + 32 >= kend) {
#pragma unroll
              for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) {
#pragma unroll
                  for (int i = 0; i < 4; ++i) tot[tm][tn][i] += (double)acc[tm][tn][i];
                  acc[tm][tn] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
          }
        }
      }
    } else {
      // NS steps from kc on, without a branch between requests: behind one the compiler waits for everything on its way,
      // the router rows just requested included.  (Whole call, with a check before every request -> this: d = 2048, 27 rows, 4096
      // tokens 16.2 -> 14.8 us, 700 10.4 -> 9.7; d = 4096, 68 rows 47.1 -> 45.2; d = 2560, 66 rows, 1500 tokens 26.8 -> 25.4.)
      auto chunk = [&](int kc, auto NSC) {
        constexpr int NS = decltype(NSC)::value;
        uint4 xraw[TM][NS];
#pragma unroll
        for (int st = 0; st < NS; ++st)
#pragma unroll
          for (int tm = 0; tm < TM; ++tm)
            xraw[tm][st] = *reinterpret_cast<const uint4*>(static_cast<const char*>(a.x) + (xrow[tm] + kc + 32 * st + 8 * q) * 2);
        float wb[2][TN][8];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) load8<false>(wrow[tn], (size_t)(kc + 8 * q), wb[0][tn]);
#pragma unroll
        for (int st = 0; st < NS; ++st) {
          if (st + 1 < NS) {
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) load8<false>(wrow[tn], (size_t)(kc + 32 * st + 32 + 8 * q), wb[(st + 1) & 1][tn]);
          }
          __builtin_amdgcn_sched_barrier(0);
          float xa[TM][8];
#pragma unroll
          for (int tm = 0; tm < TM; ++tm) {
            const uint4 u = xraw[tm][st];
            xa[tm][0] = __uint_as_float(u.x << 16); xa[tm][1] = __uint_as_float(u.x & 0xffff0000u);
            xa[tm][2] = __uint_as_float(u.y << 16); xa[tm][3] = __uint_as_float(u.y & 0xffff0000u);
            xa[tm][4] = __uint_as_float(u.z << 16); xa[tm][5] = __uint_as_float(u.z & 0xffff0000u);
            xa[tm][6] = __uint_as_float(u.w << 16); xa[tm][7] = __uint_as_float(u.w & 0xffff0000u);
          }
#pragma unroll
          for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
              for (int tn = 0; tn < TN; ++tn)
                acc[tm][tn] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[tm][j], wb[st & 1][tn][j], acc[tm][tn], 0, 0, 0);
          if ((st & 1) || st + 1 == NS) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
              for (int tn = 0; tn < TN; ++tn) {
#pragma unroll
                for (int i = 0; i < 4; ++i) tot[tm][tn][i] += (double)acc[tm][tn][i];
                acc[tm][tn] = f32x4{0.f, 0.f, 0.f, 0.f};
              }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      int kc = kbeg;
      for (; kend - kc >= 512; kc += 512) chunk(kc, std::integral_constant<int, 16>{});
      if (kend - kc >= 256) { chunk(kc, std::integral_constant<int, 8>{}); kc += 256; }
      if (kend - kc >= 128) { chunk(kc, std::integral_constant<int, 4>{}); kc += 128; }
      if (kend - kc >= 64) { chunk(kc, std::integral_constant<int, 2>{}); kc += 64; }
      if (kend - kc >= 32) chunk(kc, std::integral_constant<int, 1>{});
    }
    // Accumulator element i of lane (r, q) is token 4q+i, router row r of the 16x16 tile.
    // Every wave stores its fp64 totals in its own slice; then they are added in wave order.
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          part[((size_t)w * BT + 16 * tm + 4 * q + i) * NC + 16 * tn + r] = tot[tm][tn][i];
    __syncthreads();
    for (int idx = threadIdx.x; idx < BT * NC; idx += blockDim.x) {
      const int tl = idx / NC, ol = idx % NC;
      double sum = 0.0;
      for (int ww = 0; ww < NW; ++ww) sum += part[(size_t)ww * BT * NC + idx];
      if (nc + ol < a.NO) {
        if (a.dsplit > 1) {
          if (t0 + tl < a.T) a.gpart[((size_t)blockIdx.y * a.T + t0 + tl) * a.NO + nc + ol] = sum;
        } else {
          lg[tl * a.NOpad + nc + ol] = (float)sum;
        }
      }
    }
    __syncthreads();
  }

  if (a.dsplit > 1) return;          // route_finish_kernel takes over
  route_select(a, smem, lg, t0, BT, NW, w, lane);
}

// ---------------------------------------------------------------------------------------
// Prefill form (bf16 tokens, many tokens): the logits on the bf16 matrix cores, exactly.
// A router weight (fp32, 24 significant bits) is the exact sum of three bf16 numbers (its
// leading 8 bits, the next 8, the rest: each taken by truncation, the remainders are exact
// in fp32), a token element is one bf16 number, and a product of two bf16 numbers is exact in
// fp32.  So  x . w = x . w_hi + x . w_mid + x . w_lo  with v_mfma_f32_16x16x32_bf16, whose only
// rounding is that of its fp32 sums.  It cuts them off downwards, so few may follow each other: the large part (w_hi) of
// every 32 hidden elements is added to an fp64 total.  That keeps the logit error below that of the fp32 form above (2-norm
// against float64, d = 128 to 8192: 3.9e-8 against 1.07e-7 at d = 128 and 1.5e-7 from d = 384 on; mean error, of the logits'
// rms, at most 2e-9, downwards).  Sixteen times the fp32 matrix rate at three times the work.
//
// A small kernel first splits the router rows into the three bf16 planes (workspace:
// [3][rows padded to whole passes][d], padding rows zero).  In the main kernel a workgroup of 8
// waves owns 16*TG tokens: waves = TG token groups of 16 x (8/TG) parts of every 64- or 128-deep chunk
// of the hidden dimension.  A wave loads its token fragments straight from global memory in
// operand layout (several chunks ahead); the three planes of a chunk go global -> LDS without
// passing registers (global_load_lds, up to three chunks ahead, 16-byte pieces XOR-swizzled by the row so
// that the 128-bit fragment reads are conflict free).  The waves of a token group add their fp64
// totals through LDS in fixed order.  Router rows are processed 16*TN at a time (TN <= 5 column
// tiles: more would not fit the registers); wider routers make several passes over the token rows.
// The logits go to the workspace and a second kernel selects, one wave per token: inside this one, with two waves per SIMD, the
// selection of a workgroup's 64 tokens took as long as a pass (d = 1024, 136 rows, 12000 tokens: 119 us for the call with
// it, 93 without).  SEL: it selects all the same, which saves the second kernel and the logits' way through memory.  That
// is faster where the reduction is short or two workgroups fit a compute unit: see prefill_plan.
// Bound by the planes, which every compute unit reads from L2 (1.9 MB at 68 rows, d = 4096) and its waves from LDS.
// ---------------------------------------------------------------------------------------
typedef __bf16 rbf16x8 __attribute__((ext_vector_type(8)));

constexpr int kPfDepth = 128;            // the hidden size is a multiple of it

// Hidden elements per chunk and chunks in LDS: four where they fit, so that several are on their way while one is used.  (One
// workgroup per compute unit has all of its LDS.  Two chunks: 68 router rows, d = 4096, 16384 tokens 80 us for the call, now 65.)
// SEL (up to two column tiles, or three with 32 tokens): two chunks, registers and LDS for two workgroups per compute unit.
template <int TG, int TN, bool SEL>
struct PrefillShape {
  static constexpr int CH = !SEL && TG == 4 && TN >= 4 ? 64 : 128;
  static constexpr int NB = !SEL && 4 * 3 * 16 * TN * CH * 2 <= 150 * 1024 ? 4 : 2;
  static constexpr int LDS = NB * 3 * 16 * TN * CH * 2;
};

// planes[p][row][k], p = 0 (leading bits), 1, 2; rows >= NO are zero
__global__ void __launch_bounds__(256) route_split_kernel(const float* __restrict__ wg, const float* __restrict__ we,
                                                          uint16_t* __restrict__ planes, int Ng, int NO,
                                                          int rows, int d) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;      // one thread per 4 hidden elements
  const int per_row = d / 4;
  if (idx >= (long long)rows * per_row) return;
  const int o = (int)(idx / per_row), k = (int)(idx % per_row) * 4;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (o < NO) v = *reinterpret_cast<const float4*>(((o < Ng) ? wg + (size_t)o * d : we + (size_t)(o - Ng) * d) + k);
  const float f[4] = {v.x, v.y, v.z, v.w};
  uint32_t hi[4], mid[4], lo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!__builtin_isfinite(f[i])) {                         // as it is (the differences below would be NaN)
      hi[i] = __builtin_isnan(f[i]) ? 0x7fc00000u : __float_as_uint(f[i]);
      mid[i] = lo[i] = 0u;
      continue;
    }
    hi[i] = __float_as_uint(f[i]) & 0xffff0000u;
    const float r1 = f[i] - __uint_as_float(hi[i]);          // exact
    mid[i] = __float_as_uint(r1) & 0xffff0000u;
    const float r2 = r1 - __uint_as_float(mid[i]);           // exact, at most 8 significant bits
    lo[i] = __float_as_uint(r2) & 0xffff0000u;
  }
  const size_t plane = (size_t)rows * d, at = (size_t)o * d + k;
  *reinterpret_cast<uint2*>(planes + at) = make_uint2((hi[0] >> 16) | hi[1], (hi[2] >> 16) | hi[3]);
  *reinterpret_cast<uint2*>(planes + plane + at) = make_uint2((mid[0] >> 16) | mid[1], (mid[2] >> 16) | mid[3]);
  *reinterpret_cast<uint2*>(planes + 2 * plane + at) = make_uint2((lo[0] >> 16) | lo[1], (lo[2] >> 16) | lo[3]);
}

template <int TG, int TN, bool SEL>
__global__ void __launch_bounds__(512, SEL ? 4 : 2) route_prefill_kernel(const RouteArgs a, const uint16_t* __restrict__ planes,
                                                            int plane_rows) {
  extern __shared__ __align__(1024) unsigned char smem[];
  constexpr int KQ = 8 / TG;                 // waves along the hidden dimension
  constexpr int CH = PrefillShape<TG, TN, SEL>::CH, NB = PrefillShape<TG, TN, SEL>::NB;
  constexpr int KS = CH / 32 / KQ;           // 32-deep MFMA steps of a wave per chunk
  constexpr int BT = 16 * TG, NC = 16 * TN;
  constexpr int ROW = CH * 2, PLANE = NC * ROW, BUF = 3 * PLANE;
  constexpr int RPC = 1024 / ROW, PPR = ROW / 16;   // rows per wave-wide copy, 16-byte pieces per row
  constexpr int NCOPY = 3 * NC / RPC;        // wave-wide copies per chunk
  constexpr int WCOPY = (NCOPY + 7) / 8;     // ... per wave (the last ones twice: the same bytes to the same place)
  constexpr int XP = 512 / CH;               // token chunks in flight
  static_assert(KS >= 1 && NC % RPC == 0 && XP % NB == 0 && (NB - 1) * (WCOPY + KS) + KS <= 63, "waits");
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tg = w / KQ, kq = w % KQ;
  const int r = lane & 15, q = lane >> 4;
  const int t0 = blockIdx.x * BT;
  double* red = reinterpret_cast<double*>(smem);                  // [BT][NC], after the chunk loop
  float* lg = reinterpret_cast<float*>(smem + a.region0);         // SEL: [BT][NOpad]
  const int nchunks = a.d / CH;

  const int tok = t0 + tg * 16 + r;
  const uint16_t* xrow = static_cast<const uint16_t*>(a.x) + (size_t)(tok < a.T ? tok : a.T - 1) * a.d +
                         kq * 32 * KS + 8 * q;
  const size_t plane_elems = (size_t)plane_rows * a.d;

  for (int nc = 0; nc < a.NO; nc += NC) {
    f32x4 acc_l[TN];
    double tot[TN][4];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      acc_l[tn] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) tot[tn][i] = 0.0;
    }
    // copy idx (wave-uniform) of a chunk: plane idx / (NC/RPC), rows RPC*(idx % (NC/RPC)) .. of the
    // pass; lane l fills row l/PPR, physical piece l%PPR, which holds logical piece (l%PPR) ^ (row % PPR)
    auto copy_one = [&](int c, int b, int idx) {
      const int p = idx / (NC / RPC), row = RPC * (idx % (NC / RPC)) + lane / PPR;
      const int piece = (lane % PPR) ^ (row % PPR);
      const uint16_t* src = planes + p * plane_elems + (size_t)(nc + row) * a.d + (size_t)c * CH + piece * 8;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)(smem + b * BUF + idx * 1024),
                                       16, 0, 0);
    };
    auto copy_w = [&](int c, int b) {
      if constexpr (SEL) {               // (unrolled, its addresses would take the second workgroup's registers)
        for (int idx = w; idx < NCOPY; idx += 8) copy_one(c, b, idx);
      } else {
#pragma unroll
        for (int i = 0; i < WCOPY; ++i) copy_one(c, b, min(w + 8 * i, NCOPY - 1));
      }
    };
    uint4 xr[XP][KS];
    auto load_x = [&](int c, int slot) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        xr[slot][ks] = *reinterpret_cast<const uint4*>(xrow + (size_t)c * CH + 32 * ks);
    };

    __syncthreads();                     // the previous pass has left the buffers
#pragma unroll
    for (int u = 0; u < NB - 1; ++u)
      if (u < nchunks) copy_w(u, u);
#pragma unroll
    for (int u = 0; u < XP; ++u)
      if (u < nchunks) load_x(u, u);
    // vmcnt(0), known to the compiler: the loop's waits then count what the loop itself requests
    __builtin_amdgcn_s_waitcnt(0x0f70);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // XP chunks from c0 on.  FULL: all that they request exists, so there are no branches between the requests and the
    // compiler's own waits for the token fragments are exact (behind a branch it waits for everything on its way).
    auto group = [&](int c0, auto FULL) {
      constexpr bool full = decltype(FULL)::value;
#pragma unroll
      for (int u = 0; u < XP; ++u) {
        const int c = c0 + u;
        if (full || c < nchunks) {
          rbf16x8 xa[KS];
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) xa[ks] = __builtin_bit_cast(rbf16x8, xr[u][ks]);
          // a later chunk's planes into the buffer that the previous chunk had (nobody reads it any more:
          // barrier at its end), then the token fragments of a later chunk
          if (full || c + NB - 1 < nchunks) copy_w(c + NB - 1, (u + NB - 1) % NB);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (SEL) {
            if (c + XP < nchunks) load_x(c + XP, u);
            __builtin_amdgcn_sched_barrier(0);
          }
          const unsigned char* fb = smem + (u % NB) * BUF + r * ROW;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const int piece = ((kq * KS + ks) * 4 + q) ^ (r % PPR);
            f32x4 h[TN];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
              const unsigned char* f = fb + 16 * tn * ROW + piece * 16;
              const rbf16x8 bh = *reinterpret_cast<const rbf16x8*>(f);
              const rbf16x8 bm = *reinterpret_cast<const rbf16x8*>(f + PLANE);
              const rbf16x8 bl = *reinterpret_cast<const rbf16x8*>(f + 2 * PLANE);
              h[tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[ks], bh, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
              acc_l[tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[ks], bm, acc_l[tn], 0, 0, 0);
              acc_l[tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[ks], bl, acc_l[tn], 0, 0, 0);
            }
            // the large part goes into the fp64 totals at once.  (Every second time, which of two sums are added in fp32 first depends
            // on the tokens per workgroup: error 3.9e-8 with 32 and 5.0e-8 with 64 at d = 128, 4.9e-8 with both from d = 1024 on.  Time
            // within 0.2 %.)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
              for (int i = 0; i < 4; ++i) tot[tn][i] += (double)h[tn][i];
          }
          // (not SEL: behind the last use of the registers; in front of it the compiler copies them, once all of them have landed)
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (!SEL)
            if (full || c + XP < nchunks) load_x(c + XP, u);
          // my pieces of the next chunk's planes have landed when at most what was issued after them is outstanding
          // (loads complete in order): the planes of NB - 2 further chunks and the token loads of NB - 1 (SEL: NB is 2, whatever
          // a wave's number of copies)
          if (full || c + XP < nchunks) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NB - 2) * WCOPY + (NB - 1) * KS) : "memory");
          else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    int c0 = 0;
    if constexpr (!SEL)
      for (; c0 + 2 * XP <= nchunks; c0 += XP) group(c0, std::true_type{});
    for (; c0 < nchunks; c0 += XP) group(c0, std::false_type{});
    // the small parts, then the waves of a token group in fixed order
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int i = 0; i < 4; ++i) tot[tn][i] += (double)acc_l[tn][i];
    for (int step = 0; step < KQ; ++step) {
      if (kq == step) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            // accumulator element i of lane (r, q): token 4q+i, router row r of the tile
            const int tl = tg * 16 + 4 * q + i, ol = 16 * tn + r;
            double v = tot[tn][i];
            if (step > 0) v += red[tl * NC + ol];
            if (step < KQ - 1) red[tl * NC + ol] = v;
            else if (nc + ol < a.NO) {
              if constexpr (SEL) lg[tl * a.NOpad + nc + ol] = (float)v;
              else if (t0 + tl < a.T) a.glog[(size_t)(t0 + tl) * a.NO + nc + ol] = (float)v;
            }
          }
      }
      __syncthreads();
    }
  }
  if constexpr (SEL) route_select(a, smem, lg, t0, BT, 8, w, lane);
}

template <int TG, int TN, bool SEL>
static hipError_t launch_prefill(RouteArgs a, const uint16_t* planes, int plane_rows, hipStream_t s) {
  typedef PrefillShape<TG, TN, SEL> Shape;
  static_assert(16 * TG * 16 * TN * sizeof(double) <= Shape::LDS, "the sums");
  size_t smem = Shape::LDS;
  if (SEL) {
    static_assert(8 * 5 * 64 * sizeof(float) <= Shape::LDS, "the selection's rows: three tiles hold at most 47 experts");
    a.region0 = (int)smem;
    smem += (size_t)16 * TG * a.NOpad * sizeof(float);            // (79 KB at most)
  }
  auto kern = route_prefill_kernel<TG, TN, SEL>;
  static std::atomic<unsigned long long> allowed{0};
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), 160 * 1024, allowed);
  if (e != hipSuccess) return e;
  constexpr int BT = 16 * TG;
  hipLaunchKernelGGL(kern, dim3((a.T + BT - 1) / BT), dim3(512), smem, s, a, planes, plane_rows);
  return hipGetLastError();
}

// Second kernel of the split form: a workgroup takes four tokens (phase 2 is one wave per token, and with few
// tokens its latency is the cost), adds the dsplit partial logit sums of its tokens in index order and
// runs phase 2.  All partial sums of a logit are requested before the first is added: one after the other
// they were a chain of up to 16 memory latencies, most of the 9 to 14 us this kernel took.
constexpr int kSplitMax = 16;            // the most partial sums of a logit
constexpr int kFinishTokens = 4;
constexpr int kPrefillTokens = 8;

// SUMS: fp64 partial sums in gpart, else finished logits in glog
template <int BT, bool SUMS>
__global__ void __launch_bounds__(512) route_finish_kernel(const RouteArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NW = 8;                    // (a constant: 41 registers instead of 98, the waves of four workgroups per compute unit)
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t0 = blockIdx.x * BT;
  float* lg = reinterpret_cast<float*>(smem + a.region0);         // [BT][NOpad]
  for (int idx = threadIdx.x; idx < BT * a.NO; idx += blockDim.x) {
    const int tl = idx / a.NO, o = idx % a.NO;
    if constexpr (!SUMS) {
      lg[tl * a.NOpad + o] = t0 + tl < a.T ? a.glog[(size_t)(t0 + tl) * a.NO + o] : 0.f;
      continue;
    }
    double sum = 0.0;
    if (t0 + tl < a.T) {
      const double* p = a.gpart + (size_t)(t0 + tl) * a.NO + o;
      double v[kSplitMax];
#pragma unroll
      for (int sp = 0; sp < kSplitMax; ++sp) v[sp] = sp < a.dsplit ? p[(size_t)sp * a.T * a.NO] : 0.0;
#pragma unroll
      for (int sp = 0; sp < kSplitMax; ++sp) sum += v[sp];
    }
    lg[tl * a.NOpad + o] = (float)sum;
  }
  __syncthreads();
  route_select(a, smem, lg, t0, BT, NW, w, lane);
}

template <bool BF16, int TM, int TN>
static hipError_t launch_one(const RouteArgs& a, dim3 grid, dim3 block, size_t smem, hipStream_t s) {
  auto kern = route_kernel<BF16, TM, TN>;
  static std::atomic<unsigned long long> allowed{0};
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), 160 * 1024, allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid, block, smem, s, a);
  return hipGetLastError();
}

template <bool BF16, int TM>
static hipError_t launch_tn(const RouteArgs& a, int TN, dim3 grid, dim3 block, size_t smem,
                            hipStream_t s) {
  if (TN == 1) return launch_one<BF16, TM, 1>(a, grid, block, smem, s);
  if constexpr (TM == 1) {                       // (two token tiles take at most two of router rows)
    if (TN == 3) return launch_one<BF16, TM, 3>(a, grid, block, smem, s);
    if (TN == 5) return launch_one<BF16, TM, 5>(a, grid, block, smem, s);
  }
  return launch_one<BF16, TM, 2>(a, grid, block, smem, s);
}

// Split form: used for at most kSplitMaxT tokens; the workspace holds split_most() (up to 256 tokens
// kSplitMax) partial sums of every logit.  (Above 2048 tokens every
// second compute unit has a workgroup, and two kernels without a split took 28 us where one took 23: 4096
// tokens, d = 2048.)
constexpr int kSplitMaxT = 2048;

// The most workgroups along d for T tokens: a power of two that keeps the launch within one workgroup per
// compute unit (half of that for decode-sized calls, whose second kernel pays for every partial sum).
static int split_most(int T) {
  const int blocks = (T + 15) / 16, room = T <= 256 ? 128 : 256;
  int ds = 1;
  while (ds * 2 <= kSplitMax && blocks * ds * 2 <= room) ds *= 2;
  return ds;
}
static int tile_cus() {
  static std::atomic<int> known{0};       // (GPUs of one kind: any thread's answer serves)
  int n = known.load(std::memory_order_relaxed);
  if (!n) {
    int dev = 0;
    hipDeviceProp_t p;
    n = (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess && p.multiProcessorCount > 0)
            ? p.multiProcessorCount : 256;
    known.store(n, std::memory_order_relaxed);
  }
  return n;
}

// column tiles of 16 router rows: in all, and per pass of the bf16 matrix-core form
static int router_tiles(const LayerDesc& L) { return (L.Ng + L.Ne + 15) / 16; }
static int pass_tiles(const LayerDesc& L) { const int t = router_tiles(L); return t >= 5 ? 5 : t; }

// The bf16 matrix-core form: bf16 tokens, enough of them, whole 128-deep chunks.  Up to 4096 tokens every compute unit has one
// workgroup of the fp32 form; beyond, some have two.  The fp32 form stays up to 8191 tokens where there is little to
// multiply: with one column tile, and with two of a short reduction.  Whole call in us, fp32 form / this, 4097 and 8191
// tokens: one tile, d = 128 6.4 / 11.6 and 7.3 / 11.5, d = 4096 20 / 23 and 25 / 31; two tiles (27 rows), d = 256 12.6 / 13.1 and
// 13.6 / 14.7, d = 512 14.7 / 14.3 and 16.1 / 16.2, d = 4096 39.5 / 28 and 45.5 / 35; 68 rows, d = 1024 32.5 / 23 and 34.5 / 26.
static bool prefill_form(const LayerDesc& L, int dtype) {
  if (dtype != MOHGE_BF16 || L.T <= 4096 || L.d % kPfDepth != 0) return false;
  const int tiles = router_tiles(L);
  return L.T >= 8192 || tiles > 2 || (tiles == 2 && L.d >= 512);
}

// How the bf16 matrix-core form runs: token groups of 16 per workgroup, and whether it selects itself.  Whole call in us,
// itself / with the second kernel, tokens per workgroup as chosen; 32 and 64 tokens per compute unit are whole rounds:
//   more than 64 per unit: itself with 64 tokens where two workgroups share a unit, up to two tiles (32768 tokens: 10 rows,
//     d = 128 20.5 / 24, d = 2048 38.6 / 44; 27 rows 24 / 30, 46 / 55), else the second kernel (68 rows, d = 1024 80 / 63)
//   32 to 64: one tile itself, with 32 tokens (12000 tokens: d = 128 13.1 / 14.6, d = 2048 23.2 / 24.1), unless d is large (d = 4096
//     39 / 35); two tiles in the last quarter, where the second kernel has the most to do (d = 1024: 12000 tokens 22.5 / 22.1, 16384
//     22.9 / 24.6; d = 2048 30.9 / 30.9); three while the reduction is short (16384 tokens: d = 128 16.6 / 19.6, d = 512
//     21.3 / 23.1, d = 1024 26.4 / 26.7, 12000 tokens 26 / 24); more: the second kernel (68 rows, 16384 tokens, d = 128 29 / 25)
//   up to 32: one tile itself unless d is large (8192 tokens, d = 128 11.5 / 13.2, d = 1024 15.2 / 15.8, d = 3072 24.5 / 22.9); two
//     and three while the reduction is short (8192 tokens, 40 rows: d = 128 14.0 / 15.3, d = 512 17.1 / 17.6, d = 1024 20.6 / 20.2);
//     more: the second kernel (68 rows, d = 128 18.4 / 18.8, d = 1024 28.4 / 26.0; 4097 tokens 18.3 / 15.8)
struct PrefillPlan { int tg; bool sel; };
static PrefillPlan prefill_plan(const LayerDesc& L, int cus) {
  const int tn = pass_tiles(L);
  if (L.T > 64ll * cus) return {4, tn <= 2};
  if (L.T <= 32ll * cus) return {2, tn == 1 ? L.d < 2048 : tn <= 3 && 16ll * L.d <= L.T};
  if (tn == 1 ? L.d < 4096 : tn == 2 ? L.T > 48ll * cus && L.d < 2048 : tn == 3 && 20ll * L.d <= L.T) return {2, true};
  return {4, false};
}

static size_t plane_bytes(size_t rows, int d) { return (3 * rows * d * sizeof(uint16_t) + 255) / 256 * 256; }

size_t route_workspace_bytes(const LayerDesc& L, int dtype) {
  if (prefill_form(L, dtype)) {
    // the three bf16 planes of the router rows, rows padded to whole passes of 16 * TN, and the logits
    const int tiles = router_tiles(L), TNp = pass_tiles(L);
    const size_t rows = (size_t)(tiles + TNp - 1) / TNp * TNp * 16;
    return plane_bytes(rows, L.d) + ((size_t)L.T * (L.Ng + L.Ne) * sizeof(float) + 255) / 256 * 256;
  }
  if (L.T > kSplitMaxT) return 0;
  const int most = L.T <= 256 ? kSplitMax : split_most(L.T);
  return ((size_t)most * (L.T > 0 ? L.T : 1) * (L.Ng + L.Ne) * sizeof(double) + 255) / 256 * 256;
}

hipError_t launch_route(const LayerDesc& L, int dtype, const void* x, const float* w_group,
                        const float* w_expert, const float* bias, int32_t* group_idx,
                        int32_t* expert_idx, float* gates, float* gs_out, float* es1_out,
                        void* ws, size_t ws_bytes, hipStream_t s) {
  RouteArgs a;
  a.x = x; a.wg = w_group; a.we = w_expert; a.bias = bias;
  a.gidx = group_idx; a.eidx = expert_idx; a.gates = gates; a.gs = gs_out; a.es1 = es1_out;
  a.T = L.T; a.d = L.d; a.Ng = L.Ng; a.N = L.N; a.Ne = L.Ne; a.Kg = L.Kg; a.Ke = L.Ke;
  a.mode = L.select_mode;
  a.NO = L.Ng + L.Ne;
  a.NOpad = ((a.NO + 15) / 16) * 16 + 4;
  a.Nepad = ((L.Ne + 63) / 64) * 64;
  // Slices of the hidden dimension, whole 32-element steps: one per wave, eight waves.  Few tokens: spread over more
  // workgroups as well, down to one step.  (With equal slices only, two or four waves where d is no multiple of 256 and
  // no spreading where the slices would not stay whole: d = 1344, 30 router rows, 32 to 1000 tokens 52 us, now 13; d = 2560, 66
  // rows, 23, now 17; d = 128, 15 rows, where four waves more share the selection, 10, now 7.)
  constexpr int NW = 8;
  const int steps = L.d / 32;
  a.dsplit = 1;
  a.gpart = nullptr;
  a.glog = nullptr;
  if (ws && L.T <= kSplitMaxT && ws_bytes >= route_workspace_bytes(L, dtype)) {
    const int most = split_most(L.T);
    while (a.dsplit * 2 <= most && NW * a.dsplit * 2 <= steps) a.dsplit *= 2;
    if (a.dsplit > 1) a.gpart = static_cast<double*>(ws);
  }
  a.kslice = 32 * ((steps + NW * a.dsplit - 1) / (NW * a.dsplit));
  const int tiles = router_tiles(L);
  // many bf16 tokens and a workspace for the split router rows: the bf16 matrix-core form
  if (prefill_form(L, dtype) && ws && ws_bytes >= route_workspace_bytes(L, dtype)) {
    const int TNp = pass_tiles(L);
    const int plane_rows = (tiles + TNp - 1) / TNp * TNp * 16;
    uint16_t* planes = static_cast<uint16_t*>(ws);
    const long long quads = (long long)plane_rows * (L.d / 4);
    hipLaunchKernelGGL(route_split_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, w_group, w_expert,
                       planes, L.Ng, a.NO, plane_rows, L.d);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.glog = reinterpret_cast<float*>(static_cast<unsigned char*>(ws) + plane_bytes(plane_rows, L.d));
    const PrefillPlan plan = prefill_plan(L, tile_cus());
    auto logits = [&]() {
      if (plan.sel) {
        switch (TNp * 2 + (plan.tg == 4)) {
          case 2: return launch_prefill<2, 1, true>(a, planes, plane_rows, s);
          case 3: return launch_prefill<4, 1, true>(a, planes, plane_rows, s);
          case 4: return launch_prefill<2, 2, true>(a, planes, plane_rows, s);
          case 5: return launch_prefill<4, 2, true>(a, planes, plane_rows, s);
          default: return launch_prefill<2, 3, true>(a, planes, plane_rows, s);
        }
      }
      switch (TNp * 2 + (plan.tg == 4)) {
        case 2: return launch_prefill<2, 1, false>(a, planes, plane_rows, s);
        case 3: return launch_prefill<4, 1, false>(a, planes, plane_rows, s);
        case 4: return launch_prefill<2, 2, false>(a, planes, plane_rows, s);
        case 5: return launch_prefill<4, 2, false>(a, planes, plane_rows, s);
        case 6: return launch_prefill<2, 3, false>(a, planes, plane_rows, s);
        case 7: return launch_prefill<4, 3, false>(a, planes, plane_rows, s);
        case 8: return launch_prefill<2, 4, false>(a, planes, plane_rows, s);
        case 9: return launch_prefill<4, 4, false>(a, planes, plane_rows, s);
        case 10: return launch_prefill<2, 5, false>(a, planes, plane_rows, s);
        default: return launch_prefill<4, 5, false>(a, planes, plane_rows, s);
      }
    };
    e = logits();
    if (e != hipSuccess || plan.sel) return e;
    a.region0 = (int)((size_t)NW * 5 * a.Nepad * sizeof(float));
    const size_t smem_f = (size_t)a.region0 + (size_t)kPrefillTokens * a.NOpad * sizeof(float);
    hipLaunchKernelGGL((route_finish_kernel<kPrefillTokens, false>), dim3((L.T + kPrefillTokens - 1) / kPrefillTokens),
                       dim3(64 * NW), smem_f, s, a);
    return hipGetLastError();
  }
  // Column tiles of 16 router rows per workgroup.  Split form, few tokens: one, and the passes over the router rows side by
  // side: what counts is the length of a wave's chain (one after the other with up to five: d = 4096, 68 rows, 32
  // tokens 12.9 us, now 10.0, 160 tokens 15.4 and 12.0; d = 1024, 136 rows, 32 tokens 21.7 and 14.1, 40 rows 9.7 and 8.5).  It
  // pays while a pass leaves compute units free.  Time of one tile / of all in a workgroup, d = 512 to 8192, bf16 and fp32:
  // two tiles 0.88 to 0.96 up to 120 workgroups per pass, 0.95 to 1.12 from 136 on; three 0.85 to 0.97 up to 152, 1.06 to 1.16 from
  // 176 on; five 0.74 to 0.97 up to 152, 0.96 to 1.09 at 176 to 200; more 0.5 to 0.98 up to 176, 0.9 to 1.06 at 200.  (Two tiles
  // per workgroup, side by side: 1.15 to 1.25 where five are 1.0.)
  int TN = tiles <= 1 ? 1 : tiles == 2 ? 2 : tiles == 3 ? 3 : 5;
  if (a.dsplit > 1 && L.T <= 400 && (L.T + 15) / 16 * a.dsplit <= (tiles == 2 ? 128 : 160)) TN = 1;
  const int passes = a.dsplit > 1 ? (tiles + TN - 1) / TN : 1;
  int TM = (L.T >= 16384 && TN <= 2) ? 2 : 1;   // wider combinations would spill registers
  size_t smem = 0;
  for (;; TM = 1) {
    const size_t part_bytes = (size_t)NW * 16 * TM * 16 * TN * sizeof(double);
    const size_t rows_bytes = (size_t)NW * 5 * a.Nepad * sizeof(float);
    a.region0 = (int)(((part_bytes > rows_bytes ? part_bytes : rows_bytes) + 15) / 16 * 16);
    smem = (size_t)a.region0 + (size_t)16 * TM * a.NOpad * sizeof(float);
    if (smem <= 96 * 1024 || TM == 1) break;
  }
  const int BT = 16 * TM;
  dim3 grid((L.T + BT - 1) / BT, a.dsplit, passes), block(64 * NW);
  const bool bf = dtype == MOHGE_BF16;
  hipError_t e;
  if (TM == 2) e = bf ? launch_tn<true, 2>(a, TN, grid, block, smem, s)
                      : launch_tn<false, 2>(a, TN, grid, block, smem, s);
  else e = bf ? launch_tn<true, 1>(a, TN, grid, block, smem, s)
              : launch_tn<false, 1>(a, TN, grid, block, smem, s);
  if (e != hipSuccess || a.dsplit == 1) return e;
  // (its own LDS, at most 45 KB: the first kernel's partial totals would leave room for one workgroup per compute unit)
  a.region0 = (int)((size_t)NW * 5 * a.Nepad * sizeof(float));
  smem = (size_t)a.region0 + (size_t)kFinishTokens * a.NOpad * sizeof(float);
  hipLaunchKernelGGL((route_finish_kernel<kFinishTokens, true>), dim3((L.T + kFinishTokens - 1) / kFinishTokens), block, smem, s, a);
  return hipGetLastError();
}

}  // namespace mohge
