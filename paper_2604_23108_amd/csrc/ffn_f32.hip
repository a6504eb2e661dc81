// Expert feed-forward networks of a layer stored in fp32, on gfx950: a ragged grouped GEMM on the
// fp32 matrix cores (v_mfma_f32_32x32x2_f32, v_mfma_f32_16x16x4_f32), one launch per projection.
//
// What bounds it: the fp32 matrix rate, 256 FLOP per clock and compute unit (a sixteenth of bf16),
// and the vector instructions beside it, which the fp32 MFMA does not run in parallel with: eight of them take 522 clocks of a
// SIMD, with the 48 additions and conversions that their sums need 790, however many waves there are (a loop of
// nothing else); so every vector instruction in the main loop counts.
// Down to a few rows per expert it is the weight stream.  An MFMA keeps a SIMD busy for 64
// clocks on two operand registers, so operand delivery is never the limit and the tile is chosen for
// balance: 32 token rows (or 16, the last of an expert) x 64 weight rows (up: 32 W_gate rows and the matching 32 W_up rows), so that
// partial row blocks cost little and a layer of 3072 routed rows gives every compute unit several
// tiles.  Four waves: two weight fragments x two halves of every stage's reduction indices, which
// meet in LDS at the end.
// Measured on 512 tokens, d = 1024, 32 experts of width 256..896, six per token (10.9 GFLOP): both projections
// take 188 us (58 TFLOP/s of a possible 154; 179 with its sums in fp32 alone, see below), the one-wave-per-output
// dot products that this replaced 1.42 ms.  One 64-bit addition per request's address instead of two: the layer call 203 -> 199.  At 4096 tokens of a d = 2048 layer it runs at 84 TFLOP/s.
// (With fp32 sums, 64-row tiles were 8 % slower on the first, whose whole tiles divide worse over the compute units,
// and 6 % faster on the second.)
//
// Operands go global -> LDS (global_load_lds, 256-byte row segments, 16-byte pieces XOR-swizzled by
// the row) through two stages of 64 reduction indices (48 KB: three workgroups per compute unit), one
// barrier per stage; the fragments of a stage are in registers while the next but one is on its way.
// A lane's 128-bit fragment read holds four consecutive reduction indices of one row and feeds four
// MFMAs; both operands use the same assignment.  Sixteen indices make two groups: the first two of each four, then the last two.
//
// Every product of an MFMA rounds the running sum, so a chain of n products carries about n/2 roundings.  A chain
// here is the eight products of one such group; the sums of two groups are added, and the pairs go into an fp64
// total that is rounded once: 6.5 roundings for any length of the reduction.  The conversions and fp64 additions of
// a pair run under the MFMAs of the next one (every group folded by itself, behind its MFMAs: 144 us instead of 130 at
// 300 tokens of the layer above).
// Error of the two projections against float64 (2-norm), 64 to 4096 indices: 1.22e-7 to 1.24e-7 (tiles of at most 16 rows 1.12e-7 to
// 1.28e-7); with fp32 chains of
// 64 in a second fp32 set it was 2.1e-7 and 3.1e-7, with the dot products (a sum spread over 64 lanes, then a
// butterfly) 1.26e-7 and 2.6e-7.
//
// Why not the bf16 matrix cores, with every operand split into three bf16 parts: 512 tokens of the layer above took 139 us
// instead of 188 with the six largest of the nine products, 153 with eight.  But v_mfma_f32_32x32x16_bf16 cuts off what lies
// below its largest addend instead of rounding it, always downwards: one projection of 4096 indices with every 97th
// channel a thousand times as large was off by 8.8e-8, 70 % of it one-sided drift, 16384 indices by 1.2e-7 (here 6.5e-8, no
// drift); chains short enough to stop that cost what the products save.  Below 2^-110 the third part falls under the smallest
// bf16 number (2e-6 at 2^-116), and a launch of one round of workgroups, any layer at one token, was 1.2 times as long.
//
// No schedule launch: a workgroup finds the expert of its row tile from `offsets` with a wave-wide
// scan.  The grid covers the largest possible number of row tiles; the ones that do not exist exit.
#include "common.h"

namespace mohge {

typedef float f32v4 __attribute__((ext_vector_type(4)));   // (fragment reads as HIP's float4 struct make the
                                                          //  compiler wait for all LDS-bound loads first)
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct F32Args {
  const float* A;                 // up: x; down: H
  const int32_t* perm;            // up only, may be NULL
  const int32_t* offsets;
  const float* W[kMaxGroups];
  float* C;
  int lda, ldc, Ke, N, Ne, d, P;
  int ntm, ntn;                   // row tiles (upper bound) and column tiles (of the widest group)
  int F[kMaxGroups];
  int order[kMaxGroups];          // groups by decreasing width: the longest down tiles start first
};

constexpr int kFM = 32, kFN = 64, kFK = 64;            // tile rows (tokens), weight rows, reduction depth of a stage
constexpr int kFW = 4;                                 // waves: two weight fragments x kFW/2 parts of a stage
constexpr int kFStage = (kFM + kFN) * kFK * 4;         // 24 KB
constexpr int kFStages = 2;
constexpr int kFChunks = kFK / 4;                      // 16-byte pieces of a stage row
constexpr int kFKW = 2 * kFK / kFW;                    // reduction indices of a stage per wave

__device__ __forceinline__ void f32_copy16(const float* g, unsigned char* lds_uniform_base) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)lds_uniform_base, 16, 0, 0);
}

// expert, first sorted row and row count of row tile m; false if there is no such tile.  The same in
// every lane; called by whole waves.
__device__ __forceinline__ bool f32_row_tile(const F32Args& a, int m, int lane, int& e, int& row, int& rows) {
  int before = 0;
  for (int e0 = 0; e0 < a.Ne; e0 += 64) {
    const int v = e0 + lane;                             // position in visiting order
    const int ee = v < a.Ne ? a.order[v / a.N] * a.N + v % a.N : 0;
    const int lo = a.offsets[ee], cnt = v < a.Ne ? a.offsets[ee + 1] - lo : 0;
    const int nt = (cnt + kFM - 1) / kFM;
    const int incl = wave_incl_scan(nt);
    const int first = before + incl - nt;                // tiles before this expert
    const unsigned long long hit = __ballot(m >= first && m < first + nt);
    if (hit) {
      const int l = (int)__builtin_ctzll(hit);
      const int mi = m - __builtin_amdgcn_readlane(first, l);
      const int n = __builtin_amdgcn_readlane(cnt, l);
      e = __builtin_amdgcn_readlane(ee, l);
      row = __builtin_amdgcn_readlane(lo, l) + mi * kFM;
      rows = min(kFM, n - mi * kFM);
      return row >= 0 && rows > 0 && row + rows <= a.P;
    }
    before += __builtin_amdgcn_readlane(incl, 63);
  }
  return false;
}

// HALF: a tile of at most 16 rows.  32x32x2 would spend as long on 16 rows as on 32; 16x16x4 takes half the time for the same
// products, at the same rate.  Both add up the same groups of eight in the same order, so that the bits of a row do not depend on
// how full its tile is (a test compares them).  (For 32 rows too it was 1.5 to 2.5 % slower: twice the MFMAs.)  Layer
// call before / now: 9 tokens of 25 experts, d = 1344, 102 / 77 us, 60 tokens 105 / 85; 60 tokens of 32 experts, d = 1024, 94 / 76, 512 tokens 202 / 197.
template <bool UP, bool HALF>
__device__ __forceinline__ void f32_tile(const F32Args& a, unsigned char* lds, int e, int row, int rows, int n0,
                                         int w, int lane) {
  const int g = e / a.N, i = e % a.N, F = a.F[g], K = UP ? a.d : F;
  const int ncols = UP ? F : a.d;
  // wave-wide load j fills stage rows 4*(4j + w) .. +3: first the token rows, then the weight rows;
  // lane l fills row l/16, physical piece l%16, which holds logical piece (l%16) ^ (row & 15)
  constexpr int TM = HALF ? 16 : kFM;                            // token rows in LDS
  constexpr int RPL = 64 / kFChunks;                             // rows of a wave-wide load
  constexpr int TLOADS = TM / (RPL * kFW), LOADS = TLOADS + kFN / (RPL * kFW);   // loads per thread and stage: tokens, all
  const float* src[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int r = RPL * (kFW * j + w) + lane / kFChunks;
    const int piece = (lane % kFChunks) ^ (r & 15);
    if (j < TLOADS) {
      const int pos = row + (r < rows ? r : rows - 1);         // rows past the end: any valid row
      const long long s = UP && a.perm ? (long long)(a.perm[pos] / a.Ke) : (long long)pos;
      src[j] = a.A + s * a.lda + piece * 4;
    } else {
      const int b = r - TM;
      long long wrow;
      if constexpr (UP) {
        // weight rows of a wave: 16 of W_gate, then the matching 16 of W_up
        int f = n0 + 16 * (b >> 5) + (b & 15);
        if (f > F - 1) f = F - 1;
        wrow = (long long)i * 2 * F + ((b & 16) ? F : 0) + f;
      } else {
        int n = n0 + b;
        if (n > a.d - 1) n = a.d - 1;
        wrow = (long long)i * a.d + n;
      }
      src[j] = a.W[g] + wrow * K + piece * 4;
    }
  }
  const int KT = K / kFK;                                        // K is a multiple of 64
  // stages are requested in order: running pointers, one vector addition per request
  auto issue = [&](int kt) {
    unsigned char* dst = lds + (kt % kFStages) * kFStage + w * 1024;
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      f32_copy16(src[j], dst + j * kFW * 1024);
      src[j] += kFK;
    }
  };
#pragma unroll
  for (int kt = 0; kt < kFStages; ++kt)
    if (kt < KT) issue(kt);

  // wave: weight fragment wn (32 rows), and of every stage the reduction indices [kFKW kq, kFKW kq + kFKW)
  const int wn = w & 1, kq = w >> 1;
  // A lane's 128-bit read: piece fh of the PK pieces that a group of MFMAs takes, of fragment row fr
  constexpr int FR = HALF ? 16 : 32, PK = 64 / FR;
  const int fr = lane % FR, fh = lane / FR, sw = fr & 15;
  constexpr int NK = kFKW / (4 * PK), NW = 32 / FR;              // groups of a stage; weight fragments of a wave
  struct Frags { f32v4 b[NK][NW], x[NK]; };
  auto read = [&](int kt, Frags& f) {
    const unsigned char* st = lds + (kt % kFStages) * kFStage;
    const unsigned char* pa = st + fr * (kFK * 4);
    const unsigned char* pb = st + (TM + 32 * wn + fr) * (kFK * 4);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int off = ((PK * (NK * kq + k) + fh) ^ sw) << 4;
#pragma unroll
      for (int i = 0; i < NW; ++i) f.b[k][i] = *reinterpret_cast<const f32v4*>(pb + FR * i * (kFK * 4) + off);
      f.x[k] = *reinterpret_cast<const f32v4*>(pa + off);
    }
  };
  // total so far, and the sum of the last two groups of eight products, not in it yet
  constexpr int NS = HALF ? 8 : 16;
  double tot[NS];
  float pair[NS];
#pragma unroll
  for (int r = 0; r < NS; ++r) { tot[r] = 0.0; pair[r] = 0.f; }
  auto fold = [&]() {
#pragma unroll
    for (int r = 0; r < NS; ++r) tot[r] += (double)pair[r];
  };
  // the sums of two groups of eight products each, added: a group is four MFMAs, HALF two for each weight fragment (not in a
  // row, they would wait for each other)
  auto multiply = [&](const Frags& use, int k) {
    if constexpr (HALF) {
      f32v4 n[2][NW];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < NW; ++i) {
          const int e = c < 2 ? 2 * c : 2 * c - 3;               // elements 0 and 1 make the first group, 2 and 3 the second
          n[c & 1][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(use.b[k][i][e], use.x[k][e], c < 2 ? f32v4{0.f, 0.f, 0.f, 0.f} : n[c & 1][i], 0, 0, 0);
        }
      fold();
#pragma unroll
      for (int r = 0; r < NS; ++r) pair[r] = n[0][r / 4][r % 4] + n[1][r / 4][r % 4];
    } else {
      f32x16 n0, n1;
#pragma unroll
      for (int r = 0; r < 16; ++r) { n0[r] = 0.f; n1[r] = 0.f; }
#pragma unroll
      for (int c = 0; c < 4; ++c)
        n0 = __builtin_amdgcn_mfma_f32_32x32x2f32(use.b[k + c % 2][0][c / 2], use.x[k + c % 2][c / 2], n0, 0, 0, 0);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        n1 = __builtin_amdgcn_mfma_f32_32x32x2f32(use.b[k + c % 2][0][2 + c / 2], use.x[k + c % 2][2 + c / 2], n1, 0, 0, 0);
      fold();
#pragma unroll
      for (int r = 0; r < NS; ++r) pair[r] = n0[r] + n1[r];
    }
    // the previous pair is folded under the MFMAs of this one
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);             // one MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 2 * NS / 8, 0);    // its share of the conversions and additions
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Stage kt, whose fragments are in `use`: once the loads of stage kt+1 have landed everywhere its
  // fragments are read into `nxt` (under the MFMAs of stage kt), and stage kt+2 is requested into the
  // slot of stage kt, which every wave has in registers by the barrier.
  auto stage = [&](int kt, Frags& use, Frags& nxt) {
    if (kt + 1 < KT) {
      // (a plain barrier: __syncthreads() would also wait for the loads of later stages)
      if (kt + kFStages - 1 < KT) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((kFStages - 2) * LOADS) : "memory");
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      read(kt + 1, nxt);
      // behind the reads in program order: in front of them the compiler waits for the loads first
      __builtin_amdgcn_sched_barrier(0);
      if (kt + kFStages < KT) issue(kt + kFStages);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int k = 0; k < NK; k += HALF ? 1 : 2) multiply(use, k);
  };
  Frags f0, f1;
  if (KT >= kFStages) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kFStages - 1) * LOADS) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  read(0, f0);
  for (int kt = 0; kt < KT; kt += 2) {
    stage(kt, f0, f1);
    if (kt + 1 < KT) stage(kt + 1, f1, f0);
  }
  fold();
  // The two halves of the reduction meet in LDS and are added in order.
  __syncthreads();                                               // the stages have been read
  double* ex = reinterpret_cast<double*>(lds) + wn * 1024;       // [wn][NS][64]
  if (kq == 1)
#pragma unroll
    for (int r = 0; r < NS; ++r) ex[r * 64 + lane] = tot[r];
  __syncthreads();
  // accumulator r of a lane: token fr, weight row STEP*(r/4) + 4*fh + r%4 of the wave's 32
  constexpr int NQ = NS / 4, STEP = 32 / NQ;
  if (kq == 1 || fr >= rows) return;
  float sum[NS];
#pragma unroll
  for (int r = 0; r < NS; ++r) sum[r] = (float)(tot[r] + ex[r * 64 + lane]);
  float* crow = a.C + (long long)(row + fr) * a.ldc;
  if constexpr (UP) {
#pragma unroll
    for (int q = 0; q < NQ / 2; ++q) {
      const int col = n0 + 16 * wn + STEP * q + 4 * fh;
      float h[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float gt = sum[4 * q + j], up = sum[NS / 2 + 4 * q + j];
        h[j] = gt / (1.f + expf(-gt)) * up;
      }
      if (col < ncols) *reinterpret_cast<float4*>(crow + col) = make_float4(h[0], h[1], h[2], h[3]);
    }
  } else {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int col = n0 + 32 * wn + STEP * q + 4 * fh;
      if (col < ncols)
        *reinterpret_cast<float4*>(crow + col) = make_float4(sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]);
    }
  }
}

template <bool UP>
__global__ void __launch_bounds__(64 * kFW, 3) ffn_f32_kernel(const F32Args a) {
  extern __shared__ __align__(1024) unsigned char lds[];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // The hardware hands workgroups to the 8 XCDs in turn (a row of the grid is a multiple of 8 long): four neighbouring
  // row tiles of one column tile (mostly one expert's: one weight panel) go to the same XCD.
  const int wg = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  const int xcd = wg % 8, idx = wg / 8;
  const int tile = ((idx / 4) * 8 + xcd) * 4 + idx % 4;
  const int m = tile % a.ntm, n = tile / a.ntm;
  if (n >= a.ntn) return;
  int e, row, rows;
  if (!f32_row_tile(a, m, lane, e, row, rows)) return;
  const int n0 = n * (UP ? kFN / 2 : kFN);
  if (n0 >= (UP ? a.F[e / a.N] : a.d)) return;
  if (rows > 16) f32_tile<UP, false>(a, lds, e, row, rows, n0, w, lane);
  else f32_tile<UP, true>(a, lds, e, row, rows, n0, w, lane);
}

// Workgroups in rows of at most kFGridX: a launch has fewer than 2^32 threads per grid dimension, which a call with
// 64 GiB of hidden activations exceeds in one.
constexpr long long kFGridX = 1ll << 20;

template <bool UP>
static hipError_t launch_f32(F32Args& a, hipStream_t s) {
  constexpr int smem = kFStages * kFStage;
  static_assert(smem <= 64 * 1024 && 2 * 16 * 64 * (int)sizeof(double) <= smem, "dynamic LDS without the opt-in; the sums");
  const long long wgs = ((long long)a.ntm * a.ntn + 31) / 32 * 32;
  const long long gx = wgs < kFGridX ? wgs : kFGridX, gy = (wgs + gx - 1) / gx;
  if (gx * gy >= 1ll << 31) return hipErrorInvalidConfiguration;   // (terabytes of activations)
  hipLaunchKernelGGL(ffn_f32_kernel<UP>, dim3((unsigned)gx, (unsigned)gy), dim3(64 * kFW), smem, s, a);
  return hipGetLastError();
}

hipError_t launch_ffn_f32(const LayerDesc& L, const void* x, const int32_t* perm, const int32_t* offsets,
                          const GroupPtrs& W, void* y_perm, void* ws, hipStream_t s, int stages) {
  if (L.P == 0) return hipSuccess;
  F32Args up;
  up.A = static_cast<const float*>(x);
  up.perm = perm; up.offsets = offsets;
  up.C = static_cast<float*>(ws);
  up.lda = L.d; up.ldc = L.Fmax; up.Ke = L.Ke; up.N = L.N; up.Ne = L.Ne; up.d = L.d; up.P = L.P;
  // every expert with rows adds at most one partial tile
  const long long live = L.P < L.Ne ? L.P : L.Ne;
  up.ntm = (int)(((long long)L.P + (kFM - 1) * live) / kFM);
  up.ntn = (L.Fmax + kFN / 2 - 1) / (kFN / 2);
  F32Args dn = up;
  dn.A = static_cast<const float*>(ws);
  dn.perm = nullptr;
  dn.C = static_cast<float*>(y_perm);
  dn.lda = L.Fmax; dn.ldc = L.d;
  dn.ntn = (L.d + kFN - 1) / kFN;
  for (int g = 0; g < kMaxGroups; ++g) up.order[g] = g;
  for (int i = 1; i < L.Ng; ++i)
    for (int j = i; j > 0 && L.F[up.order[j]] > L.F[up.order[j - 1]]; --j) {
      const int t = up.order[j]; up.order[j] = up.order[j - 1]; up.order[j - 1] = t;
    }
  for (int g = 0; g < kMaxGroups; ++g) dn.order[g] = up.order[g];
  for (int g = 0; g < kMaxGroups; ++g) {
    up.F[g] = dn.F[g] = g < L.Ng ? L.F[g] : 0;
    up.W[g] = static_cast<const float*>(W.w13[g]);
    dn.W[g] = static_cast<const float*>(W.w2[g]);
  }
  hipError_t e = hipSuccess;
  if (stages & 1) e = launch_f32<true>(up, s);
  if (e == hipSuccess && (stages & 2)) e = launch_f32<false>(dn, s);
  return e;
}

}  // namespace mohge
