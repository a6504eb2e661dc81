// Expert feed-forward networks of a layer stored in fp32, on gfx950: a ragged grouped GEMM, one launch per
// projection, on the bf16 matrix cores with every fp32 operand split into three bf16 parts.
//
// The fp32 matrix instructions run at a sixteenth of the bf16 rate.  An fp32 number is the sum of three bf16 numbers
// (x rounded to bf16, the remainder rounded to bf16, the rest: exact, the remainders need no more bits), the product of
// two bf16 numbers is exact in fp32, and of the nine products of two such sums six matter: the others (mid.lo, lo.mid,
// lo.lo) are below 2^-26 of the product.  Six bf16 products cost 3/8 of one fp32 product.
//
// What bounds it: up to a few rows per expert the weight stream; beyond that, about equally, the products, the
// conversions (11 instructions per pair of values), the copies to LDS and what a tile pays before and after its main
// loop.  Tile: 32 token rows x 128 weight rows (up: 64 of W_gate and the matching 64 of W_up) in stages of 32 reduction
// indices; four waves: two halves of the weight rows x two halves of every stage, so that each wave splits what it
// multiplies and nothing but the tokens is split twice.  Two workgroups per compute unit cover each other's prologue
// and epilogue.  64 token rows per tile need more than half of the registers, so one workgroup per unit: 138 -> 154 us on
// the case below, 59 -> 70 at 9 to 68 tokens; without the interleaving described at stage() 182.
// Measured on 512 tokens, d = 1024, 32 experts of width 256..896, six per token (10.9 GFLOP), both projections: 138 us;
// on the fp32 matrix cores 188.  68 tokens of that layer 80 -> 61 us (3.7 TB/s of weights), 4096 tokens of a d = 2048
// layer 2420 -> 1630 us.  64 tokens of a layer of d = 128 and widths of 64 to 256, where a launch is a chain of latencies,
// 15 -> 18.5.
//
// Operands go global -> LDS (128-byte row segments, 16-byte pieces XOR-swizzled by the row) through four stages, three of
// them in flight, one barrier per stage.
//
// Error: the matrix instruction rounds once per eight products, and a chain here is four stages of 16 indices: 4.5
// roundings.  Chains are added with compensation (what the addition rounds away starts the next chain), the five small
// products have accumulators of their own, the halves of a stage meet in fp64 and SiLU(a) b is evaluated in fp64.
// Against float64 (2-norm of both projections) 6.2e-8 at 64 indices, 9.2e-8 from 1024 to 4096; on the fp32 matrix
// cores in chains of eight products with an fp64 total it was 1.21e-7 and 1.25e-7.  (Chains of eight stages: 1.28e-7,
// 2 % faster.)  A sum that is not finite, from an operand that is not or from the largest finite numbers, whose
// leading part rounds to infinity, is evaluated again as a plain dot product.
//
// No schedule launch: a workgroup finds the expert of its row tile from `offsets` with a wave-wide
// scan.  The grid covers the largest possible number of row tiles; the ones that do not exist exit.
#include "common.h"

namespace mohge {

typedef float f32v4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16v2 __attribute__((ext_vector_type(2)));
typedef float f32v2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32v4 __attribute__((ext_vector_type(4)));

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

constexpr int kFM = 32, kFN = 128, kFK = 32;           // token rows (at most), weight rows, reduction depth of a stage
constexpr int kFW = 4;                                 // waves: two halves of the weight rows x two halves of a stage
constexpr int kFStages = 4;
constexpr int kFStage = (kFM + kFN) * kFK * 4;         // 20 KB: two workgroups fill a compute unit's LDS
constexpr int kFChunk = 4;                             // stages per fp32 chain

// expert, first sorted row and row count of row tile m; false if there is no such tile.  The same in every lane; called by whole waves.
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

// Eight values of a row as three bf16 operand fragments
struct Split { u32v4 hi, mid, lo; };

// Splitting one pair of values, in seven steps of one to two independent instructions each: a wave's dependent
// instructions do not follow each other without a gap, so steps of different pairs are issued side by side.
struct PairSplit {
  float x0, x1, u0, u1;
  uint32_t h, m;
  __device__ __forceinline__ void step(int k, const f32v4 (&v)[2], Split& s, int j) {
    if (k == 0) { x0 = v[j >> 1][2 * (j & 1)]; x1 = v[j >> 1][2 * (j & 1) + 1]; h = pack_bf16x2(x0, x1); }
    if (k == 1) { u0 = __uint_as_float(h << 16); u1 = __uint_as_float(h & 0xffff0000u); }
    if (k == 2) { x0 -= u0; x1 -= u1; }
    if (k == 3) m = pack_bf16x2(x0, x1);
    if (k == 4) { u0 = __uint_as_float(m << 16); u1 = __uint_as_float(m & 0xffff0000u); }
    if (k == 5) { x0 -= u0; x1 -= u1; }
    if (k == 6) { s.hi[j] = h; s.mid[j] = m; s.lo[j] = pack_bf16x2(x0, x1); }
  }
};
constexpr int kSplitSteps = 7;

__device__ __forceinline__ f32x16 mfma_b(u32v4 a, u32v4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16v8, a), __builtin_bit_cast(bf16v8, b), c, 0, 0, 0);
}

// A dot product by a plain walk: for sums that are not finite.
__device__ __noinline__ double f32_plain_dot(const float* w, const float* x, int K) {
  double s = 0.0;
  for (int k = 0; k < K; ++k) s = fma((double)w[k], (double)x[k], s);
  return s;
}

// SiLU(a) b of finite numbers, rounded once.  exp(-a) = 2^n (1 + r + r^2 q(r)), |r| <= ln(2) / 2, q a Taylor polynomial in fp32
// (its part of the sum is below r^2, so that its rounding stays below 1e-8).
__device__ __forceinline__ float silu_times(double a, double b) {
  const double t = fmin(fmax(a * -1.4426950408889634, -1020.0), 1020.0);
  const double n = rint(t), r = (t - n) * 0.6931471805599453;
  const float f = (float)r;
  float q = fmaf(f, 2.4801587e-5f, 1.9841270e-4f);
  q = fmaf(f, q, 1.3888889e-3f);
  q = fmaf(f, q, 8.3333333e-3f);
  q = fmaf(f, q, 4.1666667e-2f);
  q = fmaf(f, q, 1.6666667e-1f);
  q = fmaf(f, q, 0.5f);
  const double den = 1.0 + ldexp(1.0 + (r + (double)(f * f * q)), (int)n);
  double inv = __builtin_amdgcn_rcp(den);
  inv = fma(inv, fma(-den, inv, 1.0), inv);
  return (float)(a * b * inv);
}

// 16 bytes per lane to LDS at a wave-uniform address, not modelled by the compiler (which would wait for every copy
// it knows of in front of a read of LDS); the destination is an operand in M0.
__device__ __forceinline__ void f32_copy16(const float* g, int lds_addr) {
  asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, off"
               ::"v"(g), "{m0}"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory");
}

template <bool UP>
__device__ __forceinline__ void f32_tile(const F32Args& a, unsigned char* lds, int e, int row, int rows, int n0, int w,
                                         int lane) {
  const int g = e / a.N, i = e % a.N, F = a.F[g], K = UP ? a.d : F;
  const bool half = !UP && n0 + kFN > a.d;                     // the last 64 columns of d = 64 (mod 128)
  // weight row b of the tile: up 16 rows of W_gate, then the matching 16 of W_up, and so on
  auto weight_row = [&](int b) -> const float* {
    if constexpr (UP) return a.W[g] + ((long long)i * 2 * F + ((b & 16) ? F : 0) + n0 + 16 * (b >> 5) + (b & 15)) * K;
    else return a.W[g] + ((long long)i * a.d + n0 + b) * K;
  };
  auto token_row = [&](int r) -> const float* {
    const int pos = row + (r < rows ? r : rows - 1);           // rows past the end: any valid row
    return a.A + (UP && a.perm ? (long long)(a.perm[pos] / a.Ke) : (long long)pos) * a.lda;
  };
  // A wave-wide copy fills 8 stage rows (128 bytes each): lane l row l/8, physical piece l%8, which holds logical
  // piece (l%8) ^ (row%8).  Wave w copies weight rows 32j + 8w .. +7 and token rows 8w .. +7.
  const int piece = ((lane & 7) ^ (lane >> 3)) * 4;
  const float* const src_w = weight_row(8 * w + (lane >> 3)) + piece;
  const float* const src_x = token_row(8 * w + (lane >> 3)) + piece;
  const long long wstep = (UP ? 16ll : 32ll) * K;
  constexpr int LOADS = kFN / 32 + 1;
  const int lds0 = (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)lds;
  auto issue = [&](int kt, int slot) {
    const int dst = lds0 + slot * kFStage + w * 1024;
#pragma unroll
    for (int j = 0; j < kFN / 32; ++j)
      f32_copy16(src_w + (half && j >= 2 ? j - 2 : j) * wstep + kt * kFK, dst + j * 4096);
    f32_copy16(src_x + kt * kFK, dst + kFN * kFK * 4);
  };
  const int KT = K / kFK;                                      // K is a multiple of 64: an even number of stages
  // (a request past the end repeats the last stage, so that every stage waits for the same number of copies)
#pragma unroll
  for (int kt = 0; kt < kFStages - 1; ++kt) issue(min(kt, KT - 1), kt);

  const int wm = w & 1, kq = w >> 1, fr = lane & 31, fh = lane >> 5;
  const int p0 = ((4 * kq + 2 * fh) ^ (fr & 7)) << 4, p1 = p0 ^ 16;
  const unsigned char* const pw = lds + (64 * wm + fr) * (kFK * 4);
  const unsigned char* const px = lds + (kFN + fr) * (kFK * 4);
  struct Raw { f32v4 v[3][2]; };                               // two weight fragments, the token fragment
  struct Planes { Split v[3]; };
  f32x16 big[2], small[2], tot[2];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int r = 0; r < 16; ++r) { big[f][r] = 0.f; small[f][r] = 0.f; tot[f][r] = 0.f; }
  int slot = 0;                                                // of the stage read next
  auto fetch = [&](int kt, Raw& raw) {                         // stage kt, once it has landed everywhere
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kFStages - 2) * LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int so = slot * kFStage;
#pragma unroll
    for (int f = 0; f < 3; ++f) {
      const unsigned char* p = f < 2 ? pw + so + f * 4096 : px + so;
      raw.v[f][0] = *reinterpret_cast<const f32v4*>(p + p0);
      raw.v[f][1] = *reinterpret_cast<const f32v4*>(p + p1);
    }
    // the slot of the stage before, which every wave had in registers by the barrier, takes a new one
    issue(min(kt + kFStages - 1, KT - 1), slot == 0 ? kFStages - 1 : slot - 1);
    slot = slot == kFStages - 1 ? 0 : slot + 1;
    __builtin_amdgcn_sched_barrier(0);
  };
  // product i of a stage: the six pairs of parts that matter, on both accumulators in turn
  auto product = [&](const Planes& p, int i) {
    const int k = i / 2, f = i % 2;
    const Split &b = p.v[f], &x = p.v[2];
    if (k == 0) small[f] = mfma_b(b.lo, x.hi, small[f]);
    if (k == 1) big[f] = mfma_b(b.hi, x.hi, big[f]);
    if (k == 2) small[f] = mfma_b(b.hi, x.lo, small[f]);
    if (k == 3) small[f] = mfma_b(b.mid, x.mid, small[f]);
    if (k == 4) small[f] = mfma_b(b.mid, x.hi, small[f]);
    if (k == 5) small[f] = mfma_b(b.hi, x.mid, small[f]);
  };
  constexpr int kProducts = 12, kPairs = 12;
  // compensated: what the addition rounds away starts the next chain
  auto fold = [&](int f, int r) {
    const float s = tot[f][r] + big[f][r];
    big[f][r] -= s - tot[f][r];
    tot[f][r] = s;
  };
  // The products of stage kt.  Under them stage kt+1 is read and split, a step of seven neighbouring pairs behind every
  // product, and one accumulator may be folded (its own product of this stage is long done by then).
  auto stage = [&](int kt, const Planes& now, Planes& next, int folded) {
    Raw raw;
    PairSplit ps[kPairs];
    fetch(kt + 1, raw);
#pragma unroll
    for (int i = 0; i < kProducts; ++i) {
      product(now, i);
      constexpr int first = 1, slots = kProducts - first;      // (the fragments are on their way during the first)
#pragma unroll
      for (int c = 0; c < kPairs; ++c)
#pragma unroll
        for (int k = 0; k < kSplitSteps; ++k)
          if (first + (c + k) * slots / (kPairs + kSplitSteps - 1) == i)
            ps[c].step(k, raw.v[c / 4], next.v[c / 4], c % 4);
      if (folded >= 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (5 + r * (kProducts - 5) / 16 == i) fold(folded, r);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  Planes pa, pb;
  {
    Raw raw;
    PairSplit ps[kPairs];
    fetch(0, raw);
#pragma unroll
    for (int k = 0; k < kSplitSteps; ++k)
#pragma unroll
      for (int c = 0; c < kPairs; ++c) ps[c].step(k, raw.v[c / 4], pa.v[c / 4], c % 4);
  }
  // (the last stage reads and splits itself once more: code for a stage without a next one costs more at short
  // reductions than it saves)
  static_assert(kFChunk == 4, "stages of the loop below");
  for (int kt = 0;;) {
    stage(kt, pa, pb, 0);
    stage(kt + 1, pb, pa, 1);
    if ((kt += 2) >= KT) break;
    stage(kt, pa, pb, -1);
    stage(kt + 1, pb, pa, -1);
    if ((kt += 2) >= KT) break;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the repeated copies
  // The two halves of the reduction meet in LDS in fp64: wave kq finishes weight fragment kq of its 64 rows.
  __syncthreads();                                             // the stages have been read
  double* const ex = reinterpret_cast<double*>(lds);           // [4 waves][16][64]
  double mine[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const double s0 = (double)tot[0][r] + ((double)big[0][r] + (double)small[0][r]);
    const double s1 = (double)tot[1][r] + ((double)big[1][r] + (double)small[1][r]);
    ex[(w * 16 + r) * 64 + lane] = kq ? s0 : s1;
    mine[r] = kq ? s1 : s0;
  }
  __syncthreads();
  if (fr >= rows || (half && wm)) return;
  const int f = 2 * wm + kq;
  // accumulator r of a lane: token lane%32, weight row 8*(r/4) + 4*(lane/32) + r%4 of the fragment's 32
  bool finite = true;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    mine[r] += ex[((w ^ 2) * 16 + r) * 64 + lane];
    finite = finite && __builtin_isfinite(mine[r]);
  }
  float* const crow = a.C + (long long)(row + fr) * a.ldc + n0 + (UP ? 16 : 32) * f + 4 * fh;
  if (!finite) {
#pragma unroll 1
    for (int c = 0; c < (UP ? 8 : 16); ++c) {
      const int col = 8 * (c >> 2) + (c & 3);
      const float* wr = weight_row(32 * f + col + 4 * fh);
      const double v = f32_plain_dot(wr, token_row(fr), K);
      if constexpr (UP) {
        const double u = f32_plain_dot(wr + (long long)F * K, token_row(fr), K);
        const float gt = (float)v;
        crow[col] = __builtin_isfinite(v) && __builtin_isfinite(u) ? silu_times(v, u) : gt / (1.f + expf(-gt)) * (float)u;
      } else {
        crow[col] = (float)v;
      }
    }
    return;
  }
  if constexpr (UP) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      *reinterpret_cast<float4*>(crow + 8 * q) =
          make_float4(silu_times(mine[4 * q], mine[8 + 4 * q]), silu_times(mine[4 * q + 1], mine[9 + 4 * q]),
                      silu_times(mine[4 * q + 2], mine[10 + 4 * q]), silu_times(mine[4 * q + 3], mine[11 + 4 * q]));
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(crow + 8 * q) =
          make_float4((float)mine[4 * q], (float)mine[4 * q + 1], (float)mine[4 * q + 2], (float)mine[4 * q + 3]);
  }
}

template <bool UP>
__global__ void __launch_bounds__(64 * kFW, 2) ffn_f32_kernel(const F32Args a) {
  extern __shared__ __align__(1024) unsigned char lds[];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long wg = (long long)blockIdx.y * gridDim.x + blockIdx.x;
  // The hardware hands workgroups to the 8 XCDs in turn and a row of column tiles is a multiple of 8 long: the row
  // tiles of an expert that share a weight panel meet in one XCD's L2.  Narrow groups start at different XCDs.
  // (512 tokens of the layer above 136 us; four neighbouring row tiles of one column to an XCD 144, and 114 instead of 77
  // at 70 tokens of 25 experts; all column tiles of a row tile to one XCD 149.)
  const int m = (int)(wg / a.ntn), c = (int)(wg % a.ntn);
  int e, row, rows;
  if (m >= a.ntm || !f32_row_tile(a, m, lane, e, row, rows)) return;
  const int n0 = (c + 3 * e) % a.ntn * (UP ? kFN / 2 : kFN);
  if (n0 >= (UP ? a.F[e / a.N] : a.d)) return;
  f32_tile<UP>(a, lds, e, row, rows, n0, w, lane);
}

// Workgroups in rows of at most kFGridX: a launch has fewer than 2^32 threads per grid dimension, which a call with
// 64 GiB of hidden activations exceeds in one.
constexpr long long kFGridX = 1ll << 20;

template <bool UP>
static hipError_t launch_f32(const F32Args& a, hipStream_t s) {
  const long long wgs = (long long)a.ntm * a.ntn;
  const long long gx = wgs < kFGridX ? wgs : kFGridX, gy = (wgs + gx - 1) / gx;
  if (gx * gy >= 1ll << 31) return hipErrorInvalidConfiguration;   // (terabytes of activations)
  constexpr int smem = kFStages * kFStage;
  static_assert(smem >= kFW * 16 * 64 * (int)sizeof(double), "the exchanged sums");
  auto kern = ffn_f32_kernel<UP>;
  static std::atomic<unsigned long long> allowed{0};
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), smem, allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)gx, (unsigned)gy), dim3(64 * kFW), smem, s, a);
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
  // (rows of column tiles of a multiple of 8, see the kernel; fewer than 8 would mostly start workgroups for nothing)
  auto row8 = [](int n) { return n < 8 ? n : (n + 7) / 8 * 8; };
  up.ntn = row8(L.Fmax / (kFN / 2));
  F32Args dn = up;
  dn.A = static_cast<const float*>(ws);
  dn.perm = nullptr;
  dn.C = static_cast<float*>(y_perm);
  dn.lda = L.Fmax; dn.ldc = L.d;
  dn.ntn = row8((L.d + kFN - 1) / kFN);
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
