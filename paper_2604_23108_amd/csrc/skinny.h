// Arguments and the per-workgroup unit of the bf16 decode kernels of the expert networks (a
// handful of tokens per expert: every touched expert's weights are streamed once), shared by the
// two-launch form and the single-launch decode layer.
#pragma once
#include <type_traits>

#include "common.h"

namespace mohge {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct SkinnyArgs {
  const uint16_t* A;              // up: x; down: H
  const int32_t* perm;            // up only, may be NULL
  const int32_t* offsets;
  const uint16_t* W[kMaxGroups];  // bf16 weights, or E4M3 codes (W8)
  const float* S[kMaxGroups];     // W8: scale per weight row, same row order as W
  const uint8_t* S4[kMaxGroups];  // W4: E8M0 scale per 32 elements of a weight row, [rows][K/32]
  uint16_t* C;
  int lda, ldc, Ke, Ng, N, d;
  int F[kMaxGroups];
  int blk_prefix[kMaxGroups + 1]; // first workgroup of each group
};

// host: argument blocks of the up and the down launch, nu / nd workgroups (one per unit); s13/s2:
// FP8 row scales or NULL, b13/b2: MXFP4 block scales or NULL
void skinny_args(const LayerDesc& L, const void* x, const int32_t* perm, const int32_t* offsets,
                 const GroupPtrs& W, void* y_perm, void* h, const float* const* s13, const float* const* s2,
                 const void* const* b13, const void* const* b2, SkinnyArgs& up, SkinnyArgs& dn, int& nu, int& nd);

union Frag {
  uint4 u;
  bf16x8 v;
};

// 8-byte store performed at device scope (written through the XCD's L2): once the store has
// completed (vmcnt), a workgroup on any XCD that has not cached the line before reads the new data.
__device__ __forceinline__ void store8_device_scope(void* p, const uint2 v) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 q = {v.x, v.y};
  asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(p), "v"(q) : "memory");
}

// Weight rows 4q..4q+3 of each row set for one sorted row: the SwiGLU product [UP] or both sets as they are
template <bool UP, bool COHERENT>
__device__ __forceinline__ void skinny_store(const SkinnyArgs& a, const int c0, const int q, const int ncols, const int row,
                                             const f32x4 s0, const f32x4 s1) {
  uint16_t* crow = a.C + (long long)row * a.ldc;
  if constexpr (UP) {
    float v[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) v[b] = s0[b] / (1.f + __expf(-s0[b])) * s1[b];
    uint2 o;
    o.x = pack_bf16x2(v[0], v[1]);
    o.y = pack_bf16x2(v[2], v[3]);
    if constexpr (COHERENT) store8_device_scope(crow + c0 + 4 * q, o);
    else *reinterpret_cast<uint2*>(crow + c0 + 4 * q) = o;
  } else {
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const f32x4 s = f ? s1 : s0;
      const int col = c0 + 16 * f + 4 * q;
      if (col < ncols) {
        uint2 o;
        o.x = pack_bf16x2(s[0], s[1]);
        o.y = pack_bf16x2(s[2], s[3]);
        if constexpr (COHERENT) store8_device_scope(crow + col, o);
        else *reinterpret_cast<uint2*>(crow + col) = o;
      }
    }
  }
}

// One unit of the bf16 decode kernels: 16 hidden units [UP: 16 W_gate rows and the matching 16 W_up rows] or
// 32 output features [down] of one expert, all its rows, 32 at a time.  The four waves of the workgroup take
// the same weight rows and a quarter of the reduction indices each; their partial sums meet in LDS and are
// added in wave order.  Bound by the weight stream, i.e. by the loads in flight: a wave has the weights
// and token rows of 128 (64 with more than 16 rows) reduction indices on the way while it multiplies the
// previous ones, and requests its first weights before it looks up the expert's tokens.  The quarters
// also start a quarter of a row apart, which spreads the waves over the memory channels (rows begin at
// multiples of the row size, a power of two at the usual hidden sizes).
// Measured against a wave per 32 weight rows that walked the whole reduction, up + down of d = 4096, 64
// experts (widths 768..2048): 88 -> 33 us with one token (352 waves, not two per compute unit, each with 16
// steps of memory latency), 194 -> 170 at 8 tokens, 357 -> 328 (5.9 TB/s) at 32; d = 1024, 32 experts:
// 36 -> 29 at 32 tokens.
constexpr int kSplitWaves = 4;
constexpr int kSplitLdsBytes = (kSplitWaves - 1) * 4 * 64 * 16;

// expert e = group g, index i inside it; c0: first of 16 hidden units [UP] or 32 output features [down].
// red: LDS, kSplitLdsBytes.  Called by the whole workgroup of 4 waves, the same arguments in all of them.
template <bool UP>
__device__ __forceinline__ void skinny_unit(const SkinnyArgs& a, const int g, const int i, const int c0,
                                                  const int row0, const int cnt, f32x4* const red) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  const int F = a.F[g];
  const int K = UP ? a.d : F;
  const int ncols = UP ? F : a.d;
  const uint16_t* wp[2];
  if constexpr (UP) {
    const uint16_t* base = a.W[g] + (long long)i * 2 * F * K;
    wp[0] = base + (long long)(c0 + r) * K + 8 * q;
    wp[1] = base + (long long)(F + c0 + r) * K + 8 * q;
  } else {
    const uint16_t* base = a.W[g] + (long long)i * a.d * K;
    int n1 = c0 + 16 + r;
    if (n1 > a.d - 1) n1 = a.d - 1;
    wp[0] = base + (long long)(c0 + r) * K + 8 * q;
    wp[1] = base + (long long)n1 * K + 8 * q;
  }
  // this wave's indices: whole blocks of 64 (none where the reduction is shorter than 256)
  const int nb = K / 64;
  const int kb = nb * w / kSplitWaves * 64, ke = nb * (w + 1) / kSplitWaves * 64;
  for (int tb0 = 0; tb0 < cnt; tb0 += 32) {
    auto pass = [&](auto NTBC) {
      constexpr int NTB = decltype(NTBC)::value;             // token blocks of 16
      constexpr int U = NTB == 1 ? 4 : 2;                    // 32-deep matrix-core steps per request
      constexpr int S = 32 * U;
      // The token numbers are requested before the first weights (loads return in order) and waited for behind them.  (Waited for
      // in front: d = 1024, 128 experts 158.9 us at 32 tokens, 64 experts 54.9 instead of 53.5 at 8, longer than with the checks.)
      int row[NTB];
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) {
        const int tt = tb0 + 16 * tb + r;
        row[tb] = row0 + (tt < cnt ? tt : 0);                // columns past the count: any of its rows, never stored
        if (UP && a.perm) row[tb] = a.perm[row[tb]];
      }
      struct Step { Frag w[2][U], x[NTB][U]; };
      // The first pieces of 32 indices from k on.  No branch between requests, so that the compiler's waits count: behind one
      // it waits for everything on its way, the step just requested included.  (It did, and no step was multiplied before the
      // next had landed.  Layer calls, that -> this: d = 4096, 64 experts, one token 52.7 -> 47.3 us, 4 123.6 -> 112.9, 32 356 -> 341;
      // d = 2560 32 tokens 273 -> 243; d = 2048 one token 35 -> 33; d = 1024, 128 experts, 32 tokens 157.6 -> 148.5.)
      const uint16_t* pw[2] = {wp[0] + kb, wp[1] + kb};
      const uint16_t* xp[NTB];
      auto find_rows = [&]() {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) xp[tb] = a.A + 8 * q + kb + (long long)(UP && a.perm ? row[tb] / a.Ke : row[tb]) * a.lda;
      };
      auto load_w = [&](Step& st, int k, auto NC) {
#pragma unroll
        for (int u = 0; u < decltype(NC)::value; ++u)
#pragma unroll
          for (int f = 0; f < 2; ++f) st.w[f][u].u = *reinterpret_cast<const uint4*>(pw[f] + k + 32 * u);
      };
      auto load_x = [&](Step& st, int k, auto NC) {
#pragma unroll
        for (int u = 0; u < decltype(NC)::value; ++u)
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) st.x[tb][u].u = *reinterpret_cast<const uint4*>(xp[tb] + k + 32 * u);
      };
      f32x4 acc[2][NTB];
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) acc[f][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
      auto multiply = [&](const Step& st, auto NC) {
        __builtin_amdgcn_sched_barrier(0);                   // (the requests in front stay there)
#pragma unroll
        for (int u = 0; u < decltype(NC)::value; ++u)
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
              acc[f][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.w[f][u].v, st.x[tb][u].v, acc[f][tb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      };
      using All = std::integral_constant<int, U>;
      using Half = std::integral_constant<int, 2>;           // (the indices come in blocks of 64)
      auto advance = [&](int n) {
#pragma unroll
        for (int f = 0; f < 2; ++f) pw[f] += n;
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) xp[tb] += n;
      };
      int rem = ke - kb;
      if (rem >= S) {
        // two sets of registers in turn: copied from one to the other, they would have to have landed
        Step s0, s1;
        load_w(s0, 0, All{});
        find_rows();
        load_x(s0, 0, All{});
        for (; rem >= 3 * S; rem -= 2 * S) {
          load_w(s1, S, All{});
          load_x(s1, S, All{});
          multiply(s0, All{});
          load_w(s0, 2 * S, All{});
          load_x(s0, 2 * S, All{});
          multiply(s1, All{});
          advance(2 * S);
        }
        if (rem >= 2 * S) {
          load_w(s1, S, All{});
          load_x(s1, S, All{});
          multiply(s0, All{});
          multiply(s1, All{});
          advance(2 * S);
          rem -= 2 * S;
        } else {
          multiply(s0, All{});
          advance(S);
          rem -= S;
        }
      } else {
        find_rows();
      }
      if (U > 2 && rem > 0) {
        Step st;
        load_w(st, 0, Half{});
        load_x(st, 0, Half{});
        multiply(st, Half{});
      }
      if (w > 0)
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) red[((w - 1) * 4 + 2 * f + tb) * 64 + lane] = acc[f][tb];
      __syncthreads();
      if (w == 0) {
        // lane holds token r of each token block, weight rows 4q..4q+3 of each row set
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int ww = 0; ww < kSplitWaves - 1; ++ww) acc[f][tb] += red[(ww * 4 + 2 * f + tb) * 64 + lane];
          const int tt = tb0 + 16 * tb + r;
          if (tt >= cnt) continue;
          skinny_store<UP, false>(a, c0, q, ncols, row0 + tt, acc[0][tb], acc[1][tb]);
        }
      }
      __syncthreads();                                       // the sums have been read
    };
    if (cnt - tb0 > 16) pass(std::integral_constant<int, 2>{});
    else pass(std::integral_constant<int, 1>{});
  }
}

// The same rows of C for a wave by itself: 16 hidden units or 32 output features from c0, the four quarters of the
// reduction one after the other, each summed by itself and the sums added in order, so that the bits are those of
// skinny_unit.  For the single-launch decode layer, whose workgroups take 64 hidden units or 128 output features at a
// time: four waves side by side need no barrier and no LDS, and the workgroup one pass.  (Four of the units above
// after one another took the whole layer 2 to 17 % longer than a wave per 32 rows had, at most sizes: 205 -> 214 us at
// one token of d = 4096, 64 experts, 32 -> 37 at d = 128; this form takes 197 and 30.)  128 indices at a time: with
// 256 the layer's registers spill.  All waves starting at the same quarter cost up to 7 % at 4 to 16 tokens.  The
// rows are stored at device scope, for a consumer in the same launch.
template <bool UP>
__device__ __forceinline__ void skinny_wave_unit(const SkinnyArgs& a, const int g, const int i, const int c0,
                                                 const int row0, const int cnt) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  const int F = a.F[g];
  const int K = UP ? a.d : F;
  const int ncols = UP ? F : a.d;
  if (c0 >= ncols) return;
  const uint16_t* wp[2];
  if constexpr (UP) {
    const uint16_t* base = a.W[g] + (long long)i * 2 * F * K;
    wp[0] = base + (long long)(c0 + r) * K + 8 * q;
    wp[1] = base + (long long)(F + c0 + r) * K + 8 * q;
  } else {
    const uint16_t* base = a.W[g] + (long long)i * a.d * K;
    int n1 = c0 + 16 + r;
    if (n1 > a.d - 1) n1 = a.d - 1;
    wp[0] = base + (long long)(c0 + r) * K + 8 * q;
    wp[1] = base + (long long)n1 * K + 8 * q;
  }
  const int nb = K / 64;
  for (int tb0 = 0; tb0 < cnt; tb0 += 32) {
    auto pass = [&](auto NTBC) {
      constexpr int NTB = decltype(NTBC)::value;             // token blocks of 16
      const uint16_t* xp[NTB];
      bool xv[NTB];
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) {
        const int tt = tb0 + 16 * tb + r;
        xv[tb] = tt < cnt;
        const int pos = row0 + (xv[tb] ? tt : 0);
        long long src;
        if constexpr (UP) src = a.perm ? (long long)(a.perm[pos] / a.Ke) : (long long)pos;
        else src = pos;
        xp[tb] = a.A + src * a.lda + 8 * q;
      }
      auto step = [&](f32x4 (&acc)[2][NTB], int k0, auto UC) {
        constexpr int U = decltype(UC)::value;
        Frag wf[2][U], xf[NTB][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
          for (int f = 0; f < 2; ++f) wf[f][u].u = *reinterpret_cast<const uint4*>(wp[f] + k0 + 32 * u);
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) {
            xf[tb][u].u = make_uint4(0u, 0u, 0u, 0u);
            if (xv[tb]) xf[tb][u].u = *reinterpret_cast<const uint4*>(xp[tb] + k0 + 32 * u);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
              acc[f][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[f][u].v, xf[tb][u].v, acc[f][tb], 0, 0, 0);
      };
      auto quarter = [&](f32x4 (&sum)[2][NTB], int qt) {
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) sum[f][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
        int k0 = nb * qt / kSplitWaves * 64;
        const int ke = nb * (qt + 1) / kSplitWaves * 64;
        for (; k0 + 128 <= ke; k0 += 128) step(sum, k0, std::integral_constant<int, 4>{});
        for (; k0 < ke; k0 += 64) step(sum, k0, std::integral_constant<int, 2>{});
      };
      f32x4 acc[2][NTB];
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) acc[f][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (NTB == 1) {
        // Starting at quarter w, which spreads the waves over the memory channels; added in order.
        f32x4 p0[2], p1[2], p2[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) p0[f] = p1[f] = p2[f] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int v = 0; v < kSplitWaves; ++v) {
          const int qt = (w + v) & (kSplitWaves - 1);
          f32x4 part[2][1];
          quarter(part, qt);
          if (qt == 0) { p0[0] = part[0][0]; p0[1] = part[1][0]; }
          else if (qt == 1) { p1[0] = part[0][0]; p1[1] = part[1][0]; }
          else if (qt == 2) { p2[0] = part[0][0]; p2[1] = part[1][0]; }
          else { acc[0][0] = part[0][0]; acc[1][0] = part[1][0]; }
        }
#pragma unroll
        for (int f = 0; f < 2; ++f) { p0[f] += p1[f]; p0[f] += p2[f]; acc[f][0] = p0[f] + acc[f][0]; }
      } else {
#pragma unroll 1
        for (int qt = 0; qt < kSplitWaves; ++qt) {
          f32x4 part[2][NTB];
          quarter(part, qt);
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) acc[f][tb] += part[f][tb];
        }
      }
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) {
        const int tt = tb0 + 16 * tb + r;
        if (tt < cnt) skinny_store<UP, true>(a, c0, q, ncols, row0 + tt, acc[0][tb], acc[1][tb]);
      }
    };
    if (cnt - tb0 > 16) pass(std::integral_constant<int, 2>{});
    else pass(std::integral_constant<int, 1>{});
  }
}

}  // namespace mohge
