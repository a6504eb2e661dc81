// Backward pass of the two-level router (section 3.2) including the gradients of the
// Group-Wise Auxiliary Loss (3.3) and the Intra-Group Experts Auxiliary Loss (3.4.2), and the
// assembly of the layer's input gradient, for gfx950 (x in bf16, everything else fp32).
//
// The routing decisions and the routing frequencies f are constants.  Per token, with the
// forward's GS, ES' (zero outside kept groups), gates, and the incoming dgate:
//   D      = sum_kept ES'_e GS_g(e),      gd = sum_kept dgate_e gate_e
//   dES''_e = (dgate_e - gd) / D                     (kept experts, else 0)
//   dES'_e  = dES''_e GS_g + v_e/(sigma_g+eps) - (sum_i v_i ES'_i)/(sigma_g+eps)^2   (kept groups)
//   dGS_g   = sum_i dES''_i ES'_i + (u_g - sum_j u_j GS_j/S)/S,   S = sum_j GS_j     (all groups)
//   dzE_e   = ES'_e (dES'_e - sum_i dES'_i ES'_i),   dzG_g = dGS_g GS_g (1 - GS_g)
// with u_g = alpha_G (F_g/F_max) f^G_g / T and v_e = alpha_E f^E_e / T.  Then
//   dW_G = dzG^T x,  dW_E = dzE^T x,  dx_t = sum_slot dx_perm[r(t,slot)] + dzG_t W_G + dzE_t W_E.
//
// Kernels: (1) one wave per token for the scalar chain above; (2) the two weight gradients as a
// reduction over tokens, split over the grid with partial sums added in a fixed order (no
// atomics: bit-identical from run to run); (3) the input gradient, up to 8 tokens per thread so
// that every router weight is fetched once per 8 tokens, in one launch with the partial sums of (2).
#include "common.h"

namespace mohge {

struct RouteBwdArgs {
  const uint16_t* x;
  const float* w_group;
  const float* w_expert;
  const float* gs;
  const float* es1;
  const int32_t* gidx;
  const int32_t* eidx;
  const float* gates;
  const float* dgates;
  const float* stats;        // f^G[Ng], p^G[Ng], f^E[Ne], p^E[Ne] or NULL (no auxiliary terms)
  const uint16_t* dx_perm;
  const int32_t* inv_perm;
  uint16_t* dx;
  float* dw_group;
  float* dw_expert;
  float* dz;                 // [T, Z], Z = Ng + Ne: group logits first
  float* part;               // [S, Z, d]
  int T, d, Ng, N, Ne, Kg, Ke, Z, S, tok_per_split;
  float alpha_g, alpha_e, eps;
  float ratio[kMaxGroups];
};

// Value of position i of a row spread over a wave (64 per register), i the same in every lane
template <typename T>
__device__ __forceinline__ T row_value(const T (&v)[4], int i) {
  const T m = i < 64 ? v[0] : i < 128 ? v[1] : i < 192 ? v[2] : v[3];
  return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, m), i & 63));
}

// A wave's token: everything of its rows is requested at once and read from other lanes' registers (loaded where it was
// needed, every sum over kept experts was a chain of three loads per expert: 8.0 us at 777 tokens, now 7.5; 11.3 at
// 8192, now 10.5).
__global__ void __launch_bounds__(256) route_bwd_token_kernel(const RouteBwdArgs a) {
  __shared__ float sh_v[kMaxExperts], sh_u[kMaxGroups];
  __shared__ float ex[4][3][kMaxExperts];   // per wave: ES', dES'', dES'
  __shared__ float gq[4][4][kMaxGroups];    // per wave: sigma, sum v ES', sum dES'' ES', sum dES' ES'
  __shared__ float s_gs[4][kMaxGroups];     // per wave: GS
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float invT = 1.f / (float)a.T;
  const int t = blockIdx.x * 4 + w;
  const bool live = t < a.T;
  const int tt = live ? t : a.T - 1;         // idle waves redo the last token and store nothing
  float es[4] = {0.f, 0.f, 0.f, 0.f}, dg[4] = {0.f, 0.f, 0.f, 0.f}, gt[4] = {0.f, 0.f, 0.f, 0.f};
  float g0[4] = {0.f, 0.f, 0.f, 0.f};
  int ei[4] = {0, 0, 0, 0}, gi[4] = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < 4; ++j) {              // (K_e <= N_e <= 256)
    const int i = lane + 64 * j;
    if (i < a.Ne) es[j] = a.es1[(size_t)tt * a.Ne + i];
    if (i < a.Ke) {
      const size_t at = (size_t)tt * a.Ke + i;
      ei[j] = a.eidx[at]; dg[j] = a.dgates[at]; gt[j] = a.gates[at];
    }
  }
  if (lane < a.Ng) g0[0] = a.gs[(size_t)tt * a.Ng + lane];
  if (lane < a.Kg) gi[0] = a.gidx[(size_t)tt * a.Kg + lane];
  for (int e = threadIdx.x; e < a.Ne; e += 256)
    sh_v[e] = a.stats ? a.alpha_e * a.stats[2 * a.Ng + e] * invT : 0.f;
  if (threadIdx.x < a.Ng)
    sh_u[threadIdx.x] = a.stats ? a.alpha_g * a.ratio[threadIdx.x] * a.stats[threadIdx.x] * invT : 0.f;
  if (lane < a.Ng) s_gs[w][lane] = g0[0];
  const float* const gs = s_gs[w];

  // gates -> ES''
  float D = 0.f, gd = 0.f, d2[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < a.Ke; ++s) {
    const int e = row_value(ei, s);
    D += row_value(es, e) * row_value(g0, e / a.N);
    gd = fmaf(row_value(dg, s), row_value(gt, s), gd);
  }
  const float invD = 1.f / D;
  for (int s = 0; s < a.Ke; ++s) {
    const int e = row_value(ei, s);
    const float v = (row_value(dg, s) - gd) * invD;
#pragma unroll
    for (int j = 0; j < 4; ++j) d2[j] = e == lane + 64 * j ? v : d2[j];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = lane + 64 * j;
    if (e < a.Ne) {
      ex[w][0][e] = es[j];
      ex[w][1][e] = d2[j];
    }
  }
  __syncthreads();
  if (lane < a.Ng) {
    float sigma = 0.f, vs = 0.f, dg = 0.f;
    for (int i = 0; i < a.N; ++i) {
      const int e = lane * a.N + i;
      sigma += ex[w][0][e];
      vs = fmaf(sh_v[e], ex[w][0][e], vs);
      dg = fmaf(ex[w][1][e], ex[w][0][e], dg);
    }
    gq[w][0][lane] = sigma; gq[w][1][lane] = vs; gq[w][2][lane] = dg;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = lane + 64 * j;
    if (e < a.Ne) {
      const int g = e / a.N;
      bool kept = false;
      for (int s = 0; s < a.Kg; ++s) kept |= row_value(gi, s) == g;
      float d1 = 0.f;
      if (kept) {
        const float den = gq[w][0][g] + a.eps;
        d1 = ex[w][1][e] * gs[g] + sh_v[e] / den - gq[w][1][g] / (den * den);
      }
      ex[w][2][e] = d1;
    }
  }
  __syncthreads();
  if (lane < a.Ng) {
    const int g = lane;
    float wsum = 0.f;
    for (int i = 0; i < a.N; ++i) wsum = fmaf(ex[w][2][g * a.N + i], ex[w][0][g * a.N + i], wsum);
    gq[w][3][g] = wsum;
    float S = 0.f, us = 0.f;
    for (int j = 0; j < a.Ng; ++j) S += gs[j];
    for (int j = 0; j < a.Ng; ++j) us = fmaf(sh_u[j], gs[j] / S, us);
    bool kept = false;
    for (int s = 0; s < a.Kg; ++s) kept |= row_value(gi, s) == g;
    const float dGS = (kept ? gq[w][2][g] : 0.f) + (sh_u[g] - us) / S;
    if (live) a.dz[(size_t)t * a.Z + g] = dGS * gs[g] * (1.f - gs[g]);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = lane + 64 * j;
    if (e < a.Ne && live) {
      const int g = e / a.N;
      // ES' is zero outside kept groups, and so is dES'
      a.dz[(size_t)t * a.Z + a.Ng + e] = ex[w][0][e] * (ex[w][2][e] - gq[w][3][g]);
    }
  }
}

// partial sums of dW[z, c] = sum_t dz[t, z] x[t, c] on the fp32 matrix cores
// (v_mfma_f32_32x32x2_f32: C[32x32] += A[32x2] B[2x32]): grid (ceil(d/128), ceil(Z/32), S).  A
// workgroup owns 128 columns and 32 rows z for the tokens of one split; its four waves take four
// neighbouring stretches of them and their sums meet in LDS, added in wave order.  Lane
// (j = lane%32, k = lane/32) loads dz[t+k, z0+j] (the A operand as it is) and the 4 columns
// c0 + 4j .. +3 of x[t+k] (one 8-byte load); MFMA m takes element m of every lane's four, so
// its 32 B-columns are the tile columns {4j + m}.  A lane ends up with 4 consecutive columns of
// 16 rows.  Loads run one group of 8 steps ahead of the arithmetic.
// What bounds it is the chain of 64-clock MFMAs of a wave (4 per two tokens) and, over short stretches,
// memory latency: the work has to be spread, with several waves per SIMD.  With a wave per 256 columns
// that walked all row passes and all tokens of a split alone, 777 tokens of a d = 1024 layer made 13
// workgroups and took 43 us; 256 columns per wave also need 280 registers, one wave per SIMD (8192
// tokens at d = 2048: 36 to 40 us with either split of the tokens).  With 128 columns, 120
// registers: 9 us and 28 us.
typedef float f32x16_t __attribute__((ext_vector_type(16)));
constexpr int kZC = 32, kTU = 8, kWGradWaves = 4;

constexpr int kWGradLds = (kWGradWaves - 1) * 16 * 64 * 16;   // 48 KB: three workgroups per compute unit

// block (bx, by, bz) of the reduction's grid; red: LDS, kWGradLds
__device__ __forceinline__ void wgrad_block(const RouteBwdArgs& a, int bx, int by, int bz, float4* red) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int j = lane & 31, k = lane >> 5;
  const int c = bx * 128 + 4 * j;
  const bool col_ok = c < a.d;
  const int cc = col_ok ? c : 0;
  const int s0 = bz * a.tok_per_split;
  const int s1 = min(a.T, s0 + a.tok_per_split);
  // (an even number of tokens per wave; a wave past the end adds zeros)
  const int per_wave = ((s1 - s0 + 2 * kWGradWaves - 1) / (2 * kWGradWaves)) * 2;
  const int t0 = min(s1, s0 + w * per_wave), t1 = min(s1, t0 + per_wave);
  const int z0 = by * kZC, zl = z0 + j;
  // step at token t: this lane's token is t + k (dz = 0 past the stretch or past Z)
  auto load = [&](int t, uint2& xv, float& dzv) {
    const int tok = t + k, tt = min(tok, a.T - 1);
    xv = *reinterpret_cast<const uint2*>(a.x + (size_t)tt * a.d + cc);
    const float v = a.dz[(size_t)tt * a.Z + min(zl, a.Z - 1)];
    dzv = (tok < t1 && zl < a.Z) ? v : 0.f;
  };
  f32x16_t acc[4];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
  uint2 xc[kTU];
  float dc[kTU];
#pragma unroll
  for (int i = 0; i < kTU; ++i) load(t0 + 2 * i, xc[i], dc[i]);
  for (int t = t0; t < t1; t += 2 * kTU) {
    uint2 xn[kTU];
    float dn[kTU];
#pragma unroll
    for (int i = 0; i < kTU; ++i) load(t + 2 * kTU + 2 * i, xn[i], dn[i]);
#pragma unroll
    for (int i = 0; i < kTU; ++i) {
      const uint32_t u[2] = {xc[i].x, xc[i].y};
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const float xf = __uint_as_float((m & 1) ? (u[m >> 1] & 0xffff0000u) : (u[m >> 1] << 16));
        acc[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(dc[i], xf, acc[m], 0, 0, 0);
      }
    }
#pragma unroll
    for (int i = 0; i < kTU; ++i) { xc[i] = xn[i]; dc[i] = dn[i]; }
  }
  // accumulator r of a lane: row 8*(r/4) + 4*k + r%4 of the 32, B-column j
  if (w > 0)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      red[((w - 1) * 16 + r) * 64 + lane] = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
  __syncthreads();
  if (w == 0 && col_ok) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int z = z0 + 8 * (r / 4) + 4 * k + (r % 4);
      if (z < a.Z) {
        float4 s = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
#pragma unroll
        for (int ww = 0; ww < kWGradWaves - 1; ++ww) {
          const float4 v = red[(ww * 16 + r) * 64 + lane];
          s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        *reinterpret_cast<float4*>(a.part + ((size_t)bz * a.Z + z) * a.d + c) = s;
      }
    }
  }
}

// dW = sum of the S partial slices, in a fixed order: thread (q, j) of a workgroup adds slices
// j, j + 8, ... of four neighbouring elements, then the 8 sums are added in index order.
__global__ void __launch_bounds__(256) route_bwd_wsum_kernel(const RouteBwdArgs a) {
  __shared__ float4 red[8][32];
  const size_t n4 = (size_t)a.Z * a.d / 4;                 // d is a multiple of 4
  const int q = threadIdx.x & 31, j = threadIdx.x >> 5;
  const size_t i4 = (size_t)blockIdx.x * 32 + q;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i4 < n4) {
    const float4* p = reinterpret_cast<const float4*>(a.part) + i4;
    for (int k = j; k < a.S; k += 8) {
      const float4 v = p[(size_t)k * n4];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
  }
  red[j][q] = s;
  __syncthreads();
  if (j == 0 && i4 < n4) {
    float4 t = red[0][q];
#pragma unroll
    for (int k = 1; k < 8; ++k) { t.x += red[k][q].x; t.y += red[k][q].y; t.z += red[k][q].z; t.w += red[k][q].w; }
    const size_t i = i4 * 4, z = i / a.d, c = i % a.d;
    float* dst = z < (size_t)a.Ng ? a.dw_group + z * a.d + c : a.dw_expert + (z - a.Ng) * a.d + c;
    *reinterpret_cast<float4*>(dst) = t;
  }
}

// dx: a thread owns 8 columns of TB tokens, a workgroup as many such token blocks as its 256 threads
// cover (rows of d <= 1024 leave room for two or more); grid (token blocks, ceil(d/2048)).
// Bound by the gathered rows of dx_perm, K_e of them per token: the rows of a token block are named
// in LDS before the first one is requested, and the rows of two tokens are in flight together.  The
// router weights come from L2 once per TB tokens, two rows ahead of their use; TB = 8 where that still
// gives every compute unit two workgroups, fewer tokens otherwise.
template <int TB>
__device__ __forceinline__ void dx_block(const RouteBwdArgs& a, int tpr, int bx, int by, unsigned char* dx_smem) {
  // tpr threads per row of this column block (a power of two up to 256), 256 / tpr token blocks
  const int sub = threadIdx.x / tpr, nsub = 256 / tpr;
  const int c = (by * 256 + (int)(threadIdx.x % tpr)) * 8;     // c >= d: helps staging only
  const int b0 = bx * nsub * TB;                               // first token of the workgroup
  const int t0 = b0 + sub * TB;
  float* dzs = reinterpret_cast<float*>(dx_smem);                      // [nsub * TB][Z]
  int* rows = reinterpret_cast<int*>(dzs + nsub * TB * a.Z);           // [nsub * TB][Ke]
  {
    const int n = nsub * TB * a.Z;
    const size_t base = (size_t)b0 * a.Z, lim = (size_t)a.T * a.Z;
    for (int i = threadIdx.x; i < n; i += 256) dzs[i] = base + i < lim ? a.dz[base + i] : 0.f;
    if (a.dx_perm) {
      const int m = nsub * TB * a.Ke;
      const size_t rb = (size_t)b0 * a.Ke, rl = (size_t)a.T * a.Ke;
      for (int i = threadIdx.x; i < m; i += 256) rows[i] = rb + i < rl ? a.inv_perm[rb + i] : 0;
    }
  }
  __syncthreads();
  if (c >= a.d) return;
  const float* dzr = dzs + sub * TB * a.Z;
  const int* rw = rows + sub * TB * a.Ke;
  float acc[TB][8];
#pragma unroll
  for (int k = 0; k < TB; ++k)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[k][i] = 0.f;
  if (a.dx_perm) {
    constexpr int TP = TB >= 2 ? 2 : 1;
#pragma unroll
    for (int k0 = 0; k0 < TB; k0 += TP) {
      // four slots of TP tokens at a time: the row loads are issued together, then added in slot order
      // (tokens past the end name row 0 and are not stored)
      for (int s0 = 0; s0 < a.Ke; s0 += 4) {
        uint4 u[TP][4];
#pragma unroll
        for (int p = 0; p < TP; ++p)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (s0 + i < a.Ke)
              u[p][i] = *reinterpret_cast<const uint4*>(a.dx_perm + (size_t)rw[(k0 + p) * a.Ke + s0 + i] * a.d + c);
#pragma unroll
        for (int p = 0; p < TP; ++p)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (s0 + i < a.Ke) {
              float (&ac)[8] = acc[k0 + p];
              const uint4 v = u[p][i];
              ac[0] += __uint_as_float(v.x << 16); ac[1] += __uint_as_float(v.x & 0xffff0000u);
              ac[2] += __uint_as_float(v.y << 16); ac[3] += __uint_as_float(v.y & 0xffff0000u);
              ac[4] += __uint_as_float(v.z << 16); ac[5] += __uint_as_float(v.z & 0xffff0000u);
              ac[6] += __uint_as_float(v.w << 16); ac[7] += __uint_as_float(v.w & 0xffff0000u);
            }
      }
    }
  }
  // router rows: four at a time, the next four requested before the present ones are used
  auto wrow = [&](int z) {
    return z < a.Ng ? a.w_group + (size_t)z * a.d + c : a.w_expert + (size_t)(z - a.Ng) * a.d + c;
  };
  constexpr int ZU = 4;
  float4 wc[ZU][2];
#pragma unroll
  for (int i = 0; i < ZU; ++i) {
    const float* p = wrow(min(i, a.Z - 1));
    wc[i][0] = *reinterpret_cast<const float4*>(p);
    wc[i][1] = *reinterpret_cast<const float4*>(p + 4);
  }
  for (int z0 = 0; z0 < a.Z; z0 += ZU) {
    float4 wn[ZU][2];
#pragma unroll
    for (int i = 0; i < ZU; ++i) {
      const float* p = wrow(min(z0 + ZU + i, a.Z - 1));
      wn[i][0] = *reinterpret_cast<const float4*>(p);
      wn[i][1] = *reinterpret_cast<const float4*>(p + 4);
    }
#pragma unroll
    for (int i = 0; i < ZU; ++i) {
      if (z0 + i < a.Z) {
        const float4 w0 = wc[i][0], w1 = wc[i][1];
#pragma unroll
        for (int k = 0; k < TB; ++k) {
          const float dzv = dzr[k * a.Z + z0 + i];
          acc[k][0] = fmaf(dzv, w0.x, acc[k][0]); acc[k][1] = fmaf(dzv, w0.y, acc[k][1]);
          acc[k][2] = fmaf(dzv, w0.z, acc[k][2]); acc[k][3] = fmaf(dzv, w0.w, acc[k][3]);
          acc[k][4] = fmaf(dzv, w1.x, acc[k][4]); acc[k][5] = fmaf(dzv, w1.y, acc[k][5]);
          acc[k][6] = fmaf(dzv, w1.z, acc[k][6]); acc[k][7] = fmaf(dzv, w1.w, acc[k][7]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < ZU; ++i) { wc[i][0] = wn[i][0]; wc[i][1] = wn[i][1]; }
  }
#pragma unroll
  for (int k = 0; k < TB; ++k) {
    const int t = t0 + k;
    if (t < a.T) {
      uint4 o;
      o.x = pack_bf16x2(acc[k][0], acc[k][1]); o.y = pack_bf16x2(acc[k][2], acc[k][3]);
      o.z = pack_bf16x2(acc[k][4], acc[k][5]); o.w = pack_bf16x2(acc[k][6], acc[k][7]);
      *reinterpret_cast<uint4*>(a.dx + (size_t)t * a.d + c) = o;
    }
  }
}

// The partial sums of dW and dx in one launch: both need dz only, the first is bound by its matrix instructions, the
// second by memory.  The n_w workgroups of the first come first: 777 tokens, d = 1024, 8.5 + 11.5 us one after the other, 14
// together; 8192 tokens, d = 2048: 28 + 54, 79 together (in turn, eight and eight, 83).
template <int TB>
__global__ void __launch_bounds__(256, 3) route_bwd_main_kernel(const RouteBwdArgs a, int tpr, int n_w, int dx_cb) {
  extern __shared__ __align__(16) unsigned char smem[];
  static_assert(64 * kWGradWaves == 256, "one workgroup shape");
  const int b = blockIdx.x;
  if (b < n_w) {
    const int cols = (a.d + 127) / 128, rows = (a.Z + kZC - 1) / kZC;
    wgrad_block(a, b % cols, b / cols % rows, b / (cols * rows), reinterpret_cast<float4*>(smem));
  } else {
    dx_block<TB>(a, tpr, (b - n_w) / dx_cb, (b - n_w) % dx_cb, smem);
  }
}

// token splits of the weight-gradient reduction: enough for three workgroups per compute unit, at least
// 32 tokens each (8 per wave: shorter stretches cost more in partial sums than they save in MFMAs), at
// most 256 splits and at most 64 MB of partial sums.  A wide layer has its workgroups without many splits, but the
// fp32 chain of a wave's tokens is what the rounding error grows with (half its length, and a sixteenth of the splits in
// the final sum): no worse than chains of 64 tokens, at most 256 of them or 64 MB, added by eight threads each, which
// takes a little over a quarter of their number, four waves to a split.  (d = 4096, 68 router rows, 8192 tokens: 16
// splits, error against float64 1.64e-7 and 253 us for the call; with the 8 that fill the compute units 2.16e-7, 243 us.)
static int wgrad_splits(const LayerDesc& L) {
  const long long per_split = (long long)((L.d + 127) / 128) * ((L.Ng + L.Ne + kZC - 1) / kZC);
  const long long cap = (64ll << 20) / ((long long)(L.Ng + L.Ne) * L.d * 4);
  long long s = (768 + per_split - 1) / per_split;
  long long chains = (L.T + 63) / 64;
  if (chains > cap) chains = cap;
  if (chains > 256) chains = 256;
  const long long least = (chains + 3) / 4 + 1;
  if (s < least) s = (least + s - 1) / s * s;             // (whole rounds of workgroups)
  if (s > (L.T + 31) / 32) s = (L.T + 31) / 32;
  if (s > cap) s = cap;
  if (s > 256) s = 256;
  return s < 1 ? 1 : (int)s;
}

static size_t up256(size_t b) { return (b + 255) / 256 * 256; }

// workspace: dz [T, Z] fp32, then the partial sums [S, Z, d] fp32
size_t route_bwd_workspace_bytes(const LayerDesc& L) {
  const size_t Z = L.Ng + L.Ne, T = L.T > 0 ? L.T : 1;
  return up256(T * Z * 4) + up256((size_t)wgrad_splits(L) * Z * L.d * 4);
}

static void launch_main(const RouteBwdArgs& a, hipStream_t s) {
  // threads per row: a power of two that covers a row of up to 2048 columns; the staged dz and row
  // numbers of the workgroup's tokens stay below 32 KB
  int tpr = 8;
  while (tpr < 256 && tpr * 8 < a.d) tpr *= 2;
  const unsigned cb = (unsigned)((a.d + 2047) / 2048);
  const unsigned n_w = (unsigned)((a.d + 127) / 128) * ((a.Z + kZC - 1) / kZC) * a.S;
  for (int TB = 8; TB >= 2; TB /= 2) {
    auto lds = [&](int t) { return (size_t)(256 / t) * TB * (a.Z + a.Ke) * 4; };
    int t = tpr;
    while (t < 256 && lds(t) > 32 * 1024) t *= 2;
    const int per_wg = 256 / t * TB;
    const unsigned tb = (unsigned)((a.T + per_wg - 1) / per_wg);
    if (TB > 2 && (long long)tb * cb < 512) continue;
    auto kern = TB == 8 ? route_bwd_main_kernel<8> : TB == 4 ? route_bwd_main_kernel<4> : route_bwd_main_kernel<2>;
    const size_t smem = lds(t) > (size_t)kWGradLds ? lds(t) : (size_t)kWGradLds;
    hipLaunchKernelGGL(kern, dim3(n_w + tb * cb), dim3(256), smem, s, a, t, (int)n_w, (int)cb);
    return;
  }
}

hipError_t launch_route_bwd(const LayerDesc& L, const mohge_config& cfg, const void* x,
                            const float* w_group, const float* w_expert, const float* gs,
                            const float* es1, const int32_t* group_idx, const int32_t* expert_idx,
                            const float* gates, const float* dgates, const float* stats,
                            const void* dx_perm, const int32_t* inv_perm, void* dx, float* dw_group,
                            float* dw_expert, float* dz_out, void* ws, hipStream_t s) {
  RouteBwdArgs a{};
  a.x = static_cast<const uint16_t*>(x);
  a.w_group = w_group; a.w_expert = w_expert; a.gs = gs; a.es1 = es1;
  a.gidx = group_idx; a.eidx = expert_idx; a.gates = gates; a.dgates = dgates; a.stats = stats;
  a.dx_perm = static_cast<const uint16_t*>(dx_perm); a.inv_perm = inv_perm;
  a.dx = static_cast<uint16_t*>(dx); a.dw_group = dw_group; a.dw_expert = dw_expert;
  a.T = L.T; a.d = L.d; a.Ng = L.Ng; a.N = L.N; a.Ne = L.Ne; a.Kg = L.Kg; a.Ke = L.Ke;
  a.Z = L.Ng + L.Ne;
  a.S = wgrad_splits(L);
  a.tok_per_split = (L.T + a.S - 1) / a.S;
  a.alpha_g = cfg.alpha_g; a.alpha_e = cfg.alpha_e; a.eps = cfg.eps;
  for (int g = 0; g < kMaxGroups; ++g) a.ratio[g] = g < L.Ng ? (float)L.F[g] / (float)L.Fmax : 0.f;
  unsigned char* base = static_cast<unsigned char*>(ws);
  const size_t dz_bytes = up256((size_t)L.T * a.Z * 4);
  a.dz = dz_out ? dz_out : reinterpret_cast<float*>(base);
  a.part = reinterpret_cast<float*>(base + dz_bytes);
  hipLaunchKernelGGL(route_bwd_token_kernel, dim3((unsigned)((L.T + 3) / 4)), dim3(256), 0, s, a);
  launch_main(a, s);
  hipLaunchKernelGGL(route_bwd_wsum_kernel, dim3((unsigned)(((size_t)a.Z * L.d / 4 + 31) / 32)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace mohge
