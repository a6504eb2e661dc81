// Gated un-permute and combine for gfx950 (appendix, background: y = sum_i G_i(x) E_i(x)).
// Bandwidth-bound: every thread owns 16 bytes of one output row, reads the K_e expert
// rows of its token through inv_perm with 16-byte loads and accumulates in fp32 in slot
// order, so the result does not depend on scheduling.
#include "common.h"

namespace mohge {

template <bool BF16>
__global__ void __launch_bounds__(256) combine_kernel(const uint4* __restrict__ y_perm,
                                                      const int32_t* __restrict__ inv_perm,
                                                      const float* __restrict__ gates,
                                                      const uint4* y_add, uint4* y, int T, int Ke,
                                                      int vec_per_row) {
  const long long total = (long long)T * vec_per_row;
  for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long long)gridDim.x * blockDim.x) {
    const int t = (int)(idx / vec_per_row), v = (int)(idx % vec_per_row);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (y_add) {          // the term added to the gated sum (may be y itself: read before written)
      const uint4 u = y_add[idx];
      if constexpr (BF16) {
        acc[0] = __uint_as_float(u.x << 16); acc[1] = __uint_as_float(u.x & 0xffff0000u);
        acc[2] = __uint_as_float(u.y << 16); acc[3] = __uint_as_float(u.y & 0xffff0000u);
        acc[4] = __uint_as_float(u.z << 16); acc[5] = __uint_as_float(u.z & 0xffff0000u);
        acc[6] = __uint_as_float(u.w << 16); acc[7] = __uint_as_float(u.w & 0xffff0000u);
      } else {
        acc[0] = __uint_as_float(u.x); acc[1] = __uint_as_float(u.y);
        acc[2] = __uint_as_float(u.z); acc[3] = __uint_as_float(u.w);
      }
    }
    // four slots at a time: their gates and row numbers are requested together, then their rows (one slot
    // after the other cost two memory latencies per slot); added in slot order
    for (int s0 = 0; s0 < Ke; s0 += 4) {
      float g[4];
      int r[4];
      uint4 row[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const size_t at = (size_t)t * Ke + min(s0 + i, Ke - 1);
        g[i] = gates[at];
        r[i] = inv_perm[at];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (s0 + i < Ke) row[i] = y_perm[(size_t)r[i] * vec_per_row + v];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (s0 + i < Ke) {
          const uint4 u = row[i];
          if constexpr (BF16) {
            acc[0] = fmaf(g[i], __uint_as_float(u.x << 16), acc[0]);
            acc[1] = fmaf(g[i], __uint_as_float(u.x & 0xffff0000u), acc[1]);
            acc[2] = fmaf(g[i], __uint_as_float(u.y << 16), acc[2]);
            acc[3] = fmaf(g[i], __uint_as_float(u.y & 0xffff0000u), acc[3]);
            acc[4] = fmaf(g[i], __uint_as_float(u.z << 16), acc[4]);
            acc[5] = fmaf(g[i], __uint_as_float(u.z & 0xffff0000u), acc[5]);
            acc[6] = fmaf(g[i], __uint_as_float(u.w << 16), acc[6]);
            acc[7] = fmaf(g[i], __uint_as_float(u.w & 0xffff0000u), acc[7]);
          } else {
            acc[0] = fmaf(g[i], __uint_as_float(u.x), acc[0]);
            acc[1] = fmaf(g[i], __uint_as_float(u.y), acc[1]);
            acc[2] = fmaf(g[i], __uint_as_float(u.z), acc[2]);
            acc[3] = fmaf(g[i], __uint_as_float(u.w), acc[3]);
          }
        }
      }
    }
    uint4 o;
    if constexpr (BF16) {
      o.x = pack_bf16x2(acc[0], acc[1]);
      o.y = pack_bf16x2(acc[2], acc[3]);
      o.z = pack_bf16x2(acc[4], acc[5]);
      o.w = pack_bf16x2(acc[6], acc[7]);
    } else {
      o.x = __float_as_uint(acc[0]);
      o.y = __float_as_uint(acc[1]);
      o.z = __float_as_uint(acc[2]);
      o.w = __float_as_uint(acc[3]);
    }
    y[idx] = o;
  }
}

hipError_t launch_combine(const LayerDesc& L, int dtype, const void* y_perm,
                          const int32_t* inv_perm, const float* gates, const void* y_add, void* y,
                          hipStream_t s) {
  const bool bf = dtype == MOHGE_BF16;
  const int vec_per_row = L.d * (bf ? 2 : 4) / 16;
  const long long total = (long long)L.T * vec_per_row;
  long long blocks = (total + 255) / 256;
  if (blocks > 1ll << 23) blocks = 1ll << 23;      // (a cap of 64 workgroups per compute unit cost 3 to 10 % from 16384 tokens on)
  if (bf)
    hipLaunchKernelGGL((combine_kernel<true>), dim3((unsigned)blocks), dim3(256), 0, s,
                       static_cast<const uint4*>(y_perm), inv_perm, gates,
                       static_cast<const uint4*>(y_add), static_cast<uint4*>(y), L.T, L.Ke, vec_per_row);
  else
    hipLaunchKernelGGL((combine_kernel<false>), dim3((unsigned)blocks), dim3(256), 0, s,
                       static_cast<const uint4*>(y_perm), inv_perm, gates,
                       static_cast<const uint4*>(y_add), static_cast<uint4*>(y), L.T, L.Ke, vec_per_row);
  return hipGetLastError();
}

// Routing of always-on ("shared") experts: every token goes to every one of the N experts of
// the single group with gate 1.  Sorted position r = s*T + t <-> pair p = t*N + s.
__global__ void __launch_bounds__(256) shared_routing_kernel(int T, int N, int32_t* expert_idx,
                                                             float* gates, int32_t* counts,
                                                             int32_t* offsets, int32_t* perm,
                                                             int32_t* inv_perm) {
  const long long P = (long long)T * N;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < P; i += (long long)gridDim.x * 256) {
    const int t_of_p = (int)(i / N), s_of_p = (int)(i % N);     // i as pair id
    expert_idx[i] = s_of_p;
    gates[i] = 1.f;
    inv_perm[i] = s_of_p * T + t_of_p;
    const int s_of_r = (int)(i / T), t_of_r = (int)(i % T);     // i as sorted position
    perm[i] = t_of_r * N + s_of_r;
  }
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i <= N; i += 256) {      // N can equal the block size
      offsets[i] = i * T;
      if (i < N) counts[i] = T;
    }
}

hipError_t launch_shared_routing(const LayerDesc& L, int32_t* expert_idx, float* gates,
                                 int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv_perm,
                                 hipStream_t s) {
  long long blocks = ((long long)L.P + 255) / 256;
  if (blocks < 1) blocks = 1;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(shared_routing_kernel, dim3((unsigned)blocks), dim3(256), 0, s, L.T, L.N, expert_idx,
                     gates, counts, offsets, perm, inv_perm);
  return hipGetLastError();
}

}  // namespace mohge

// ---------------------------------------------------------------------------------------
// backward of the gated combine (bf16):  y_t = sum_slot gate[t,slot] * y_perm[r(t,slot)]
//   dgates[t,slot] = <dy_t, y_perm[r]>,   dy_perm[r] = gate[t,slot] * dy_t
// One wave per token; lanes stride the row in 16-byte chunks; the dot product is folded with a
// butterfly, so the result does not depend on scheduling.
// Bound by memory: dy, K_e rows of y_perm and K_e rows of dy_perm per token.  NS slots at a time: dy is read once
// for them and their rows of y_perm are in flight together (d = 4096, four slots: 24.4 -> 20.3 us at 1500 tokens,
// 12.5 -> 6.8 at 100).  Past what the last-level cache holds (256 MB) one slot at a time is the faster walk, two rows
// read and one written at a time instead of five and four: at 8192 tokens 164 us against 171 to 181 with four slots,
// 129 against 137 to 144 with three (inputs not in the cache; 131 against 154 to 165 when calls follow each
// other).  The line lies at 300 MB: at 302 million bytes four slots are still 3 to 6 % ahead, at 336 one slot 7 to 22 %.
// ---------------------------------------------------------------------------------------
namespace mohge {

template <int NS>
__global__ void __launch_bounds__(256) combine_bwd_kernel(const uint4* __restrict__ dy,
                                                          const uint4* __restrict__ y_perm,
                                                          const int32_t* __restrict__ inv_perm,
                                                          const float* __restrict__ gates,
                                                          float* __restrict__ dgates,
                                                          uint4* __restrict__ dy_perm, int T, int Ke,
                                                          int vec_per_row) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  for (int s0 = 0; s0 < Ke; s0 += NS) {
    float g[NS], dot[NS];
    int r[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const size_t at = (size_t)t * Ke + s0 + i;
      g[i] = gates[at];
      r[i] = inv_perm[at];
      dot[i] = 0.f;
    }
    for (int v = lane; v < vec_per_row; v += 64) {
      const uint4 a = dy[(size_t)t * vec_per_row + v];
      uint4 b[NS];
#pragma unroll
      for (int i = 0; i < NS; ++i) b[i] = y_perm[(size_t)r[i] * vec_per_row + v];
      const uint32_t aw[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const uint32_t bw[4] = {b[i].x, b[i].y, b[i].z, b[i].w};
        uint32_t ow[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float a0 = __uint_as_float(aw[k] << 16), a1 = __uint_as_float(aw[k] & 0xffff0000u);
          const float b0 = __uint_as_float(bw[k] << 16), b1 = __uint_as_float(bw[k] & 0xffff0000u);
          dot[i] = fmaf(a0, b0, dot[i]);
          dot[i] = fmaf(a1, b1, dot[i]);
          ow[k] = pack_bf16x2(g[i] * a0, g[i] * a1);
        }
        dy_perm[(size_t)r[i] * vec_per_row + v] = make_uint4(ow[0], ow[1], ow[2], ow[3]);
      }
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) {
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) dot[i] += __shfl_xor(dot[i], off, 64);
      if (lane == 0) dgates[(size_t)t * Ke + s0 + i] = dot[i];
    }
  }
}

hipError_t launch_combine_bwd(const LayerDesc& L, const void* dy, const void* y_perm,
                              const int32_t* inv_perm, const float* gates, float* dgates,
                              void* dy_perm, hipStream_t s) {
  const int vec_per_row = L.d * 2 / 16;
  const bool one = (long long)L.T * (2 * L.Ke + 1) * L.d * 2 > (300ll << 20);
  auto kern = one ? combine_bwd_kernel<1> : L.Ke % 4 == 0 ? combine_bwd_kernel<4> : L.Ke % 3 == 0 ? combine_bwd_kernel<3>
              : L.Ke % 2 == 0 ? combine_bwd_kernel<2> : combine_bwd_kernel<1>;
  hipLaunchKernelGGL(kern, dim3((unsigned)((L.T + 3) / 4)), dim3(256), 0, s,
                     static_cast<const uint4*>(dy), static_cast<const uint4*>(y_perm), inv_perm, gates,
                     dgates, static_cast<uint4*>(dy_perm), L.T, L.Ke, vec_per_row);
  return hipGetLastError();
}

}  // namespace mohge
