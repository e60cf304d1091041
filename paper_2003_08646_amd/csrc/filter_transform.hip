// Stage 1: u^ = Q(G g G^T) for every filter (Algorithm 1; Eq. 7).  Runs once per set of
// weights (Sec. 3.4).
//
//   filter_range_kernel  `ga` workgroups: transform every (k,c) of their share, reduce (min,max) per
//                        position e to one record.
//   filter_quant_kernel  `gb` workgroups of a few filters each: reduce the records to the ranges and
//                        form the Eq. 7 parameters, transform again, quantize, store the codes in
//                        the blocked/permuted layout, reduce the code sums -> u_rowsum[e][k].
//
// The call has no scratch memory, so the records lie in uq itself - one private copy for every
// workgroup of the second kernel, inside the rows that this workgroup will write: it has read its
// copy before it writes its first code, and no other workgroup touches those rows.  (One copy for
// all would need a kernel between the two, as it did before: one workgroup's codes would overwrite
// records that another one has not read.)  Small sets of filters need no first kernel: every
// workgroup finds the ranges by itself.
//
// A thread of the second kernel forms whole dwords of a code row (four channels), so that 16 lanes
// store 64 contiguous bytes per position.
//
// What bounds it: launches and latencies.  Kernel times before, with a one-workgroup reduction kernel
// between the two: 512 -> 512 channels (9.4 MB of weights) 9.1 + 4.7 + 9.2 us, 64 -> 64 6.6 + 4.6 + 6.6
// us; now 9.3 + 8.6 us, and about 7 us in one kernel.
#include "lance_device.h"
#include "lance_internal.h"

namespace lance {
namespace {

// Rows of uq that workgroup j of n of the second kernel owns: filters first_filter(j) .. (j+1).
__device__ __host__ __forceinline__ int first_filter(int j, int n, int K) {
  return (int)((long long)j * K / n);
}

struct FtArgs {
  const float* w;
  int8_t* uq;
  float* u_range;
  int32_t* u_rowsum;
  int C, K, CB, NB, Q, row;  // row: bytes of a code row
  int bits, natural, packed, per_tensor;
  int ga, gb, cap;  // workgroups of the two kernels; records per code-row strip of a workgroup
};

// Address of position e of record r in the copy of the workgroup whose first filter is k0.
__device__ __forceinline__ float2* record(const FtArgs& a, int k0, int e, int r) {
  return reinterpret_cast<float2*>(a.uq + (((size_t)e * a.NB + r / a.cap) * a.K + k0) * a.row) + r % a.cap;
}

// Running (min,max) per position of filters i0, i0 + step, ... below n; four are requested together.
template <int M>
__device__ __forceinline__ void range_of(const float* w, int i0, int step, int n,
                                         float (&mn)[(M + 2) * (M + 2)], float (&mx)[(M + 2) * (M + 2)]) {
  constexpr int A = M + 2, E = A * A, kBatch = M == 2 ? 4 : 2;
#pragma unroll
  for (int e = 0; e < E; e++) { mn[e] = INFINITY; mx[e] = -INFINITY; }
  for (int i = i0; i < n; i += kBatch * step) {
    float g[kBatch][9];
#pragma unroll
    for (int b = 0; b < kBatch; b++) {
      const float* src = w + (size_t)min(i + b * step, n - 1) * 9;  // (the last filter twice: harmless)
#pragma unroll
      for (int r = 0; r < 9; r++) g[b][r] = src[r];
    }
#pragma unroll
    for (int b = 0; b < kBatch; b++) {
      float gq[3][3], u[A][A];
#pragma unroll
      for (int r = 0; r < 9; r++) gq[r / 3][r % 3] = g[b][r];
      dev::filter_tile_transform<M>(gq, u);
#pragma unroll
      for (int e = 0; e < E; e++) {
        mn[e] = fminf(mn[e], u[e / A][e % A]);
        mx[e] = fmaxf(mx[e], u[e / A][e % A]);
      }
    }
  }
}

// Reduces the workgroup's (min,max) sets into res_s[e] = {min, max}; all threads; ends in a barrier.
template <int M, int NT>
__device__ __forceinline__ void reduce_range(const float (&mn)[(M + 2) * (M + 2)],
                                             const float (&mx)[(M + 2) * (M + 2)], float2* red, float2* res_s) {
  constexpr int E = (M + 2) * (M + 2), NP = M == 2 ? 16 : 32, kWaves = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float lo, hi;
  dev::wave_minmax_scatter<NP>(mn, mx, lane, &lo, &hi);
  if (lane % (64 / NP) == 0) red[wave * E + lane / (64 / NP)] = float2{lo, hi};
  if constexpr (M == 4) {
#pragma unroll
    for (int e = 32; e < E; e++) {
      const float l = dev::wave_min(mn[e]), h = dev::wave_max(mx[e]);
      if (lane == 0) red[wave * E + e] = float2{l, h};
    }
  }
  __syncthreads();
  if (threadIdx.x < E) {
    float2 v = red[threadIdx.x];
#pragma unroll
    for (int wv = 1; wv < kWaves; wv++) {
      const float2 x = red[wv * E + threadIdx.x];
      v.x = fminf(v.x, x.x); v.y = fmaxf(v.y, x.y);
    }
    res_s[threadIdx.x] = v;
  }
  __syncthreads();
}

template <int M, int NT>
__global__ __launch_bounds__(NT) void filter_range_kernel(const FtArgs a) {
  constexpr int E = (M + 2) * (M + 2);
  __shared__ float2 red[NT / 64 * E], res_s[E];
  float mn[E], mx[E];
  range_of<M>(a.w, blockIdx.x * NT + threadIdx.x, a.ga * NT, a.K * a.C, mn, mx);
  reduce_range<M, NT>(mn, mx, red, res_s);
  // the same record into every workgroup's copy: threads walk (copy, position)
  for (int i = threadIdx.x; i < a.gb * E; i += NT) {
    const int j = i / E, e = i % E;
    *record(a, first_filter(j, a.gb, a.K), e, blockIdx.x) = res_s[e];
  }
}

// NARROW: codes of fewer than 8 bits.
template <int M, int NT, bool NARROW>
__global__ __launch_bounds__(NT) void filter_quant_kernel(const FtArgs a) {
  constexpr int A = M + 2, E = A * A, kThreads = NT, kParts = kThreads / E;
  constexpr int kMaxFilters = 64;  // per workgroup
  __shared__ float2 red[kThreads], res_s[E], qp_s[E];
  __shared__ int sum_s[kMaxFilters * E];
  const int tid = threadIdx.x;
  const int k0 = first_filter(blockIdx.x, a.gb, a.K), k1 = first_filter(blockIdx.x + 1, a.gb, a.K);
  for (int i = tid; i < (k1 - k0) * E; i += kThreads) sum_s[i] = 0;
  // The weights of dword dw of block b of filter k: byte q of the dword is channel b*CB + dw + Q*q
  // (natural order: 4*dw + q).  mask: the bytes whose channel exists.
  auto fetch = [&](int k, int b, int dw, float (&gw)[4][9], unsigned& mask) {
    mask = 0;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int c = b * a.CB + (a.natural ? 4 * dw + q : dw + a.Q * q);
      const float* src = a.w + ((size_t)k * a.C + min(c, a.C - 1)) * 9;
#pragma unroll
      for (int i = 0; i < 9; i++) gw[q][i] = src[i];
      if (c < a.C) mask |= 0xFFu << (8 * q);
    }
  };
  const int per_row = a.packed ? 8 : a.Q;  // dwords of a code row
  const int items = (k1 - k0) * a.NB * per_row;
  // the first item's weights arrive while the ranges are reduced
  float gw[4][9];
  unsigned mask = 0;
  if (tid < items) fetch(k0 + tid / per_row / a.NB, tid / per_row % a.NB, tid % per_row, gw, mask);
  if (a.ga == 0) {
    float mn[E], mx[E];
    range_of<M>(a.w, tid, kThreads, a.K * a.C, mn, mx);
    reduce_range<M, kThreads>(mn, mx, red, res_s);
  } else {
    const int e = tid % E, part = tid / E;
    float2 v = {INFINITY, -INFINITY};
    if (part < kParts) {
      constexpr int kBatch = 8;
      for (int r0 = part; r0 < a.ga; r0 += kBatch * kParts) {
        float2 x[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; u++) {
          const int r = r0 + u * kParts;
          x[u] = r < a.ga ? *record(a, k0, e, r) : v;
        }
#pragma unroll
        for (int u = 0; u < kBatch; u++) { v.x = fminf(v.x, x[u].x); v.y = fmaxf(v.y, x[u].y); }
      }
      red[tid] = v;
    }
    __syncthreads();  // also: the workgroup's copy of the records has been read
    if (tid < E) {
#pragma unroll
      for (int q = 1; q < kParts; q++) {
        const float2 x = red[q * E + tid];
        v.x = fminf(v.x, x.x); v.y = fmaxf(v.y, x.y);
      }
      res_s[tid] = v;
    }
    __syncthreads();
  }
  if (tid < E) {
    float2 v = res_s[tid];
    if (a.per_tensor)
      for (int e = 0; e < E; e++) { v.x = fminf(v.x, res_s[e].x); v.y = fmaxf(v.y, res_s[e].y); }
    float inv, scale;
    dev::quant_params(v.x, v.y, a.bits, &inv, &scale);
    qp_s[tid] = float2{v.x, inv};
    if (blockIdx.x == 0) { a.u_range[2 * tid] = v.x; a.u_range[2 * tid + 1] = v.y; }
  }
  __syncthreads();

  const float L = (float)((1 << a.bits) - 1);
  const unsigned h = 1u << (a.bits - 1), hh = h * 0x01010101u, H8 = 0x80808080u;
  // codes: Eq. 7's unsigned codes of the four channels, 0 where the channel does not exist
  auto dword_of = [&](const float (&gw)[4][9], unsigned mask, unsigned (&codes)[E]) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      float gq[3][3], u[A][A];
#pragma unroll
      for (int i = 0; i < 9; i++) gq[i / 3][i % 3] = gw[q][i];
      dev::filter_tile_transform<M>(gq, u);
#pragma unroll
      for (int e = 0; e < E; e++) {
        const float2 p = qp_s[e];
        // clamp(rne((x - min) * inv), 0, L): the conversion rounds to nearest even and saturates to
        // [0, 255].  The ranges are those of these filters, but where x - min overflows the product is
        // infinite, and 0 * infinity is undefined: those are L and (the median with one undefined value
        // is the least of the others; the conversion's result, too) 0
        float t = (u[e / A][e % A] - p.x) * p.y;
        if constexpr (NARROW) t = __builtin_amdgcn_fmed3f(t, 0.0f, L);
        codes[e] = __builtin_amdgcn_cvt_pk_u8_f32(t, q, q == 0 ? 0u : codes[e]);
      }
      // (one channel after the other, and the parameters read again for each)
#pragma unroll
      for (int e = 0; e < E; e++) asm volatile("" : "+v"(codes[e]));
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int e = 0; e < E; e++) codes[e] &= mask;
  };
  // bytes u - h (mod 256) where the channel exists, else 0; u <= 127 for codes below 8 bits
  auto to_signed = [&](unsigned u, unsigned mask) -> unsigned {
    return (h == 128u ? u ^ H8 : ((u | H8) - hh) ^ H8) & mask;
  };
  for (int i = tid; i < items; i += kThreads) {
    const int dw = i % per_row, t = i / per_row;
    const int b = t % a.NB, kl = t / a.NB;
    int8_t* dst = a.uq + ((size_t)b * a.K + k0 + kl) * a.row + 4 * dw;
    const size_t estride = (size_t)a.NB * a.K * a.row;
    unsigned codes[E];
    if (i != tid) fetch(k0 + kl, b, dw, gw, mask);
    dword_of(gw, mask, codes);
    if (a.packed) {
      // byte q: the codes at positions 4*dw + q (low nibble) and 32 + 4*dw + q, each as code + 8
      unsigned hi[E], mask_hi;
      fetch(k0 + kl, b, dw + 8, gw, mask_hi);
      dword_of(gw, mask_hi, hi);
      const int off = (int)(h * (unsigned)((__popc(mask) + __popc(mask_hi)) / 8));
#pragma unroll
      for (int e = 0; e < E; e++) {
        const int sum = (int)__builtin_amdgcn_sad_u8(hi[e], 0u, __builtin_amdgcn_sad_u8(codes[e], 0u, 0u)) - off;
        atomicAdd(&sum_s[kl * E + e], sum);
        const unsigned lo4 = (to_signed(codes[e], mask) & 0x0F0F0F0Fu) ^ 0x08080808u;
        const unsigned hi4 = (to_signed(hi[e], mask_hi) & 0x0F0F0F0Fu) ^ 0x08080808u;
        *reinterpret_cast<unsigned*>(dst + e * estride) = lo4 | (hi4 << 4);
      }
    } else {
      const int off = (int)(h * (unsigned)(__popc(mask) / 8));
#pragma unroll
      for (int e = 0; e < E; e++) {
        *reinterpret_cast<unsigned*>(dst + e * estride) = to_signed(codes[e], mask);
        int sum = (int)__builtin_amdgcn_sad_u8(codes[e], 0u, 0u) - off;
        if (per_row == 16) {  // the 16 lanes of a code row: one filter, all present
          sum = dev::row16_sum(sum);
          if (dw == 0) atomicAdd(&sum_s[kl * E + e], sum);
        } else {
          atomicAdd(&sum_s[kl * E + e], sum);
        }
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < (k1 - k0) * E; i += kThreads) {
    const int e = i / (k1 - k0), kl = i % (k1 - k0);
    a.u_rowsum[(size_t)e * a.K + k0 + kl] = sum_s[kl * E + e];
  }
}

}  // namespace

hipError_t launch_filter_transform(const Geo& g, const float* w, int8_t* uq, float* u_range,
                                   int32_t* u_rowsum, hipStream_t s) {
  FtArgs a{w, uq, u_range, u_rowsum, g.C, g.K, g.CB, g.NB, g.Q, code_row_bytes(g), g.bits_w,
           is_nhwc(g) ? 1 : 0, is_packed(g) ? 1 : 0, (g.flags & LANCE_RANGE_PER_TENSOR) ? 1 : 0, 0, 0, 1};
  const long long filters = (long long)g.K * g.C;
  // Small workgroups have the shorter chain of steps, large ones keep the number of records and
  // copies down: 256 threads up to 80 K filters (32 -> 400 channels: 9.8 us against 11.9 with 1024 and
  // 512 threads), then 1024 and 512 (443 -> 222: 15.5 us against 17.1).
  const bool large = filters > 81920;
  const int nt_range = large ? 1024 : 256, nt_quant = large ? 512 : 256;
  // Workgroups of the second kernel: one item (four or eight channels) per thread, at most 64
  // filters each.
  const long long items = (long long)g.K * g.NB * (is_packed(g) ? 8 : g.Q);
  long long gb = (items + nt_quant - 1) / nt_quant;
  if (gb < (g.K + 63) / 64) gb = (g.K + 63) / 64;
  if (gb > g.K) gb = g.K;
  a.gb = (int)gb;
  // Records that fit into the rows of the workgroup with the fewest filters.
  a.cap = (int)(g.K / gb) * a.row / 8;
  const long long room = (long long)a.cap * g.NB;
  long long ga = large ? (filters + 2047) / 2048 : (filters + 1023) / 1024;
  if (large && ga > 64) ga = 64;
  if (ga > room) ga = room;
  // Up to 4096 filters every workgroup of the second kernel finds the ranges itself (16 -> 16
  // channels: 7.5 us in two kernels, 5.2 in one; 80 -> 192: 13.9 us in two, 39 in one).
  a.ga = filters <= 4096 ? 0 : (int)ga;
  auto run = [&](auto range, auto quant) -> hipError_t {
    if (a.ga > 0) {
      range<<<a.ga, nt_range, 0, s>>>(a);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    quant<<<a.gb, nt_quant, 0, s>>>(a);
    return hipGetLastError();
  };
  auto sized = [&](auto narrow) -> hipError_t {
    constexpr bool kNarrow = decltype(narrow)::value;
    if (g.m == 2)
      return large ? run(filter_range_kernel<2, 1024>, filter_quant_kernel<2, 512, kNarrow>)
                   : run(filter_range_kernel<2, 256>, filter_quant_kernel<2, 256, kNarrow>);
    return large ? run(filter_range_kernel<4, 1024>, filter_quant_kernel<4, 512, kNarrow>)
                 : run(filter_range_kernel<4, 256>, filter_quant_kernel<4, 256, kNarrow>);
  };
  return g.bits_w < 8 ? sized(std::true_type{}) : sized(std::false_type{});
}

}  // namespace lance
