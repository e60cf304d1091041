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
// A wave of the second kernel takes the 64 codes of one channel block of a filter (or of four filters of at most 16
// channels): lane = channel, so that a wave reads 2304 contiguous bytes of weights and a thread transforms one filter
// channel.  The codes cross LDS, wave by wave and without a barrier, into 16-byte pieces of code rows: one store per
// thread and one addition of row sums, where a thread of four channels made 16 and 16.
//
// What bounds it: launches and latencies, and for the largest layers the copies of the records, which the start of the
// second kernel waits for.  By the workgroups' clocks, 64 -> 128 channels: range kernel 2.4 us (1.2 weights, 0.6
// reduction), 1.2 until the next kernel starts, its records 1.8, constants 0.5, codes 0.9, sums 0.5.  Whole call, four
// channels per thread / now, on weights in the last-level cache and (cold) on sets that rotate past it: 3 -> 64 6.7 / 4.4
// (cold 6.6 / 5.1) us, 64 -> 64 7.8 / 6.6 (8.4 / 6.6), 128 -> 128 9.5 / 8.5 (9.8 / 8.7), 256 -> 256 11.4 / 10.8 (12.2 / 11.4), 512 -> 512
// 15.7 / 15.8 (17.5 / 17.5), 1024 -> 1024 41 / 30 (46 / 35), 64 -> 64 F(4x4) 15.9 / 12.8 (16.9 / 13.4); the thirteen 3x3
// layers of VGG-16 162 / 153 (186 / 176).  1500 random sets of 1 to 8192 channels and up to 65535 filters 1.26 at the median,
// five slower by more than 4 %.  (Weights through LDS in 16-byte loads were slower at every size.)
#include "lance_device.h"
#include "lance_internal.h"

namespace lance {
namespace {

struct FtArgs {
  const float* w;
  int8_t* uq;
  float* u_range;
  int32_t* u_rowsum;
  int C, K, CB, NB, row;  // row: bytes of a code row
  int bits, natural, packed, per_tensor;
  int ga, gb, cap;  // workgroups of the two kernels; records per code-row strip of a workgroup
  int base, extra;           // filters of a workgroup of the second kernel; the first `extra` have one more
  unsigned cap_magic, nb_magic;  // divisors for dev::fast_div (a division by a variable takes 0.1 us here)
};

// First filter of workgroup j of the second kernel: it owns these rows of uq.
__device__ __forceinline__ int first_filter(const FtArgs& a, int j) { return j * a.base + min(j, a.extra); }

// Address of position e of record r in the copy of the workgroup whose first filter is k0.
__device__ __forceinline__ float2* record(const FtArgs& a, int k0, int e, int r) {
  const int strip = dev::fast_div(r, a.cap_magic);
  return reinterpret_cast<float2*>(a.uq + (((size_t)e * a.NB + strip) * a.K + k0) * a.row) + (r - strip * a.cap);
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
    *record(a, first_filter(a, j), e, blockIdx.x) = res_s[e];
  }
}

// NARROW: codes of fewer than 8 bits.
template <int M, int NT, bool NARROW>
__global__ __launch_bounds__(NT) void filter_quant_kernel(const FtArgs a) {
  constexpr int A = M + 2, E = A * A, kThreads = NT, kParts = kThreads / E, kWaves = NT / 64;
  constexpr int kMaxFilters = 64;  // per workgroup
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  __shared__ float2 red[kThreads], res_s[E], qp_s[E];
  __shared__ int sum_s[kMaxFilters * E];
  __shared__ __align__(16) uint8_t rows_s[kWaves][E * 64 + 64];  // a wave's 64 codes of every position; byte mask
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k0 = first_filter(a, blockIdx.x), k1 = first_filter(a, blockIdx.x + 1);
  // the records of the range kernel are requested before the weights: loads return in order
  constexpr int kBatch = 8;
  const int e_red = tid % E, part = min(tid / E, kParts - 1);  // (threads beyond kParts * E repeat others)
  float2 rec[kBatch] = {};
  if (a.ga > 0) {
#pragma unroll
    for (int u = 0; u < kBatch; u++)  // (past the last record: the last one again)
      rec[u] = *record(a, k0, e_red, min(part + u * kParts, a.ga - 1));
  }
  // Unit: the 64 codes of one channel block of a filter, or of four filters of at most 16 channels.  Lane = code:
  // channel c of filter k.
  const bool wide = a.CB == 64;
  const int units = wide ? (k1 - k0) * a.NB : (k1 - k0 + 3) / 4;  // (narrow: one block)
  const int in_block = wide ? lane : lane & 15, sub = wide ? 0 : lane >> 4;
  auto filter_of = [&](int unit) { return wide ? dev::fast_div(unit, a.nb_magic) : 4 * unit; };  // from k0 on, the first
  auto block_of = [&](int unit) { return wide ? unit - dev::fast_div(unit, a.nb_magic) * a.NB : 0; };
  auto fetch = [&](int unit, float (&g)[9]) {
    const int c = block_of(unit) * 64 + in_block, k = k0 + filter_of(unit) + sub;
    const float* src = a.w + ((size_t)min(k, a.K - 1) * a.C + min(c, a.C - 1)) * 9;
#pragma unroll
    for (int i = 0; i < 9; i++) g[i] = src[i];
  };
  // the first unit's weights arrive while the ranges are reduced
  float g[9];
  if (wave < units) fetch(wave, g);
  for (int i = tid; i < (k1 - k0) * E; i += kThreads) sum_s[i] = 0;
  if (a.ga == 0) {
    float mn[E], mx[E];
    range_of<M>(a.w, tid, kThreads, a.K * a.C, mn, mx);
    reduce_range<M, kThreads>(mn, mx, red, res_s);
  } else {
    float2 v = rec[0];
#pragma unroll
    for (int u = 1; u < kBatch; u++) { v.x = fminf(v.x, rec[u].x); v.y = fmaxf(v.y, rec[u].y); }
    for (int r = part + kBatch * kParts; r < a.ga; r += kParts) {
      const float2 x = *record(a, k0, e_red, r);
      v.x = fminf(v.x, x.x); v.y = fmaxf(v.y, x.y);
    }
    red[tid] = v;
    __syncthreads();  // also: the workgroup's copy of the records has been read
    if (tid < E) {
#pragma unroll
      for (int q = 1; q < kParts; q++) {
        const float2 x = red[q * E + tid];
        v.x = fminf(v.x, x.x); v.y = fmaxf(v.y, x.y);
      }
      res_s[tid] = v;
    }
    if (a.per_tensor) __syncthreads();
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
  // bytes u - h (mod 256); u <= 127 for codes below 8 bits
  auto to_signed = [&](unsigned u) -> unsigned { return h == 128u ? u ^ H8 : ((u | H8) - hh) ^ H8; };
  float2 qp[E];  // (F(4x4): read again for every unit instead of living in 72 registers)
#pragma unroll
  for (int e = 0; e < E; e++)
    if constexpr (M == 2) qp[e] = qp_s[e];
  // byte of the lane's code among the unit's 64: its code row's, NCHW channel c of a block at 4 * (c % Q) + c / Q
  const int byte = sub * 16 + (a.natural ? in_block : wide ? 4 * (in_block & 15) + (in_block >> 4)
                                                          : 4 * (in_block & 3) + (in_block >> 2));
  uint8_t* mine = rows_s[wave];
  for (int unit = wave; unit < units; unit += kWaves) {
    const int b = block_of(unit), kl = filter_of(unit);
    float gq[3][3], u[A][A];
#pragma unroll
    for (int i = 0; i < 9; i++) gq[i / 3][i % 3] = g[i];
    dev::filter_tile_transform<M>(gq, u);
    if (unit + kWaves < units) fetch(unit + kWaves, g);  // (in flight under this unit's codes)
    mine[E * 64 + byte] = b * 64 + in_block < a.C ? 0xFF : 0;  // bytes of channels that do not exist become 0
#pragma unroll
    for (int e = 0; e < E; e++) {
      const float2 p = M == 2 ? qp[e] : qp_s[e];
      // clamp(rne((x - min) * inv), 0, L): the conversion rounds to nearest even and saturates to
      // [0, 255].  The ranges are those of these filters, but where x - min overflows the product is
      // infinite, and 0 * infinity is undefined: those are L and (the median with one undefined value
      // is the least of the others; the conversion's result, too) 0
      float t = (u[e / A][e % A] - p.x) * p.y;
      if constexpr (NARROW) t = __builtin_amdgcn_fmed3f(t, 0.0f, L);
      mine[e * 64 + byte] = (uint8_t)__builtin_amdgcn_cvt_pk_u8_f32(t, 0, 0u);
    }
    asm volatile("" ::: "memory");  // (a wave's LDS operations complete in order)
    // Back as 16-byte pieces of the rows: position i / 4, piece i % 4.  Pieces of narrow rows belong to filters.
#pragma unroll
    for (int i = lane; i < E * 4; i += 64) {
      const int e = i >> 2, piece = i & 3;
      const int own = kl + (wide ? 0 : piece);
      v4u v = *reinterpret_cast<const v4u*>(mine + i * 16);
      const v4u mask = *reinterpret_cast<const v4u*>(mine + E * 64 + piece * 16);
      int sum = 0;
#pragma unroll
      for (int d = 0; d < 4; d++) {
        v[d] = to_signed(v[d]) & mask[d];
        sum = __builtin_amdgcn_sdot4((int)v[d], 0x01010101, sum, false);
      }
      const bool ok = k0 + own < k1;
      int8_t* row = a.uq + (((size_t)e * a.NB + b) * a.K + k0 + own) * a.row;
      if (a.packed) {
        // byte q: the codes of bytes q (low nibble) and 32 + q, each as code + 8
        if (piece < 2) {
          const v4u hi = *reinterpret_cast<const v4u*>(mine + i * 16 + 32);
          const v4u hi_mask = *reinterpret_cast<const v4u*>(mine + E * 64 + piece * 16 + 32);
          v4u w;
#pragma unroll
          for (int d = 0; d < 4; d++)
            w[d] = ((v[d] & 0x0F0F0F0Fu) ^ 0x08080808u) |
                   ((((to_signed(hi[d]) & hi_mask[d]) & 0x0F0F0F0Fu) ^ 0x08080808u) << 4);
          *reinterpret_cast<v4u*>(row + 16 * piece) = w;
        }
      } else if (ok) {
        *reinterpret_cast<v4u*>(row + (wide ? 16 * piece : 0)) = v;
      }
      if (wide) {  // the four pieces of a row
        sum += __builtin_amdgcn_update_dpp(0, sum, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
      }
      if (ok && (!wide || piece == 0)) atomicAdd(&sum_s[own * E + e], sum);
    }
    asm volatile("" ::: "memory");
  }
  __syncthreads();
  for (int i = tid; i < E * kMaxFilters; i += kThreads) {
    const int e = i / kMaxFilters, kl = i % kMaxFilters;
    if (kl < k1 - k0) a.u_rowsum[(size_t)e * a.K + k0 + kl] = sum_s[kl * E + e];
  }
}

}  // namespace

hipError_t launch_filter_transform(const Geo& g, const float* w, int8_t* uq, float* u_range,
                                   int32_t* u_rowsum, hipStream_t s) {
  FtArgs a{w, uq, u_range, u_rowsum, g.C, g.K, g.CB, g.NB, code_row_bytes(g), g.bits_w,
           is_nhwc(g) ? 1 : 0, is_packed(g) ? 1 : 0, (g.flags & LANCE_RANGE_PER_TENSOR) ? 1 : 0, 0, 0, 1};
  const long long filters = (long long)g.K * g.C;
  // Up to 4096 filters every workgroup of the second kernel finds the ranges itself.
  const bool one_kernel = filters <= 4096, large = filters > 81920, wide = g.CB == 64;
  const long long units = wide ? (long long)g.K * g.NB : (g.K + 3) / 4;
  // Copies of the records that the first kernel writes: at most 64, 128 or 256 (512 -> 512 channels: the start of the second
  // kernel waits 3.3 us behind the last workgroup of the first with 128 copies of 8 KB, 4.9 with 256, 1.2 where there
  // are few), the more the longer the second kernel takes.
  long long most = filters > 400000 ? 256 : large ? 128 : 64;
  if (wide && units > 1024 && most < 128) most = 128;
  if (wide && units > 6000) most = 256;
  // Small workgroups have the shorter chain of steps, large ones keep the number of records and copies down, and where
  // few filters of many channels allow few workgroups they have the waves for their units (us with 256 / 512 / 1024
  // threads: 6066 -> 2 F(2x2) 25.4 / 17.4 / 16.7, 4066 -> 4 F(4x4) 35.7 / 25.1 / 22.7).  512 or 1024 from the number of units to
  // a workgroup on; 1200 random sets of filters: 1.02 over the best of twelve choices on average.
  const int nt_range = large ? 1024 : 256;
  int nt_quant = one_kernel ? (filters > 1024 ? 1024 : 256) : (filters > 24576 ? 512 : 256);
  if (wide && !one_kernel) {
    const long long each = (units + (most < g.K ? most : g.K) - 1) / (most < g.K ? most : g.K);
    if (each > (g.m == 2 ? 12 : 8) && nt_quant < 512) nt_quant = 512;
    if (g.m == 4 && each > 32) nt_quant = 1024;
  }
  // Workgroups of the second kernel: a unit of 64 codes per wave, then several, at most 64 filters each, and all the same
  // number of filters where that takes no longer (7975 -> 248 F(4x4) on 243 workgroups, five of them with two filters, 99.6 us,
  // on 248 69.7).
  const long long waves = nt_quant / 64, per_wave = (units + waves * most - 1) / (waves * most);
  long long gb = (units + waves * per_wave - 1) / (waves * per_wave);
  if (gb < (g.K + 63) / 64) gb = (g.K + 63) / 64;
  if (gb > g.K) gb = g.K;
  const long long own = (g.K + gb - 1) / gb;
  gb = own == 2 && g.K <= most ? g.K : (g.K + own - 1) / own;
  a.gb = (int)gb;
  a.base = g.K / a.gb;
  a.extra = g.K % a.gb;
  // Records that fit into the rows of the workgroup with the fewest filters.
  a.cap = a.base * a.row / 8;
  const long long room = (long long)a.cap * g.NB;
  long long ga = large ? (filters + 2047) / 2048 : (filters + 1023) / 1024;
  if (large && ga > 64) ga = 64;
  if (ga > room) ga = room;
  a.ga = one_kernel ? 0 : (int)ga;
  a.cap_magic = div_magic(a.cap);
  a.nb_magic = div_magic(a.NB);
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
    auto tile = [&](auto m) -> hipError_t {
      constexpr int kM = decltype(m)::value;
      return large && nt_quant == 1024 ? run(filter_range_kernel<kM, 1024>, filter_quant_kernel<kM, 1024, kNarrow>)
             : large             ? run(filter_range_kernel<kM, 1024>, filter_quant_kernel<kM, 512, kNarrow>)
             : nt_quant == 1024 ? run(filter_range_kernel<kM, 256>, filter_quant_kernel<kM, 1024, kNarrow>)
             : nt_quant == 512  ? run(filter_range_kernel<kM, 256>, filter_quant_kernel<kM, 512, kNarrow>)
                                : run(filter_range_kernel<kM, 256>, filter_quant_kernel<kM, 256, kNarrow>);
    };
    return g.m == 2 ? tile(std::integral_constant<int, 2>{}) : tile(std::integral_constant<int, 4>{});
  };
  return g.bits_w < 8 ? sized(std::true_type{}) : sized(std::false_type{});
}

}  // namespace lance
