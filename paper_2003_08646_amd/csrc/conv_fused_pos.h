// Stages 2 (second pass) + 3 + 4 in one kernel for layers with few tiles, any number of channels:
// the work of 16 tiles x 16*KG filters is spread over a workgroup of 16 waves (m = 2) or 12 waves
// (m = 4), so that a layer of a few thousand outputs still fills the chip and the chain of
// dependent steps of a workgroup is short.  The other fused plans give a wave all positions of its
// filters and walk the filters one block after the other: on such layers they are a handful of
// workgroups, each a chain of tens of microseconds.
//
//   Phase T.  All waves transform and quantize (v^ = Q(B^T d B), Algorithm 1; Eq. 7) the 16 tiles'
//     channels into LDS code rows [E][blocks][16 tiles][64 B]: CPL = 4: a lane takes the four
//     channels of one dword (the layout of lance.h), CPL = 1: one channel, so that layers of at
//     most 128 channels still give every wave something to do.
//   Phase G.  Wave w owns the positions w*E/NW ..: v_mfma_i32_16x16x64_i8 over all channel blocks,
//     uq fragments straight from memory (each is used once per workgroup), codes of V from LDS.
//     One more matrix instruction per block with an operand of ones gives the column sums.
//   Exchange.  Each wave turns its positions' sums into M[e,k,p] (Eq. 8, expanded) and writes them
//     to LDS; every thread then gathers the E values of a (filter, tile) pair, applies A^T M A
//     (Eq. 9) and stores the patch.
//
// Codes narrower than 8 bits stay unsigned in LDS (they are non-negative int8 values); the filter
// row sums take the difference off the integer sums.  So do the column sums for packed filter
// codes, which are multiplied as code + 8.  Both are exact.
//
// The transform is repeated by each of the ceil(K / (16*KG)) workgroups of a tile block: the plan
// is for layers that leave the chip idle otherwise (conv_fused_pos_preferred).
//
// What bounds it: the chain launch - pixels and ranges from memory (about 2 us) - constants -
// transform - uq fragments - exchange - stores of one workgroup; 6 us for the smallest layers with
// caller-supplied ranges, launch included (N122 16->16 7x7; 19 us before on conv_fused_c16), 11 us
// with the range pass (one 16->16 32x32 image: 24.8 us before).  One image of the 512-channel 14x14
// layer: 21 -> 13.3 us, N13 100->72 37x29 F(4x4): 43 -> 18 us.
#pragma once
#include "lance_device.h"
#include "lance_internal.h"
#include "tile_loader.h"

namespace lance {
namespace pos {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

struct CpArgs {
  const float* x;
  const int8_t* uq;
  const float* u_range;     // [E][2]
  const int32_t* u_rowsum;  // [E][K]
  const float* partial;     // [count][E][2] records of the range pass (dynamic ranges)
  float* v_range;           // [E][2]: written by workgroup 0, or read when is_static
  float* y;
  int count, per_tensor, is_static;
  int N, C, H, W, K, pad, P, th, tw, Ho, Wo, bits, bits_w;
  int NB, Q;     // channel blocks; dwords per code row (16, or 4 for layers of at most 16 channels)
  int uq_mode;   // 0: 64-byte rows, 1: 16-byte rows (at most 16 channels), 2: packed 32-byte rows
  int nky;       // filter splits of 16*KG filters
  unsigned x_bytes, y_bytes;
};

constexpr unsigned kOobY = 0xFFFFFFF0u;

// channel blocks whose codes are in LDS at a time
template <int M> constexpr int chunk_blocks() { return M == 2 ? 8 : 3; }
constexpr int kConstBytes = 2048;  // parameter tables at the start of LDS

__device__ __forceinline__ int swz(int row) { return (row >> 2) & 3; }

template <int M>
__device__ __forceinline__ void store_row(float* y, unsigned y_bytes, unsigned off, const float (&v)[M]) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(y, 0, y_bytes, 0x00020000);
  if constexpr (M == 2) {
    const v2u u = {__float_as_uint(v[0]), __float_as_uint(v[1])};
    __builtin_amdgcn_raw_buffer_store_b64(u, r, off, 0, 0);
  } else {
    const v4u u = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
    __builtin_amdgcn_raw_buffer_store_b128(u, r, off, 0, 0);
  }
}
__device__ __forceinline__ void store_b32(float* y, unsigned y_bytes, unsigned off, float v) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(y, 0, y_bytes, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, 0, 0);
}

// MULTI: more channel blocks than LDS holds at a time (KG = 1 only: the sums live across phase T).
template <int M, int NW, int CPL, int KG, int LOAD, bool CLAMP, bool MULTI>
__global__ __launch_bounds__(NW * 64, (M == 2 ? 16 : 12) / 4) void conv_fused_pos_kernel(const CpArgs a) {
  constexpr int A = M + 2, E = A * A, NT = NW * 64, PW = E / NW;
  constexpr int NBC = chunk_blocks<M>();
  // the next channel's pixels are requested before the current channel's arithmetic (registers)
  constexpr bool kPrefetch = !(M == 4 && MULTI);
  constexpr bool kNhwc = LOAD == kNhwc1 || LOAD == kNhwc4;
  extern __shared__ char smem[];
  float* qp_s = reinterpret_cast<float*>(smem);         // [E][2] = {min, inv} of Eq. 7
  float* res_s = qp_s + 2 * E;                          // [E][2] reduced ranges
  float* sc_s = res_s + 2 * E;                          // [E] su*sv
  float* gc_s = sc_s + E;                               // [E] sv*ou
  double* rmul_s = reinterpret_cast<double*>(gc_s + E); // [E] su*ov
  double* kc_s = rmul_s + E;                            // [E] C*ou*ov
  static_assert(E * (6 * sizeof(float) + 2 * sizeof(double)) <= kConstBytes, "parameter tables");
  char* ring = smem + kConstBytes;
  float* ex = reinterpret_cast<float*>(ring);           // the exchange reuses the code rows
  float* red = reinterpret_cast<float*>(ring);          // so does the reduction of the records

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the filter splits of a tile block are neighbours, so that with several splits each die's L2
  // holds few of them
  const int ky = blockIdx.x % a.nky, p0 = (blockIdx.x / a.nky) * 16, k0 = ky * 16 * KG;
  const int K = a.K, P = a.P, C = a.C;
  const bool b8 = a.bits == 8;

  // ---- the lane's tile ----
  // NCHW: 16 tiles x 4 dwords per wave; NHWC: channels fastest, for the coalescing of the loads
  const int trow = LOAD == kNhwc4 ? lane >> 2 : (LOAD == kNhwc1 ? 4 * (wave & 3) + (lane >> 4) : lane & 15);
  const int dl = LOAD == kNhwc4 ? lane & 3 : (LOAD == kNhwc1 ? lane & 15 : lane >> 4);
  const TileGeo tg{a.x, a.x_bytes, a.N, C, a.H, a.W, a.pad, P, a.th, a.tw};
  TileLoader<M, LOAD> tl;
  tl.setup(tg, min(p0 + trow, P - 1), dl);
  auto load = [&](int cu, float (&b)[A * A]) { tl.load(tg, cu, b); };
  const float L = (float)((1 << a.bits) - 1);
  // code q (byte) of the dword codes[e] from the patch b
  auto quantize = [&](const float (&b)[A * A], auto qc, unsigned (&codes)[E]) {
    constexpr int q = decltype(qc)::value;
    // (F(4x4): the parameters are read again for every channel instead of living in 72 registers)
    if constexpr (M == 4) asm volatile("" ::: "memory");
    float d[A][A];
    tl.mask(b, d);
    dev::input_tile_transform<M>(d);
#pragma unroll
    for (int e = 0; e < E; e++) {
      const v2f mi = *reinterpret_cast<const v2f*>(qp_s + 2 * e);
      float t = (d[e / A][e % A] - mi[0]) * mi[1];
      if constexpr (CLAMP) t = fminf(t, L);  // above 8 bits' range the conversion saturates by itself
      codes[e] = __builtin_amdgcn_cvt_pk_u8_f32(t, q, q == 0 ? 0u : codes[e]);
    }
    // ties this channel's arithmetic to its step (left alone, the compiler moves all channels'
    // arithmetic behind the last load)
#pragma unroll
    for (int e = 0; e < E; e++) asm volatile("" : "+v"(codes[e]));
  };
  const unsigned flip = b8 ? 0x80808080u : 0u;  // 8-bit codes are stored signed

  // ---- Eq. 7 / Eq. 8 constants ----
  auto constants = [&]() {
    float su = 0.0f;
    double ou = 0.0;
    float ur0 = 0.0f, ur1 = 0.0f;
    if (tid < E) { ur0 = a.u_range[2 * tid]; ur1 = a.u_range[2 * tid + 1]; }
    if (a.is_static) {
      if (tid < 2 * E) res_s[tid] = a.v_range[tid];
    } else {
      constexpr int kCols = 2 * E, kGroups = NT / kCols, kBatch = 8;
      const int col = tid % kCols, grp = tid / kCols;
      const bool is_max = col & 1;
      float v = is_max ? -INFINITY : INFINITY;
      if (grp < kGroups) {
        for (int row0 = grp; row0 < a.count; row0 += kBatch * kGroups) {
          float xv[kBatch];
#pragma unroll
          for (int u = 0; u < kBatch; u++) {
            const int row = row0 + u * kGroups;
            xv[u] = row < a.count ? a.partial[(size_t)row * kCols + col] : v;
          }
#pragma unroll
          for (int u = 0; u < kBatch; u++) v = is_max ? fmaxf(v, xv[u]) : fminf(v, xv[u]);
        }
      }
      red[tid] = v;
      __syncthreads();
      if (tid < kCols) {
#pragma unroll
        for (int g2 = 1; g2 < kGroups; g2++) {
          const float y = red[g2 * kCols + tid];
          v = is_max ? fmaxf(v, y) : fminf(v, y);
        }
        res_s[tid] = v;
      }
    }
    if (tid < E) {
      float iu;
      dev::quant_params(ur0, ur1, a.bits_w, &iu, &su);
      ou = (double)ur0 + (double)su * (double)(1 << (a.bits_w - 1));
    }
    __syncthreads();
    if (tid < E) {
      float lo = res_s[2 * tid], hi = res_s[2 * tid + 1];
      if (a.per_tensor && !a.is_static)
        for (int e = 0; e < E; e++) { lo = fminf(lo, res_s[2 * e]); hi = fmaxf(hi, res_s[2 * e + 1]); }
      float inv, sv;
      dev::quant_params(lo, hi, a.bits, &inv, &sv);
      qp_s[2 * tid] = lo;
      qp_s[2 * tid + 1] = inv;
      const double ov = (double)lo + (double)sv * (double)(1 << (a.bits - 1));
      sc_s[tid] = (float)((double)su * (double)sv);
      gc_s[tid] = (float)((double)sv * ou);
      rmul_s[tid] = (double)su * ov;
      kc_s[tid] = (double)C * ou * ov;
      if (!a.is_static && blockIdx.x == 0) {
        a.v_range[2 * tid] = lo;
        a.v_range[2 * tid + 1] = hi;
      }
    }
    __syncthreads();
  };

  // ---- products: positions wave*PW .., accumulators [position][group of 16 filters] ----
  const int col = lane & 15, kq = lane >> 4;  // fragment row; 16-byte piece of the 64 channels
  const unsigned f_off = (unsigned)col * 64u + (unsigned)((kq ^ swz(col)) * 16);
  v4i acc[PW][KG], csum[PW];
  auto clear_acc = [&]() {
#pragma unroll
    for (int w = 0; w < PW; w++) {
      csum[w] = v4i{0, 0, 0, 0};
#pragma unroll
      for (int kg = 0; kg < KG; kg++) acc[w][kg] = v4i{0, 0, 0, 0};
    }
  };
  if constexpr (MULTI) clear_acc();
  auto load_uq = [&](int e, int b, int kg) -> v4i {
    const int krow = min(k0 + kg * 16 + col, K - 1);
    if (a.uq_mode == 0)
      return *reinterpret_cast<const v4i*>(a.uq + (((size_t)e * a.NB + b) * K + krow) * 64 + 16 * kq);
    v4i f = {0, 0, 0, 0};
    if (a.uq_mode == 1) {
      if (kq == 0) f = *reinterpret_cast<const v4i*>(a.uq + ((size_t)e * K + krow) * 16);
      return f;
    }
    // packed: byte q of the 64-byte row is the low nibble of byte q (q < 32) or the high one of q - 32
    f = *reinterpret_cast<const v4i*>(a.uq + (((size_t)e * a.NB + b) * K + krow) * 32 + 16 * (kq & 1));
    const int sh = 4 * (kq >> 1);
#pragma unroll
    for (int i = 0; i < 4; i++) f[i] = (int)(((unsigned)f[i] >> sh) & 0x0F0F0F0Fu);
    return f;
  };
  constexpr int UB = KG == 4 ? 2 : 4;  // blocks whose uq fragments are requested together

#pragma unroll 1
  for (int blk0 = 0; blk0 < (MULTI ? a.NB : 1); blk0 += NBC) {
    const int nb = min(NBC, a.NB - blk0);
    const unsigned plane = (unsigned)nb * 1024u;  // code rows of one position
    // ---- phase T ----
    const int c0 = blk0 * 64;
    {
      // wave items: NCHW, CPL = 4: (block, four dwords); CPL = 1: (block, four dwords, byte);
      // NHWC, CPL = 4: (block, four dwords); CPL = 1: 16 channels of four tiles
      const int per_block = a.Q / 4;  // groups of four dwords: 4, or 1 with 16-byte rows
      const int nitems = LOAD == kNhwc1 ? nb * per_block : nb * per_block * (CPL == 4 ? 1 : 4);
      const int it0 = LOAD == kNhwc1 ? wave >> 2 : wave;
      constexpr int kStep = LOAD == kNhwc1 ? NW / 4 : NW;
      // first channel of step (it, q), for the lane's dl = 0
      auto chan = [&](int it, int q) -> int {
        if constexpr (LOAD == kNhwc1) return c0 + 16 * it;
        if constexpr (CPL == 4) return c0 + (it / per_block) * 64 + 4 * (it % per_block) + a.Q * q;
        return c0 + (it / (4 * per_block)) * 64 + 4 * ((it >> 2) % per_block) + a.Q * (it & 3);
      };
      float cur[A * A], nxt[A * A];
      if constexpr (LOAD != kNhwc4) {
        if (kPrefetch && it0 < nitems) load(min(chan(it0, 0), C - 1), cur);
      }
      if (blk0 == 0) constants();
      for (int it = it0; it < nitems; it += kStep) {
        unsigned codes[E];
        unsigned real;
        unsigned dst;
        if constexpr (LOAD == kNhwc4) {
          const int bb = it / per_block, dg = it % per_block;
          const int cb = c0 + bb * 64 + (4 * dg + dl) * 4;  // the lane's four channels
          v4f w[A * A];
          tl.load4(tg, min(cb, C - 4), w);
          auto one = [&](auto qc) {
            float b[A * A];
#pragma unroll
            for (int i = 0; i < A * A; i++) b[i] = w[i][decltype(qc)::value];
            quantize(b, qc, codes);
          };
          one(std::integral_constant<int, 0>{});
          one(std::integral_constant<int, 1>{});
          one(std::integral_constant<int, 2>{});
          one(std::integral_constant<int, 3>{});
          real = cb < C ? 0xFFFFFFFFu : 0u;
          dst = (unsigned)bb * 1024u + (unsigned)trow * 64u + (unsigned)((dg ^ swz(trow)) * 16 + 4 * dl);
        } else if constexpr (CPL == 4) {
          real = 0;
          auto step = [&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const int itn = q == 3 ? it + kStep : it;
            if constexpr (!kPrefetch) load(min(chan(it, q), C - 1), cur);
            else if (itn < nitems) load(min(chan(itn, (q + 1) & 3), C - 1), nxt);
            quantize(cur, qc, codes);
            if (chan(it, q) + dl < C) real |= 0xFFu << (8 * q);
            if constexpr (kPrefetch) {
#pragma unroll
              for (int i = 0; i < A * A; i++) cur[i] = nxt[i];
            }
          };
          step(std::integral_constant<int, 0>{});
          step(std::integral_constant<int, 1>{});
          step(std::integral_constant<int, 2>{});
          step(std::integral_constant<int, 3>{});
          const int bb = it / per_block, dg = it % per_block;
          dst = (unsigned)bb * 1024u + (unsigned)trow * 64u + (unsigned)((dg ^ swz(trow)) * 16 + 4 * dl);
        } else {
          if constexpr (!kPrefetch) load(min(chan(it, 0), C - 1), cur);
          else if (it + kStep < nitems) load(min(chan(it + kStep, 0), C - 1), nxt);
          quantize(cur, std::integral_constant<int, 0>{}, codes);
          real = chan(it, 0) + dl < C ? 0xFFu : 0u;
          if constexpr (kPrefetch) {
#pragma unroll
            for (int i = 0; i < A * A; i++) cur[i] = nxt[i];
          }
          if constexpr (LOAD == kNhwc1) {
            dst = (unsigned)(it / per_block) * 1024u + (unsigned)trow * 64u +
                  (unsigned)(((it % per_block) ^ swz(trow)) * 16 + dl);
          } else {
            const int bb = it / (4 * per_block), dg = (it >> 2) % per_block;
            dst = (unsigned)bb * 1024u + (unsigned)trow * 64u +
                  (unsigned)((dg ^ swz(trow)) * 16 + 4 * dl + (it & 3));
          }
        }
#pragma unroll
        for (int e = 0; e < E; e++) {
          const unsigned u = (codes[e] ^ flip) & real;
          if constexpr (CPL == 4) *reinterpret_cast<unsigned*>(ring + e * plane + dst) = u;
          else *reinterpret_cast<uint8_t*>(ring + e * plane + dst) = (uint8_t)u;
        }
      }
    }
    // ---- phase G ----
    if constexpr (!MULTI) clear_acc();
    v4i af[UB][KG];
    auto load_batch = [&](int e, int b0) {
#pragma unroll
      for (int u = 0; u < UB; u++)
#pragma unroll
        for (int kg = 0; kg < KG; kg++) af[u][kg] = load_uq(e, blk0 + min(b0 + u, nb - 1), kg);
    };
    load_batch(wave * PW, 0);
    __syncthreads();  // the codes of all waves are in LDS
#pragma unroll
    for (int w = 0; w < PW; w++) {
      const int e = wave * PW + w;
      for (int b0 = 0; b0 < nb; b0 += UB) {
        if (w > 0 || b0 > 0) load_batch(e, b0);
#pragma unroll
        for (int u = 0; u < UB; u++) {
          if (b0 + u < nb) {
            const v4i bf = *reinterpret_cast<const v4i*>(ring + (unsigned)e * plane + (unsigned)(b0 + u) * 1024u + f_off);
            v4i af0 = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
            if (a.uq_mode == 1 && kq > 0) af0 = v4i{0, 0, 0, 0};  // only 16 bytes of the row exist
            csum[w] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af0, bf, csum[w], 0, 0, 0);
#pragma unroll
            for (int kg = 0; kg < KG; kg++)
              acc[w][kg] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[u][kg], bf, acc[w][kg], 0, 0, 0);
          }
        }
      }
    }
    __syncthreads();  // the code rows are free again
  }

  // ---- M[e,k,p] to LDS ----
  const int h = 1 << (a.bits - 1);
#pragma unroll
  for (int w = 0; w < PW; w++) {
    const int e = wave * PW + w;
    const float sc = sc_s[e], gc = gc_s[e];
    const double rmul = rmul_s[e], kc = kc_s[e];
    const int cs = csum[w][0];  // every row of the ones operand gives the same sums
    const float g = gc * (float)(b8 ? cs : cs - h * C);
    const int bias = a.uq_mode == 2 ? 8 * cs : 0;
#pragma unroll
    for (int kg = 0; kg < KG; kg++) {
      float m[4];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int k = min(k0 + kg * 16 + 4 * kq + r, K - 1);
        const int rs = a.u_rowsum[(size_t)e * K + k];
        const int v = acc[w][kg][r] - bias - (b8 ? 0 : h * rs);
        m[r] = __builtin_fmaf(sc, (float)v, (float)(rmul * (double)rs + kc) + g);
      }
      float* dst = ex + (e * KG + kg) * 256;
      if constexpr (kNhwc) {
        *reinterpret_cast<v4f*>(dst + col * 16 + 4 * kq) = v4f{m[0], m[1], m[2], m[3]};
      } else {
#pragma unroll
        for (int r = 0; r < 4; r++) dst[r * 64 + kq * 16 + col] = m[r];
      }
    }
  }
  __syncthreads();
  // ---- A^T M A and the stores: one (filter, tile) pair per thread and turn ----
  for (int i = tid; i < KG * 256; i += NT) {
    const int kg = i >> 8, idx = i & 255;
    const int kin = kNhwc ? idx & 15 : 4 * ((idx >> 4) & 3) + (idx >> 6);
    const int pin = kNhwc ? idx >> 4 : idx & 15;
    const int k = k0 + kg * 16 + kin, p = p0 + pin;
    if (k >= K || p >= P) continue;
    float t[M][A], o[M][M];
#pragma unroll
    for (int j = 0; j < A; j++) {
      float v[A], s[M];
#pragma unroll
      for (int r = 0; r < A; r++) v[r] = ex[((r * A + j) * KG + kg) * 256 + idx];
      dev::out1d<M>(v, s);
#pragma unroll
      for (int r = 0; r < M; r++) t[r][j] = s[r];
    }
#pragma unroll
    for (int r = 0; r < M; r++) dev::out1d<M>(t[r], o[r]);
    const int ox0 = (p % a.tw) * M, q2 = p / a.tw;
    const int oy0 = (q2 % a.th) * M, on = q2 / a.th;
    if constexpr (kNhwc) {
      const unsigned base = (((unsigned)on * (unsigned)a.Ho + (unsigned)oy0) * (unsigned)a.Wo + (unsigned)ox0) *
                                (unsigned)K + (unsigned)k;
#pragma unroll
      for (int r = 0; r < M; r++)
#pragma unroll
        for (int s = 0; s < M; s++)
          store_b32(a.y, a.y_bytes, (oy0 + r < a.Ho && ox0 + s < a.Wo)
                                        ? (base + ((unsigned)r * (unsigned)a.Wo + (unsigned)s) * (unsigned)K) * 4u
                                        : kOobY, o[r][s]);
    } else {
      const unsigned base = (((unsigned)on * (unsigned)K + (unsigned)k) * (unsigned)a.Ho + (unsigned)oy0) *
                                (unsigned)a.Wo + (unsigned)ox0;
      const bool whole = ox0 + M <= a.Wo;
#pragma unroll
      for (int r = 0; r < M; r++) {
        const unsigned off = (base + (unsigned)r * (unsigned)a.Wo) * 4u;
        const bool row = oy0 + r < a.Ho;
        if (whole) {
          store_row<M>(a.y, a.y_bytes, row ? off : kOobY, o[r]);
        } else {
#pragma unroll
          for (int s = 0; s < M; s++)
            store_b32(a.y, a.y_bytes, row && ox0 + s < a.Wo ? off + 4u * s : kOobY, o[r][s]);
        }
      }
    }
  }
}

}  // namespace pos
}  // namespace lance

namespace lance {
namespace pos {

template <int M, int NW, int CPL, int KG, int LOAD, bool CLAMP, bool MULTI>
inline hipError_t launch_one(const CpArgs& a, unsigned grid, size_t lds, hipStream_t s) {
  auto kern = conv_fused_pos_kernel<M, NW, CPL, KG, LOAD, CLAMP, MULTI>;
  constexpr int kMost = kConstBytes + (KG > chunk_blocks<M>() ? KG : chunk_blocks<M>()) * (M + 2) * (M + 2) * 1024;
  const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), kMost);
  if (e != hipSuccess) return e;
  note_kernel("conv_fused_pos_kernel");
  kern<<<grid, NW * 64, lds, s>>>(a);
  return hipGetLastError();
}

template <int M, int NW, int CPL, int LOAD, bool CLAMP>
inline hipError_t launch_kg(const CpArgs& a, int kg, unsigned grid, size_t lds, hipStream_t s) {
  if constexpr (NW != 8 && (CPL == 4 || LOAD == kNhwc1))
    if (a.NB > chunk_blocks<M>()) return launch_one<M, NW, CPL, 1, LOAD, CLAMP, true>(a, grid, lds, s);
  switch (kg) {
    case 1: return launch_one<M, NW, CPL, 1, LOAD, CLAMP, false>(a, grid, lds, s);
    case 2: return launch_one<M, NW, CPL, 2, LOAD, CLAMP, false>(a, grid, lds, s);
    default: return launch_one<M, NW, CPL, 4, LOAD, CLAMP, false>(a, grid, lds, s);
  }
}

// load: kRowsEdge, kRowsAny, kNhwc1 or (m = 2) kNhwc4; kg: 1, 2 or 4 groups of 16 filters.
template <int M, int NW, bool CLAMP>
inline hipError_t launch(const CpArgs& a, int cpl, int load, int kg, hipStream_t s) {
  constexpr int E = (M + 2) * (M + 2);
  const unsigned grid = (unsigned)((a.P + 15) / 16) * (unsigned)a.nky;
  const int nb = a.NB < chunk_blocks<M>() ? a.NB : chunk_blocks<M>();
  const size_t lds = kConstBytes + (size_t)(nb > kg ? nb : kg) * E * 1024;
  switch (load) {
    case kRowsEdge:
      return cpl == 4 ? launch_kg<M, NW, 4, kRowsEdge, CLAMP>(a, kg, grid, lds, s)
                      : launch_kg<M, NW, 1, kRowsEdge, CLAMP>(a, kg, grid, lds, s);
    case kRowsAny:
      return cpl == 4 ? launch_kg<M, NW, 4, kRowsAny, CLAMP>(a, kg, grid, lds, s)
                      : launch_kg<M, NW, 1, kRowsAny, CLAMP>(a, kg, grid, lds, s);
    case kNhwc1: return launch_kg<M, NW, 1, kNhwc1, CLAMP>(a, kg, grid, lds, s);
    default:
      if constexpr (M == 2) return launch_kg<M, NW, 4, kNhwc4, CLAMP>(a, kg, grid, lds, s);
      return hipErrorInvalidValue;
  }
}

}  // namespace pos
}  // namespace lance
