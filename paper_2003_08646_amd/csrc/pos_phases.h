// The phases that the kernels for layers with few tiles are made of (conv_fused_pos.h,
// gemm_fused_pos.hip): Eq. 7 / Eq. 8 constants, transform + quantize of 16 tiles into LDS code rows,
// and the way from integer sums to stored patches.  Workgroups of NT = 64*NW threads.
//
// Code rows in LDS are [E][blocks][16 tiles][64 B], the 16-byte chunk c of row r at c ^ swz(r).  Codes
// narrower than 8 bits stay unsigned there (they are non-negative int8 values): the filter row sums
// take the difference off the integer sums.  So do the column sums for packed filter codes, which are
// multiplied as code + 8.  Both are exact.
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
  int8_t* vq;               // codes of V, where they pass through memory (gemm_fused_pos.hip)
  int count, per_tensor, is_static;
  int N, C, H, W, K, pad, P, th, tw, Ho, Wo, bits, bits_w;
  int NB, Q;     // channel blocks; dwords per code row (16, or 4 for layers of at most 16 channels)
  int uq_mode;   // 0: 64-byte rows, 1: 16-byte rows (at most 16 channels), 2: packed 32-byte rows
  int nky;       // filter splits of 16*KG filters
  unsigned x_bytes, y_bytes, vq_bytes;
};

constexpr unsigned kOobY = 0xFFFFFFF0u;

__device__ __forceinline__ int swz(int row) { return (row >> 2) & 3; }

__device__ __forceinline__ v4i load_code(const int8_t* uq, unsigned bytes, unsigned off, unsigned soff) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uq), 0, bytes, 0x00020000);
  return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}

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


// ---- Eq. 7 / Eq. 8 constants of a workgroup, in LDS ----
constexpr int kConstBytes = 2048;
template <int M>
struct Consts {
  static constexpr int E = (M + 2) * (M + 2);
  float* qp;     // [E][2] = {min, inv} of Eq. 7
  float* sc;     // [E] su*sv
  float* gc;     // [E] sv*ou
  double* rmul;  // [E] su*ov
  double* kc;    // [E] C*ou*ov
  static_assert(E * (4 * sizeof(float) + 2 * sizeof(double)) <= kConstBytes, "parameter tables");

  __device__ __forceinline__ explicit Consts(char* smem) {
    qp = reinterpret_cast<float*>(smem);
    sc = qp + 2 * E;
    gc = sc + E;
    rmul = reinterpret_cast<double*>(gc + E);
    kc = rmul + E;
  }

  // What the constants are formed from, requested before the first pixels: loads return in order, and
  // behind the pixels these few bytes from L2 would wait for memory.
  template <int NT>
  struct Early {
    static constexpr int kCols = 2 * E, kGroups = NT / kCols, kBatch = 8;
    float umin, umax, vmin, vmax;  // threads below E: filter range, caller's input range of position tid
    float rec[kBatch];   // column tid % kCols of the records tid / kCols, + kGroups, ...

    __device__ __forceinline__ Early(const CpArgs& a, int is_static, int tid) {
      const int e = min(tid, E - 1), col = tid % kCols;
      umin = a.u_range[2 * e];
      umax = a.u_range[2 * e + 1];
      const float* given = is_static ? a.v_range : a.u_range;  // (dynamic ranges: overwritten in form())
      vmin = given[2 * e];
      vmax = given[2 * e + 1];
      if (!is_static) {
#pragma unroll
        for (int u = 0; u < kBatch; u++) {  // (past the last record: the last one again, or none of the batch)
          rec[u] = col & 1 ? -INFINITY : INFINITY;
          if (u * kGroups < a.count)
            rec[u] = a.partial[(size_t)min(tid / kCols + u * kGroups, a.count - 1) * kCols + col];
        }
      }
    }
  };

  // From v_range (is_static) or the records of the range pass; then workgroup 0 writes v_range.
  // red: NT floats of LDS that nobody else touches until this returns.  All threads; ends in a barrier.
  template <int NT>
  __device__ __forceinline__ void form(const CpArgs& a, int is_static, Early<NT>& early, float* red, int tid) const {
    if (!is_static) {
      constexpr int kCols = Early<NT>::kCols, kGroups = Early<NT>::kGroups, kBatch = Early<NT>::kBatch;
      const int col = tid % kCols, grp = tid / kCols;
      const bool is_max = col & 1;
      float v = early.rec[0];
#pragma unroll
      for (int u = 1; u < kBatch; u++) v = is_max ? fmaxf(v, early.rec[u]) : fminf(v, early.rec[u]);
      for (int row0 = grp + kBatch * kGroups; row0 < a.count; row0 += kBatch * kGroups) {
        float xv[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; u++) xv[u] = a.partial[(size_t)min(row0 + u * kGroups, a.count - 1) * kCols + col];
#pragma unroll
        for (int u = 0; u < kBatch; u++) v = is_max ? fmaxf(v, xv[u]) : fminf(v, xv[u]);
      }
      red[tid] = v;
      dev::lds_barrier();
      if (tid < E) {
        v2f r = *reinterpret_cast<const v2f*>(red + 2 * tid);
#pragma unroll
        for (int g2 = 1; g2 < kGroups; g2++) {
          const v2f y = *reinterpret_cast<const v2f*>(red + g2 * kCols + 2 * tid);
          r[0] = fminf(r[0], y[0]);
          r[1] = fmaxf(r[1], y[1]);
        }
        early.vmin = r[0];
        early.vmax = r[1];
      }
    }
    if (tid < E) {
      float lo = early.vmin, hi = early.vmax;
      if (!is_static) {
        if (a.per_tensor) {  // (all E threads are in one wave)
          for (int e = 0; e < E; e++) {
            lo = fminf(lo, __shfl(early.vmin, e, 64));
            hi = fmaxf(hi, __shfl(early.vmax, e, 64));
          }
        }
        if (blockIdx.x == 0) {
          a.v_range[2 * tid] = lo;
          a.v_range[2 * tid + 1] = hi;
        }
      }
      float iu, su, inv, sv;
      dev::quant_params(early.umin, early.umax, a.bits_w, &iu, &su);
      dev::quant_params(lo, hi, a.bits, &inv, &sv);
      const double ou = (double)early.umin + (double)su * (double)(1 << (a.bits_w - 1));
      const double ov = (double)lo + (double)sv * (double)(1 << (a.bits - 1));
      qp[2 * tid] = lo;
      qp[2 * tid + 1] = inv;
      sc[tid] = (float)((double)su * (double)sv);
      gc[tid] = (float)((double)sv * ou);
      rmul[tid] = (double)su * ov;
      kc[tid] = (double)a.C * ou * ov;
    }
    dev::lds_barrier();
  }
};

// ---- phase T: transform + quantize of the tiles p0 .. p0+15 ----
// NCHW: a wave takes 16 tiles x 4 dwords at a time, CPL = 4: all four channels of a dword per lane,
// CPL = 1: one of them (so that few blocks still give every wave something to do).  NHWC: 16-byte
// loads of a dword's channels (CPL = 4), or 4 tiles x 16 channels (CPL = 1).
template <int M, int NW, int CPL, int LOAD, bool CLAMP>
struct Quantizer {
  static constexpr int A = M + 2, E = A * A;
  const CpArgs& a;
  TileGeo tg;
  TileLoader<M, LOAD> tl;
  int wave, trow, dl;

  __device__ __forceinline__ Quantizer(const CpArgs& args, int p0, int lane, int wave_) : a(args), wave(wave_) {
    trow = LOAD == kNhwc4 ? lane >> 2 : (LOAD == kNhwc1 ? 4 * (wave & 3) + (lane >> 4) : lane & 15);
    dl = LOAD == kNhwc4 ? lane & 3 : (LOAD == kNhwc1 ? lane & 15 : lane >> 4);
    tg = TileGeo{a.x, a.x_bytes, a.N, a.C, a.H, a.W, a.pad, a.P, a.th, a.tw};
    tl.setup(tg, min(p0 + trow, a.P - 1), dl);
  }

  // byte q of the dwords codes[e] from the patch b
  template <int q>
  __device__ __forceinline__ void one(const float (&b)[A * A], const float* qp, unsigned (&codes)[E]) const {
    // (F(4x4): the parameters are read again for every channel instead of living in 72 registers)
    if constexpr (M == 4) asm volatile("" ::: "memory");
    float d[A][A];
    tl.mask(b, d);
    dev::input_tile_transform<M>(d);
    const float L = (float)((1 << a.bits) - 1);
#pragma unroll
    for (int e = 0; e < E; e++) {
      const v2f mi = *reinterpret_cast<const v2f*>(qp + 2 * e);
      float t = (d[e / A][e % A] - mi[0]) * mi[1];
      if constexpr (CLAMP) t = fminf(t, L);  // above 8 bits' range the conversion saturates by itself
      codes[e] = __builtin_amdgcn_cvt_pk_u8_f32(t, q, q == 0 ? 0u : codes[e]);
    }
    // ties this channel's arithmetic to its step (left alone, the compiler moves all channels'
    // arithmetic behind the last load)
#pragma unroll
    for (int e = 0; e < E; e++) asm volatile("" : "+v"(codes[e]));
  }

  // Blocks blk0 .. blk0+nb-1 into ring (planes of nb KB per position).  mid(): run by all threads after
  // the first pixels have been requested; qp is valid after it.
  template <class Mid>
  __device__ __forceinline__ void run(int blk0, int nb, const float* qp, char* ring, Mid&& mid) const {
    const int C = a.C, c0 = blk0 * 64;
    const unsigned plane = (unsigned)nb * 1024u;
    const unsigned flip = a.bits == 8 ? 0x80808080u : 0u;  // 8-bit codes are stored signed
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
    float px[2][A * A];
    if constexpr (LOAD != kNhwc4) {
      if (it0 < nitems) tl.load(tg, min(chan(it0, 0), C - 1), px[0]);
    }
    mid();
    for (int it = it0; it < nitems; it += kStep) {
      unsigned codes[E];
      unsigned real;
      unsigned dst;
      if constexpr (LOAD == kNhwc4) {
        const int bb = it / per_block, dg = it % per_block;
        const int cb = c0 + bb * 64 + (4 * dg + dl) * 4;  // the lane's four channels
        v4f w[A * A];
        tl.load4(tg, min(cb, C - 4), w);
        auto chan4 = [&](auto qc) {
          float b[A * A];
#pragma unroll
          for (int i = 0; i < A * A; i++) b[i] = w[i][decltype(qc)::value];
          one<decltype(qc)::value>(b, qp, codes);
        };
        chan4(std::integral_constant<int, 0>{});
        chan4(std::integral_constant<int, 1>{});
        chan4(std::integral_constant<int, 2>{});
        chan4(std::integral_constant<int, 3>{});
        real = cb < C ? 0xFFFFFFFFu : 0u;
        dst = (unsigned)bb * 1024u + (unsigned)trow * 64u + (unsigned)((dg ^ swz(trow)) * 16 + 4 * dl);
      } else if constexpr (CPL == 4) {
        real = 0;
        auto step = [&](auto qc) {
          constexpr int q = decltype(qc)::value;
          const int itn = q == 3 ? it + kStep : it;
          constexpr int now = M == 2 ? q & 1 : 0;  // (alternating buffers spill in F(4x4))
          if (itn < nitems) tl.load(tg, min(chan(itn, (q + 1) & 3), C - 1), px[now ^ 1]);
          one<q>(px[now], qp, codes);
          if (chan(it, q) + dl < C) real |= 0xFFu << (8 * q);
          if constexpr (M == 4) {
#pragma unroll
            for (int i = 0; i < A * A; i++) px[0][i] = px[1][i];
          }
        };
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
        const int bb = it / per_block, dg = it % per_block;
        dst = (unsigned)bb * 1024u + (unsigned)trow * 64u + (unsigned)((dg ^ swz(trow)) * 16 + 4 * dl);
      } else {
        if (it + kStep < nitems) tl.load(tg, min(chan(it + kStep, 0), C - 1), px[1]);
        one<0>(px[0], qp, codes);
        real = chan(it, 0) + dl < C ? 0xFFu : 0u;
#pragma unroll
        for (int i = 0; i < A * A; i++) px[0][i] = px[1][i];
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
};

// ---- filter codes ----
// uq fragments: the lane's byte offset inside a block's rows per group of 16 filters (16-byte rows: only
// the first lane group has bytes, the others read zero from beyond the buffer), the block's offset as
// the scalar offset.
template <int M, int KG>
struct UqReader {
  const int8_t* uq;
  unsigned off[KG], bytes, block;  // block: bytes of one (position, channel block)
  int NB, mode, kq;

  __device__ __forceinline__ UqReader(const CpArgs& a, int k0, int col, int kq_) {
    constexpr unsigned E = (M + 2) * (M + 2);
    uq = a.uq; NB = a.NB; mode = a.uq_mode; kq = kq_;
    const unsigned row = mode == 0 ? 64u : (mode == 1 ? 16u : 32u);
    block = (unsigned)a.K * row;
    bytes = E * (unsigned)a.NB * block;
#pragma unroll
    for (int kg = 0; kg < KG; kg++) {
      const unsigned krow = (unsigned)min(k0 + kg * 16 + col, a.K - 1);
      off[kg] = mode == 0 ? krow * 64u + 16u * kq
                          : (mode == 1 ? (kq == 0 ? krow * 16u : kOobY) : krow * 32u + 16u * (kq & 1));
    }
  }
  __device__ __forceinline__ v4i load(int e, int b, int kg) const {
    return load_code(uq, bytes, off[kg], ((unsigned)e * (unsigned)NB + (unsigned)b) * block);
  }
  // The fragment as matrix operand.  Packed rows: byte q of the 64-byte row is the low nibble of byte q
  // (q < 32) or the high one of byte q - 32, as code + 8.
  __device__ __forceinline__ v4i codes(v4i f) const {
    if (mode == 2) {
      const int sh = 4 * (kq >> 1);
#pragma unroll
      for (int i = 0; i < 4; i++) f[i] = (int)(((unsigned)f[i] >> sh) & 0x0F0F0F0Fu);
    }
    return f;
  }
  // Ones for the column sums; with 16-byte rows only where the row has bytes.
  __device__ __forceinline__ v4i ones() const {
    const int o = (mode == 1 && kq > 0) ? 0 : 0x01010101;
    return v4i{o, o, o, o};
  }
};

// Row sum at position e of filter k0 + lane (of the 16*KG; the lanes beyond hold the same ones again).
template <int KG>
__device__ __forceinline__ int load_rowsum(const CpArgs& a, int e, int k0, int lane) {
  return a.u_rowsum[(size_t)e * a.K + min(k0 + lane % (16 * KG), a.K - 1)];
}

// ---- from integer sums to patches ----
// Sums of positions e of a wave -> M[e,k,p] (Eq. 8, expanded) in LDS: ex[(e*KG + kg)*TG + t][256], NCHW
// as [r][kq][col], NHWC as [col][4*kq + r] (filter 4*kq + r of group kg, tile col of group t).
// acc/csum: accumulator registers of v_mfma_i32_16x16x64_i8 with uq and with ones as first operand.
// rs: load_rowsum().  The filter-side term su*ov*rs + C*ou*ov is formed once per filter, by the lane that holds
// the row sum, and handed to the 16 lanes that use it through the words of ex that the wave is about to
// write (one image 3 -> 64 224x224, 8 waves, four groups of filters: this step took 2.4 us of each workgroup's 7.4 with
// the binary64 term formed in every lane, and waited for 32 loads of row sums).
template <int KG, int TG, bool NHWC, class C>
__device__ __forceinline__ void sums_to_lds(const CpArgs& a, const C& cst, int e, int lane, int rs,
                                            const v4i (&acc)[TG][KG], const v4i (&csum)[TG], float* ex) {
  const int col = lane & 15, kq = lane >> 4;
  const bool b8 = a.bits == 8;
  const int h = 1 << (a.bits - 1);
  const float sc = cst.sc[e], gc = cst.gc[e];
  float* own = ex + e * (KG * TG * 256);
  own[lane] = (float)(cst.rmul[e] * (double)rs + cst.kc[e]);
  if (!b8) reinterpret_cast<int*>(own)[64 + lane] = h * rs;
  asm volatile("" ::: "memory");  // (a wave's LDS operations complete in order)
  v4f f[KG];
  v4i hr[KG];
#pragma unroll
  for (int kg = 0; kg < KG; kg++) {
    f[kg] = *reinterpret_cast<const v4f*>(own + 16 * kg + 4 * kq);
    hr[kg] = v4i{0, 0, 0, 0};
    if (!b8) hr[kg] = *reinterpret_cast<const v4i*>(own + 64 + 16 * kg + 4 * kq);
  }
  asm volatile("" ::: "memory");
#pragma unroll
  for (int t = 0; t < TG; t++) {
    const int cs = csum[t][0];  // every row of the ones operand gives the same sums
    const float g = gc * (float)(b8 ? cs : cs - h * a.C);
    const int bias = a.uq_mode == 2 ? 8 * cs : 0;
#pragma unroll
    for (int kg = 0; kg < KG; kg++) {
      float m[4];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int v = acc[t][kg][r] - bias - hr[kg][r];
        m[r] = __builtin_fmaf(sc, (float)v, f[kg][r] + g);
      }
      float* dst = ex + ((e * KG + kg) * TG + t) * 256;
      if constexpr (NHWC) {
        *reinterpret_cast<v4f*>(dst + col * 16 + 4 * kq) = v4f{m[0], m[1], m[2], m[3]};
      } else {
#pragma unroll
        for (int r = 0; r < 4; r++) dst[r * 64 + kq * 16 + col] = m[r];
      }
    }
  }
}

// A^T M A and the stores: one (filter, tile) pair per thread and turn.
template <int M, int KG, int TG, int NT, bool NHWC>
__device__ __forceinline__ void store_patches(const CpArgs& a, const float* ex, int k0, int p0, int tid) {
  constexpr int A = M + 2;
  const int K = a.K, P = a.P;
  for (int i = tid; i < KG * TG * 256; i += NT) {
    const int idx = i & 255, kt = i >> 8;
    const int kg = kt / TG, t = kt % TG;
    const int kin = NHWC ? idx & 15 : 4 * ((idx >> 4) & 3) + (idx >> 6);
    const int pin = NHWC ? idx >> 4 : idx & 15;
    const int k = k0 + kg * 16 + kin, p = p0 + t * 16 + pin;
    if (k >= K || p >= P) continue;
    float w[M][A], o[M][M];
#pragma unroll
    for (int j = 0; j < A; j++) {
      float v[A], s[M];
#pragma unroll
      for (int r = 0; r < A; r++) v[r] = ex[(r * A + j) * (KG * TG * 256) + i];
      dev::out1d<M>(v, s);
#pragma unroll
      for (int r = 0; r < M; r++) w[r][j] = s[r];
    }
#pragma unroll
    for (int r = 0; r < M; r++) dev::out1d<M>(w[r], o[r]);
    const int ox0 = (p % a.tw) * M, q2 = p / a.tw;
    const int oy0 = (q2 % a.th) * M, on = q2 / a.th;
    if constexpr (NHWC) {
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
