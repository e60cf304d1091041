// Weight-only quantization (Sec. 4, the 4-32 row of Table 2): filters quantized in the Winograd
// domain (Eq. 7, prepared by the filter transform), inputs transformed but not quantized:
//   M[e,k,p] = sum_c Q'(u^[e,k,c]) * (B^T d_{p,c} B)[e],   S = A^T M A          (Eq. 8, Eq. 9)
//
// The channel sum runs on the bf16 matrix cores without giving up binary32: a filter code is an
// integer of at most 8 bits and exact in bf16, and a binary32 value is the exact sum of three bf16
// values (its top 8 significant bits, the next 8, the rest), so three products per value pair, each
// exact, are added up in binary32; Q' is applied to the sums:
//   M = step_e * sum_c (code * 2^(8-b) - z_e) * V + ou_e * sum_c V,   step = scale / 2^(8-b),
//   ou = min + step * z,
// the second sum from the same instructions with an operand of ones.  z is the multiple of step next
// to zero (0 .. (2^b - 1) * 2^(8-b); the difference is an integer of at most 255, still exact): counted
// from there ou is at most half of 1/255 of the range wherever that holds zero, so the two terms do not
// cancel, however far the range is from symmetric and however few the codes.  V enters the split times 2^24 (the results
// leave it again): the smallest binary32 value's pieces are then normal bf16 numbers, so the split is
// exact for every V below 2^104; what overflows is formed again in the plain form (plain_results).
//
// weight_only_mfma_kernel: a workgroup of 16 waves (m = 4: 12) takes 16*TG tiles x 16*KG filters,
// wave w the positions w*E/NW ..  Turn by turn over CH channels: every lane transforms one channel
// of one tile and writes its three pieces to LDS (rows of 32 values, [E][3][CH/32][TG][16 rows]); the
// waves multiply.  Then as in conv_fused_pos.h: M to LDS, A^T M A and the stores by (filter, tile)
// pairs.  uq codes become bf16 in registers, two values per v_perm_b32.
//
// What bounds it: the vector ALUs (transform, three-way split, conversion of the codes) and, on small
// layers, the chain of steps of a workgroup.  N32 64->64 32x32: 101 us on the vector-ALU kernel, 13.6
// us now; N2 249->21 53x38: 407 -> 14.8 us; N2 16->64 106x106 F(4x4): 87 -> 10 us.  Relative error
// against binary64, vector-ALU kernel and this one: 64 channels 2.6e-7 and 1.2e-7; 512 channels 6.2e-7
// and 3.3e-7, with one filter ten times the others and of one sign (the others' error) 1.6e-6 and
// 3.4e-7, with one outlying weight 9.1e-6 and 3.3e-7, 4-bit codes 6.4e-7 and 3.2e-7; F(4x4), 512
// channels, 3.9e-6 and 2.0e-6.
//
// weight_only_kernel: the vector-ALU form (lane = tile, E multiply-adds per channel and filter), for
// layers of few channels and filters (vector_form_faster), whose rows of 32 channels and groups of 16
// filters would be mostly padding in the other, and for inputs of 2 GiB and more, beyond the 32-bit row
// offsets of the other.
#include "lance_device.h"
#include "lance_internal.h"
#include "pos_phases.h"

namespace lance {
namespace {

constexpr int kThreads = 256;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
using pos::kOobY;
using pos::v2u;
using pos::v4f;
using pos::v4u;

struct WmArgs {
  const float* x;
  const int8_t* uq;
  const float* u_range;
  float* y;
  int N, C, H, W, K, pad, P, th, tw, Ho, Wo, bits_w, NB, cb16, nky;
  unsigned x_bytes, y_bytes;
};

constexpr float kUp = 16777216.0f;  // 2^24

// Eight stored codes (two dwords of a code row) as multiples of step counted from z, in bf16;
// exact.  unit: 2^(8-b); zero: z + (128 - 2^(b-1)) * unit.
__device__ __forceinline__ bf16x8 codes_to_bf16(v2u c, float unit, float zero) {
  v4u r;
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const unsigned u = c[i] ^ 0x80808080u;  // stored code + 128
    float f[4];
    f[0] = __builtin_fmaf((float)(u & 0xFFu), unit, -zero);
    f[1] = __builtin_fmaf((float)((u >> 8) & 0xFFu), unit, -zero);
    f[2] = __builtin_fmaf((float)((u >> 16) & 0xFFu), unit, -zero);
    f[3] = __builtin_fmaf((float)(u >> 24), unit, -zero);
    // the upper halves of two binary32 values side by side
    r[2 * i] = __builtin_amdgcn_perm(__float_as_uint(f[1]), __float_as_uint(f[0]), 0x07060302u);
    r[2 * i + 1] = __builtin_amdgcn_perm(__float_as_uint(f[3]), __float_as_uint(f[2]), 0x07060302u);
  }
  return __builtin_bit_cast(bf16x8, r);
}

// o = A^T v A
template <int M>
__device__ __forceinline__ void out2d(const float (&v)[M + 2][M + 2], float (&o)[M][M]) {
  constexpr int A = M + 2;
  float tt[M][A];
#pragma unroll
  for (int jj = 0; jj < A; jj++) {
    float col[A], s[M];
#pragma unroll
    for (int r = 0; r < A; r++) col[r] = v[r][jj];
    dev::out1d<M>(col, s);
#pragma unroll
    for (int r = 0; r < M; r++) tt[r][jj] = s[r];
  }
#pragma unroll
  for (int r = 0; r < M; r++) dev::out1d<M>(tt[r], o[r]);
}

// The (filter, tile) pair that thread tid takes in turn t: filter kin and tile pin of the workgroup's.
template <int M, int TG, int KG, bool NHWC>
struct Pairs {
  static constexpr int NT = M == 2 ? 1024 : 768, kPairs = KG * TG * 256, kTurns = (kPairs + NT - 1) / NT;
  int i, kin, pin;
  __device__ __forceinline__ Pairs(int tid, int t) : i(tid + t * NT) {
    const int idx = i & 255, kt = i >> 8;
    kin = kt / TG * 16 + (NHWC ? idx & 15 : 4 * ((idx >> 4) & 3) + (idx >> 6));
    pin = kt % TG * 16 + (NHWC ? idx >> 4 : idx & 15);
  }
  __device__ __forceinline__ bool exists() const { return kPairs % NT == 0 || i < kPairs; }
};

// The workgroup's products in the plain form (binary32 on the vector ALUs, channel by channel), o of the
// bad pairs from them.  The split into three pieces has none for an infinite value (inf - inf), and its
// sums overflow before these do (2^24 and the codes against scaled codes): results that are not finite
// are formed again here.  kC channels of all tiles and filters at a time go through buf; what bounds it is
// the reads of these rows from LDS (twelve 16-byte ones per channel for two pairs).  All threads; buf is
// free before and after.  N32 64->64 32x32 with one infinite value 112 us (312 with one thread per pair
// reading its own codes and pixels, 100 on the vector-ALU kernel; 13.5 without it), with nothing else
// 115 (394, 99); N4 512->512 14x14 420 (1035, 753).
template <int M, int TG, int KG, bool NHWC>
__device__ __forceinline__ void plain_results(const WmArgs& a, const float* sc_s, int k0, int p0, int tid, float* buf,
                                           const bool (&bad)[Pairs<M, TG, KG, NHWC>::kTurns],
                                           float (&o)[Pairs<M, TG, KG, NHWC>::kTurns][M][M]) {
  using P = Pairs<M, TG, KG, NHWC>;
  constexpr int A = M + 2, E = A * A, NT = P::NT, kC = 12, kTiles = 16 * TG, kFilters = 16 * KG;
  constexpr int kRow = M == 2 ? 20 : 36;  // floats: the 16-byte pieces of 16 rows lie in different banks
  float* vs = buf;                       // [kC][kTiles][kRow]
  float* us = vs + kC * kTiles * kRow;   // [kC][kFilters][kRow]
  static_assert(kC * (kTiles + kFilters) * kRow * sizeof(float) <= (size_t)E * 3 * (M == 2 ? 2 : 1) * 1024, "LDS");
  const int lc = a.cb16 ? 4 : 6, h = 1 << (a.bits_w - 1);  // channels of a block: 2^lc
  float acc[P::kTurns][E];
#pragma unroll
  for (int t = 0; t < P::kTurns; t++)
#pragma unroll
    for (int e = 0; e < E; e++) acc[t][e] = 0.0f;
  for (int c0 = 0; c0 < a.C; c0 += kC) {
    const int nc = min(kC, a.C - c0);
    __syncthreads();
    for (int i = tid; i < nc * kTiles; i += NT) {
      const int c = c0 + i / kTiles, p = min(p0 + i % kTiles, a.P - 1);
      const int y0 = (p / a.tw) % a.th * M - a.pad, x0 = p % a.tw * M - a.pad, n = p / a.tw / a.th;
      float d[A][A];
#pragma unroll
      for (int r = 0; r < A; r++)
#pragma unroll
        for (int s = 0; s < A; s++) {
          const int gy = y0 + r, gx = x0 + s;
          const bool ok = gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
          const float v = a.x[dev::act_index(NHWC, n, c, min(max(gy, 0), a.H - 1),
                                             min(max(gx, 0), a.W - 1), a.C, a.H, a.W)];
          d[r][s] = ok ? v : 0.0f;
        }
      dev::input_tile_transform<M>(d);
#pragma unroll
      for (int e = 0; e < E; e++) vs[i * kRow + e] = d[e / A][e % A];
    }
#pragma unroll 2
    for (int i = tid; i < nc * kFilters * E; i += NT) {
      const int e = i % E, kc = i / E;
      const int c = c0 + kc / kFilters, k = min(k0 + kc % kFilters, a.K - 1);
      const int b = c >> lc, r = c & ((1 << lc) - 1), lq = lc - 2;
      const int at = NHWC ? r : 4 * (r & ((1 << lq) - 1)) + (r >> lq);
      const int code = (int)a.uq[((((size_t)e * a.NB + b) * a.K + k) << lc) + at] + h;
      us[kc * kRow + e] = (float)code * sc_s[e] + a.u_range[2 * e];
    }
    __syncthreads();
    static_assert(P::kTurns == 1 || (P::kPairs % NT == 0 && NT % (256 * TG) == 0), "one tile per thread, whatever the turn");
    for (int c = 0; c < nc && P(tid, 0).exists(); c++) {
      const float* v = vs + (c * kTiles + P(tid, 0).pin) * kRow;
#pragma unroll
      for (int t = 0; t < P::kTurns; t++) {
        const float* u = us + (c * kFilters + P(tid, t).kin) * kRow;
#pragma unroll
        for (int e = 0; e < E; e++) acc[t][e] = __builtin_fmaf(u[e], v[e], acc[t][e]);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < P::kTurns; t++)
    if (bad[t]) {
      float mm[A][A];
#pragma unroll
      for (int e = 0; e < E; e++) mm[e / A][e % A] = acc[t][e];
      out2d<M>(mm, o[t]);
    }
}

template <int M, int TG, int KG, int LOAD>
__global__ __launch_bounds__(M == 2 ? 1024 : 768) void weight_only_mfma_kernel(const WmArgs a) {
  constexpr int A = M + 2, E = A * A, NW = M == 2 ? 16 : 12, NT = NW * 64, PW = E / NW;
  constexpr bool kNhwc = LOAD == pos::kNhwc1;
  constexpr int NH = M == 2 ? 2 / TG : 1;  // rows of 32 values per turn: CH = 32 * NH channels
  static_assert(M == 2 || TG == 1, "LDS");
  extern __shared__ char smem[];
  float* sc_s = reinterpret_cast<float*>(smem);  // [E] scale
  float* ou_s = sc_s + E;                        // [E] min + step * z
  float* zero_s = ou_s + E;                      // [E] z + (128 - 2^(b-1)) * unit
  int* huge_s = reinterpret_cast<int*>(zero_s + E);  // some M might overflow on its way to an output
  const float unit = (float)(1 << (8 - a.bits_w));
  static_assert((3 * E + 1) * sizeof(float) <= 512, "parameters");
  char* ring = smem + 512;                       // [E][3][NH][TG][16 rows][64 B]
  float* ex = reinterpret_cast<float*>(ring);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ky = blockIdx.x % a.nky, p0 = (blockIdx.x / a.nky) * 16 * TG, k0 = ky * 16 * KG;
  const int K = a.K, P = a.P, C = a.C;

  // The wave's part of a turn, the same in every turn: NCHW: 16 tiles, the dwords 4g .. 4g+3 of row
  // nh, byte q of each (the lane's channel is dl = lane / 16 dwords up); NHWC: 4 tiles, 16 channels.
  const int item = kNhwc ? wave >> 2 : wave;
  constexpr int kPerRow = kNhwc ? 2 : 8;
  const bool has_item = item < kPerRow * NH * TG;
  const int sub = item % kPerRow, nh = (item / kPerRow) % NH, tgi = (item / kPerRow / NH) % TG;
  const int trow = kNhwc ? 4 * (wave & 3) + (lane >> 4) : lane & 15;
  const int dl = kNhwc ? lane & 15 : lane >> 4;
  const int g = sub >> 2, q = sub & 3;
  const pos::TileGeo tg{a.x, a.x_bytes, a.N, C, a.H, a.W, a.pad, P, a.th, a.tw};
  pos::TileLoader<M, LOAD> tl;
  tl.setup(tg, min(p0 + 16 * tgi + trow, P - 1), dl);
  // row of 32 values number r of the channel axis: half r & 1 of channel block r / 2
  const int rows = a.cb16 ? 1 : 2 * a.NB;
  // channel of the lane with dl = 0; >= C: no such channel (with 16-byte code rows the positions
  // beyond the 16th stand for no channel)
  auto chan = [&](int r) -> int {
    if (a.cb16) return kNhwc ? (sub == 0 ? 0 : C) : (g == 0 ? 4 * q : C);
    return kNhwc ? r * 32 + 16 * sub : (r >> 1) * 64 + 8 * (r & 1) + 4 * g + 16 * q;
  };
  const int j = kNhwc ? 16 * sub + dl : 4 * (4 * g + dl) + q;  // the lane's value in its row
  const unsigned dst = (unsigned)((nh * TG + tgi) * 1024 + trow * 64 + (((j >> 3) ^ ((trow >> 2) & 3)) * 16) + (j & 7) * 2);
  constexpr unsigned kPiece = NH * TG * 1024u;

  float cur[A * A];
  auto request = [&](int r0) {
    if (has_item && r0 + nh < rows) tl.load(tg, min(chan(r0 + nh), C - 1), cur);
  };
  request(0);
  if (tid < E) {
    const float mn = a.u_range[2 * tid], mx = a.u_range[2 * tid + 1];
    float inv, scale;
    dev::quant_params(mn, mx, a.bits_w, &inv, &scale);
    const double step = (double)scale / unit, most = (double)((1 << a.bits_w) - 1) * unit;
    const double z = scale > 0.0f ? fmin(fmax(rint(-(double)mn / step), 0.0), most) : 0.0;
    sc_s[tid] = scale;
    ou_s[tid] = (float)((double)mn + step * z);
    zero_s[tid] = (float)z + (float)(128 - (1 << (a.bits_w - 1))) * unit;
  }
  if (tid == 0) *huge_s = 0;

  const int col = lane & 15, kq = lane >> 4;
  const unsigned f_off = (unsigned)(col * 64 + ((kq ^ ((col >> 2) & 3)) * 16));
  v4f acc[PW][TG][KG], vsum[PW][TG];
#pragma unroll
  for (int w = 0; w < PW; w++)
#pragma unroll
    for (int t = 0; t < TG; t++) {
      vsum[w][t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kg = 0; kg < KG; kg++) acc[w][t][kg] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    }
  const v4u ones_u = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_u);

  float zero[PW];
  for (int r0 = 0; r0 < rows; r0 += NH) {
    const int nrow = min(NH, rows - r0);
    if (has_item && nh < nrow) {
      float d[A][A];
      tl.mask(cur, d);
      if (chan(r0 + nh) + dl >= C) {
#pragma unroll
        for (int e = 0; e < E; e++) d[e / A][e % A] = 0.0f;
      }
      dev::input_tile_transform<M>(d);
#pragma unroll
      for (int e = 0; e < E; e++) {
        const float v = d[e / A][e % A] * kUp;
        const unsigned hi = __float_as_uint(v) & 0xFFFF0000u;
        const float r1 = v - __uint_as_float(hi);
        const unsigned mid = __float_as_uint(r1) & 0xFFFF0000u;
        const float r2 = r1 - __uint_as_float(mid);
        char* at = ring + (unsigned)(e * 3) * kPiece + dst;
        *reinterpret_cast<uint16_t*>(at) = (uint16_t)(hi >> 16);
        *reinterpret_cast<uint16_t*>(at + kPiece) = (uint16_t)(mid >> 16);
        *reinterpret_cast<uint16_t*>(at + 2 * kPiece) = (uint16_t)(__float_as_uint(r2) >> 16);
      }
    }
    request(r0 + NH);  // in flight under the products
    v2u code[PW][NH][KG];
#pragma unroll
    for (int w = 0; w < PW; w++)
#pragma unroll
      for (int r = 0; r < NH; r++)
#pragma unroll
        for (int kg = 0; kg < KG; kg++) {
          const int e = wave * PW + w, krow = min(k0 + kg * 16 + col, K - 1);
          const int rr = min(r0 + r, rows - 1);
          const int8_t* src = a.cb16 ? a.uq + ((size_t)e * K + krow) * 16 + 8 * (kq & 1)
                                     : a.uq + (((size_t)e * a.NB + (rr >> 1)) * K + krow) * 64 + 32 * (rr & 1) + 8 * kq;
          code[w][r][kg] = *reinterpret_cast<const v2u*>(src);
          if (a.cb16 && kq > 1) code[w][r][kg] = v2u{0u, 0u};
        }
    __syncthreads();
    if (r0 == 0) {
#pragma unroll
      for (int w = 0; w < PW; w++) zero[w] = zero_s[wave * PW + w];
    }
#pragma unroll
    for (int w = 0; w < PW; w++)
#pragma unroll
      for (int r = 0; r < NH; r++) {
        if (r < nrow) {
          bf16x8 af[KG];
#pragma unroll
          for (int kg = 0; kg < KG; kg++) af[kg] = codes_to_bf16(code[w][r][kg], unit, zero[w]);
#pragma unroll
          for (int t = 0; t < TG; t++)
#pragma unroll
            for (int pc = 2; pc >= 0; pc--) {  // the small pieces first
              const char* bp = ring + (unsigned)((wave * PW + w) * 3 + pc) * kPiece + (unsigned)((r * TG + t) * 1024) + f_off;
              const bf16x8 bf = *reinterpret_cast<const bf16x8*>(bp);
              vsum[w][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, bf, vsum[w][t], 0, 0, 0);
#pragma unroll
              for (int kg = 0; kg < KG; kg++)
                acc[w][t][kg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[kg], bf, acc[w][t][kg], 0, 0, 0);
            }
        }
      }
    __syncthreads();
  }

  // ---- M to LDS; lane: tile col, filters 4*kq .. of each group ----
  bool huge = false;
#pragma unroll
  for (int w = 0; w < PW; w++) {
    const int e = wave * PW + w;
    const float sc = sc_s[e] / unit, ou = ou_s[e];
#pragma unroll
    for (int t = 0; t < TG; t++) {
      const float off = ou * vsum[w][t][0];
#pragma unroll
      for (int kg = 0; kg < KG; kg++) {
        float* dstm = ex + ((e * KG + kg) * TG + t) * 256;
        v4f m;
#pragma unroll
        for (int r = 0; r < 4; r++) {
          m[r] = __builtin_fmaf(sc, acc[w][t][kg][r], off);
          huge |= !(fabsf(m[r]) < 0x1p118f);  // (A^T M A is at most 361 times the largest M)
        }
        if constexpr (kNhwc) {
          *reinterpret_cast<v4f*>(dstm + col * 16 + 4 * kq) = m;
        } else {
#pragma unroll
          for (int r = 0; r < 4; r++) dstm[r * 64 + kq * 16 + col] = m[r];
        }
      }
    }
  }
  if (huge) *huge_s = 1;
  __syncthreads();
  using PairsT = Pairs<M, TG, KG, kNhwc>;
  float o[PairsT::kTurns][M][M];
  const bool check = __builtin_amdgcn_readfirstlane(*huge_s) != 0;
#pragma unroll
  for (int t = 0; t < PairsT::kTurns; t++) {
    const PairsT pr(tid, t);
    if (!pr.exists()) continue;
    float mm[A][A];
#pragma unroll
    for (int e = 0; e < E; e++) mm[e / A][e % A] = ex[e * KG * TG * 256 + pr.i];
    out2d<M>(mm, o[t]);
#pragma unroll
    for (int r = 0; r < M * M; r++) o[t][r / M][r % M] *= 1.0f / kUp;
  }
  if (check) {
    int own = tid;
    asm volatile("" : "+v"(own));  // (nothing of the following is computed ahead of here)
    bool bad[PairsT::kTurns];
#pragma unroll
    for (int t = 0; t < PairsT::kTurns; t++) {
      float zero = 0.0f;
#pragma unroll
      for (int r = 0; r < M * M; r++) zero += 0.0f * o[t][r / M][r % M];
      bad[t] = PairsT(own, t).exists() && zero != 0.0f;  // not finite
    }
    plain_results<M, TG, KG, kNhwc>(a, sc_s, k0, p0, own, ex, bad, o);
  }
#pragma unroll
  for (int t = 0; t < PairsT::kTurns; t++) {
    const PairsT pr(tid, t);
    const int k = k0 + pr.kin, p = p0 + pr.pin;
    if (!pr.exists() || k >= K || p >= P) continue;
    const int ox0 = (p % a.tw) * M, q2 = p / a.tw;
    const int oy0 = (q2 % a.th) * M, on = q2 / a.th;
    const bool whole = !kNhwc && ox0 + M <= a.Wo;
#pragma unroll
    for (int r = 0; r < M; r++) {
      const bool row = oy0 + r < a.Ho;
      if (whole) {
        const unsigned off = (unsigned)dev::act_index(false, on, k, oy0 + r, ox0, K, a.Ho, a.Wo) * 4u;
        pos::store_row<M>(a.y, a.y_bytes, row ? off : kOobY, o[t][r]);
      } else {
#pragma unroll
        for (int s = 0; s < M; s++)
          pos::store_b32(a.y, a.y_bytes, row && ox0 + s < a.Wo
                                     ? (unsigned)dev::act_index(kNhwc, on, k, oy0 + r, ox0 + s, K, a.Ho, a.Wo) * 4u
                                     : kOobY, o[t][r][s]);
      }
    }
  }
}

struct WoArgs {
  const float* x;
  const int8_t* uq;       // [E][NB][K][CB], layout of lance.h
  const float* u_range;   // [E][2]
  float* y;
  int N, C, H, W, K, pad, th, tw, P, Ho, Wo, bits_w, nhwc, CB, NB;
};

template <int M, int kF>
__global__ __launch_bounds__(kThreads) void weight_only_kernel(const WoArgs a) {
  constexpr int A = M + 2, E = A * A;
  static_assert(kF * E <= kThreads, "one thread per (filter, position)");
  __shared__ float us[kF][E];
  __shared__ float mn_s[E], sc_s[E];
  const int tid = threadIdx.x;
  const int p = blockIdx.x * kThreads + tid;
  const int k0 = blockIdx.y * kF;
  const bool valid = p < a.P;
  const int pt = min(p, a.P - 1);
  const int tx = pt % a.tw, t2 = pt / a.tw;
  const int ty = t2 % a.th, n = t2 / a.th;
  const int y0 = ty * M - a.pad, x0 = tx * M - a.pad;
  if (tid < E) {
    float inv, scale;
    dev::quant_params(a.u_range[2 * tid], a.u_range[2 * tid + 1], a.bits_w, &inv, &scale);
    mn_s[tid] = a.u_range[2 * tid];
    sc_s[tid] = scale;
  }
  float acc[kF][E];
#pragma unroll
  for (int f = 0; f < kF; f++)
#pragma unroll
    for (int e = 0; e < E; e++) acc[f][e] = 0.0f;
  const int h = 1 << (a.bits_w - 1);
  const int fe_f = tid / E, fe_e = tid % E;   // this thread's (filter, position) of the block
  const int kq = min(k0 + fe_f, a.K - 1);
  const int Q = a.CB / 4;

  for (int c = 0; c < a.C; c++) {
    __syncthreads();  // the previous channel's filter values have been read (and mn_s, sc_s set)
    if (tid < kF * E) {
      const int b = c / a.CB, r = c % a.CB;
      const int pos = a.nhwc ? r : 4 * (r % Q) + r / Q;
      const int code = (int)a.uq[(((size_t)fe_e * a.NB + b) * a.K + kq) * a.CB + pos] + h;
      us[fe_f][fe_e] = (float)code * sc_s[fe_e] + mn_s[fe_e];
    }
    float d[A][A];
#pragma unroll
    for (int r = 0; r < A; r++)
#pragma unroll
      for (int s = 0; s < A; s++) {
        const int gy = y0 + r, gx = x0 + s;
        const bool ok = gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
        const float v = a.x[dev::act_index(a.nhwc, n, c, min(max(gy, 0), a.H - 1),
                                           min(max(gx, 0), a.W - 1), a.C, a.H, a.W)];
        d[r][s] = ok ? v : 0.0f;
      }
    dev::input_tile_transform<M>(d);
    __syncthreads();
#pragma unroll
    for (int f = 0; f < kF; f++)
#pragma unroll
      for (int e = 0; e < E; e++) acc[f][e] = __builtin_fmaf(us[f][e], d[e / A][e % A], acc[f][e]);
  }

  if (!valid) return;
#pragma unroll
  for (int f = 0; f < kF; f++) {
    const int k = k0 + f;
    if (k >= a.K) break;
    float t[M][A];  // S = A^T M A: rows first, then columns
#pragma unroll
    for (int o = 0; o < M; o++)
#pragma unroll
      for (int j = 0; j < A; j++) {
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < A; i++) {
          const float cf = dev::Wino<M>::at(o, i);
          if (cf != 0.0f) s += cf * acc[f][i * A + j];
        }
        t[o][j] = s;
      }
#pragma unroll
    for (int o = 0; o < M; o++)
#pragma unroll
      for (int q = 0; q < M; q++) {
        float s = 0.0f;
#pragma unroll
        for (int j = 0; j < A; j++) {
          const float cf = dev::Wino<M>::at(q, j);
          if (cf != 0.0f) s += cf * t[o][j];
        }
        const int yy = ty * M + o, xx = tx * M + q;
        if (yy < a.Ho && xx < a.Wo) a.y[dev::act_index(a.nhwc, n, k, yy, xx, a.K, a.Ho, a.Wo)] = s;
      }
  }
}

}  // namespace

template <int M, int TG, int KG>
static hipError_t launch_mfma(const WmArgs& a, int load, hipStream_t s) {
  constexpr int E = (M + 2) * (M + 2), NH = M == 2 ? 2 / TG : 1;
  constexpr size_t codes = (size_t)E * 3 * NH * TG * 1024, exch = (size_t)E * KG * TG * 1024;
  constexpr size_t lds = 512 + (codes > exch ? codes : exch);
  const unsigned grid = (unsigned)((a.P + 16 * TG - 1) / (16 * TG)) * (unsigned)a.nky;
  auto go = [&](auto kern) -> hipError_t {
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds);
    if (e != hipSuccess) return e;
    kern<<<grid, M == 2 ? 1024 : 768, lds, s>>>(a);
    return hipGetLastError();
  };
  switch (load) {
    case pos::kRowsEdge: return go(weight_only_mfma_kernel<M, TG, KG, pos::kRowsEdge>);
    case pos::kRowsAny: return go(weight_only_mfma_kernel<M, TG, KG, pos::kRowsAny>);
    default: return go(weight_only_mfma_kernel<M, TG, KG, pos::kNhwc1>);
  }
}

namespace {
// How the matrix-core kernel's work is cut: 16*tg tiles x 16*kg filters per workgroup.
struct WmShape {
  int tg, kg;
  long long groups;
};

// Smallest (rounds of one workgroup per compute unit: LDS) x (relative time of a workgroup).  The
// times are from sweeps of the six shapes over layers of 3 to 400 channels; 64 -> 64 channels, 8192
// tiles: 13.6 us with (2, 4) = 256 workgroups, 16.8 with (1, 4), 25 with (1, 2), 37 with (1, 1);
// 249 -> 21 channels, 1026 tiles: 14.8 with (1, 1), 33 with (2, 4).
WmShape wm_shape(const Geo& g) {
  static constexpr double kCost[2][3] = {{1.0, 1.2, 1.55}, {1.55, 1.85, 2.45}};
  WmShape best{1, 1, 0};
  double best_cost = 0.0;
  for (int tgi = 1; tgi <= (g.m == 2 ? 2 : 1); tgi++)
    for (int i = 0; i < (g.m == 2 ? 3 : 2); i++) {
      const int kg = 1 << i;
      const long long groups = ((g.P + 16LL * tgi - 1) / (16 * tgi)) * ((g.K + 16 * kg - 1) / (16 * kg));
      const double c = (double)((groups + 255) / 256) * kCost[tgi - 1][i];
      if (best_cost == 0.0 || c < best_cost) { best = WmShape{tgi, kg, groups}; best_cost = c; }
    }
  return best;
}

// Filters per workgroup of the vector-ALU kernel.
int plain_filters(const Geo& g) { return g.m == 2 ? 8 : 4; }

// Whether the vector-ALU kernel takes less time: both times in us from fits to sweeps over 1 to 64
// channels, 1 to 600 filters, 9 to 506250 tiles, both layouts (each kernel on each of 7000 layers: of the
// 52 on which the choice costs more than 5 %, 35 take up to 1.4 times the vector form's time, 17 up to
// 1.25 times the matrix form's).  100352 tiles of F(2x2), vector and matrix form: 1 -> 8 channels 9 and 58 us,
// 16 -> 8 40 and 58, 3 -> 40 42 and 88, 16 -> 64 220 and 93; NHWC 3 -> 4 13 and 58, 3 -> 16 105 and 59.
bool vector_form_faster(const Geo& g, const WmShape& sh) {
  // Vector form: the latency of one workgroup, or its rounds where the workgroups share compute units, each
  // linear in C; the latency grows with the filters of a workgroup (their stores), too.  NHWC: stores are
  // K floats apart, worst at 16 filters (one 64-byte piece per pixel), and loads C floats.
  struct Fit { double lat, lat_c, lat_k, base, round, round_c; int most_c, nhwc_most_c, nhwc_most_k; };
  static constexpr Fit kFit[2] = {{2.1, 1.5, 0.3, 1.4, 2.1, 0.95, 64, 12, 20}, {1.5, 4.5, 1.6, 0.7, 7.1, 5.1, 20, 6, 12}};
  const bool nhwc = is_nhwc(g), m4 = g.m == 4;
  const Fit& f = kFit[m4];
  if (g.C > (nhwc ? f.nhwc_most_c : f.most_c) || (nhwc && (g.K > f.nhwc_most_k || g.K == 16))) return false;
  const int kf = plain_filters(g);
  const long long blocks = ((g.P + kThreads - 1LL) / kThreads) * ((g.K + kf - 1) / kf);
  double vector_us = f.lat + f.lat_c * g.C + f.lat_k * (g.K < kf ? g.K : kf);
  const double by_rounds = f.base + (double)((blocks + 255) / 256) * (f.round + f.round_c * g.C);
  if (blocks > 128 && by_rounds > vector_us) vector_us = by_rounds;
  if (nhwc)
    vector_us += (m4 ? 90e-6 : (g.C % 4 == 0 ? 25e-6 : 15e-6)) * (g.K > 16 ? 1.7 : 1.0) * (double)g.P * g.K;
  // Matrix form: launch + rounds of one workgroup per compute unit, by shape: {launch, the first turn
  // over 32 channels, the second}.
  struct Turn { double launch, first, second; };
  static constexpr Turn kTurn2[2][3] = {{{2.5, 2.5, 0.0}, {3.0, 3.0, 0.0}, {3.5, 3.5, 0.0}},
                                        {{1.55, 4.33, 2.24}, {1.9, 5.3, 2.8}, {2.2, 7.3, 3.4}}};
  static constexpr Turn kTurn4[2] = {{2.0, 6.2, 3.55}, {2.4, 7.6, 4.4}};
  const int ki = sh.kg == 4 ? 2 : sh.kg - 1;
  const Turn& t = m4 ? kTurn4[ki] : kTurn2[sh.tg - 1][ki];
  const bool two_turns = g.C > 16 && (m4 || sh.tg == 2);
  const double matrix_us = t.launch + (double)((sh.groups + 255) / 256) * (t.first + (two_turns ? t.second : 0.0));
  return vector_us < matrix_us;
}

hipError_t launch_vector(const Geo& g, const float* x, const int8_t* uq, const float* u_range, float* y,
                         hipStream_t s) {
  const WoArgs a{x, uq, u_range, y, g.N, g.C, g.H, g.W, g.K, g.pad, g.th, g.tw, g.P, g.Ho, g.Wo,
                 g.bits_w, is_nhwc(g) ? 1 : 0, g.CB, g.NB};
  const int kf = plain_filters(g);
  const long long bx = ((long long)g.P + kThreads - 1) / kThreads, by = (g.K + kf - 1) / kf;
  if (bx > 0x7FFFFFFFLL || by > 65535) return hipErrorInvalidValue;
  dim3 grid((unsigned)bx, (unsigned)by, 1);
  if (g.m == 2) weight_only_kernel<2, 8><<<grid, kThreads, 0, s>>>(a);
  else weight_only_kernel<4, 4><<<grid, kThreads, 0, s>>>(a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_weight_only(const Geo& g, const float* x, const int8_t* uq, const float* u_range,
                              float* y, hipStream_t s) {
  const WmShape sh = wm_shape(g);
  if ((long long)g.N * g.C * g.H * g.W * 4 >= 0x7FF00000LL || vector_form_faster(g, sh))
    return launch_vector(g, x, uq, u_range, y, s);
  const int nky = (g.K + 16 * sh.kg - 1) / (16 * sh.kg);
  if (((g.P + 15LL) / 16) * nky > 0x7FFFFFFFLL) return hipErrorInvalidValue;
  const WmArgs a{x, uq, u_range, y, g.N, g.C, g.H, g.W, g.K, g.pad, g.P, g.th, g.tw, g.Ho, g.Wo,
                 g.bits_w, g.NB, g.CB == 16 ? 1 : 0, nky,
                 (unsigned)((size_t)g.N * g.C * g.H * g.W * 4),
                 (unsigned)((size_t)g.N * g.K * g.Ho * g.Wo * 4)};
  const int load = is_nhwc(g) ? pos::kNhwc1 : (patch_edge_cols_only(g) ? pos::kRowsEdge : pos::kRowsAny);
  if (g.m == 4)
    return sh.kg == 1 ? launch_mfma<4, 1, 1>(a, load, s) : launch_mfma<4, 1, 2>(a, load, s);
  if (sh.tg == 1)
    return sh.kg == 1 ? launch_mfma<2, 1, 1>(a, load, s)
                      : (sh.kg == 2 ? launch_mfma<2, 1, 2>(a, load, s) : launch_mfma<2, 1, 4>(a, load, s));
  return sh.kg == 1 ? launch_mfma<2, 2, 1>(a, load, s)
                      : (sh.kg == 2 ? launch_mfma<2, 2, 2>(a, load, s) : launch_mfma<2, 2, 4>(a, load, s));
}

}  // namespace lance
