// Stages 2 (second pass) + 3 + 4 in one kernel for F(2x2,3x3) layers with one or two 64-channel
// blocks whose tiles pair up (NCHW, pad 1, width a multiple of 4; NHWC, C a multiple of 4, X 16-byte aligned, any
// padding and width): v^ = Q(B^T d B) (Algorithm 1; Eq. 7) is formed in registers and written to LDS only, the int8 products of Sec. 3.3 run on
// the matrix cores from there, and the de-quantization (Eq. 8) and output transform (Eq. 9) are
// applied to the register accumulators.  The codes of V never touch device memory.
//
// A workgroup of eight waves owns 32 pairs of tiles (one channel block) or 16 (two) and all
// filters; its codes take 64 KB of LDS, so two workgroups and four waves per SIMD share a compute
// unit (128 registers).
//
// Phase T (quant_pairs.h): every wave quantizes four channels of its pairs per lane.  Phase G: wave
// w takes 16 filters of a block of 64 or 128 and 16 pairs (v_mfma_i32_16x16x64_i8, one accumulator
// for the left and one for the right tiles): B fragments from LDS, A fragments (uq, cache resident)
// three positions ahead.  A lane ends up with four neighbouring output pixels of two rows: 16-byte
// stores.  Epilogue algebra: M[e,k,p] = s_e*ACC + f[e,k] + g[e,p]; the three terms go through the
// linear map S = A^T M A separately; f is formed from the filter row sums (binary64) once per
// workgroup, g from the column sums.
//
// What bounds it, N64 128 -> 128 56x56 with caller's ranges (44 K cycles per workgroup): vector ALUs
// about half of the time (20.8 M wave instructions), the rest memory that is not overlapped: without
// the stores of Y the kernel took 23 us less, without the pixel loads 18.  So, all measured there:
//  * half as many loads as one tile per lane needs, and the column beside a group of lanes in one
//    load per channel (a load per row: 23 us more, the addresses' cache lines counted twice);
//  * constants before pixels (EarlyLoads): 77 -> 67 us;
//  * non-temporal stores where they pay (store_rule.h);
//  * one block of tiles per workgroup: persistent workgroups, which form the constants once, were
//    10 to 20 us slower - their next loads wait for the stores before them.
// Against one tile per lane (conv_fused_c64.hip, conv_fused_c128.hip), whole call, dynamic ranges: N64
// 128 -> 128 56x56 103.9 -> 89.3 us, N128 64 -> 64 32x32 29.9 -> 27.5, N16 64 -> 64 224x224 (caller's
// ranges) 137 -> 115, N16 128 -> 128 112x112 100 -> 81.
//
// NHWC.  A thread takes one pair and four channels; a pair's window is six columns of four 16-byte loads, four
// columns in flight before the constants are formed.  That leaves no registers for the filter row sums there,
// so the filter-side terms are formed behind phase T (before it, with two columns in flight: 64 bytes spilled, N64
// 128 -> 128 56x56 with caller's ranges 81 us instead of 67).  A pixel's 16 filters of a wave are one 64-byte run of Y.
// Against four tiles per thread in workgroups of four waves, two tile columns of the window kept from tile to
// tile, whole call with the faster range pass, dynamic ranges: N64 128 -> 128 56x56 106 -> 93 us, N16 64 -> 64
// 224x224 190 -> 162, N128 64 -> 64 32x32 36.7 -> 30.5, N30 128 -> 512 33x35 68.2 -> 57.4.  This kernel between two
// events, same buffers (X in the last-level cache): 82.0 -> 73.2, 144 -> 124, 29.6 -> 24.6, 62.5 -> 52.9, and the range pass
// 24.7, 43.0, 10.9, 9.6: about 5 us more than the call, for the events and a launch behind an idle chip each.  With inputs and
// outputs that rotate past the cache the calls take 111 -> 97, 201 -> 179, 40.9 -> 34.8, 71.6 -> 61.5.  Bound by the same
// things as above.
//
// The last, partial round: a workgroup beyond a multiple of 256 takes its whole time on an almost idle chip.  128 -> 128
// 56x56 with caller's ranges, 62 / 63 / 64 images (5.93, 6.03 and 6.13 times 256 workgroups): NCHW 53.9 / 58.4 / 58.7 us,
// NHWC 61.7 / 68.3 / 68.7.
#include "lance_device.h"
#include "lance_internal.h"
#include "quant_pairs.h"
#include <utility>

namespace lance {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int kCodeBytes = 65536;  // codes of a block of tiles: 64 tiles x 1 or 32 x 2 channel blocks
constexpr unsigned kOob = 0xFFFFFFF0u;

struct CpArgs {
  dev::PairGeo g;
  const int8_t* uq;
  const float* u_range;      // [E][2]
  const int32_t* u_rowsum;   // [E][K]
  const float* partial;      // [count][E][2] records of the range pass
  float* v_range;            // [E][2]: written by workgroup 0, or read when is_static
  float* y;
  int count, per_tensor, is_static, bits_w;
  int K;
  unsigned uq_bytes, y_bytes;
  int stream;                // Y is stored past the caches
};

template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{})
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// A^T of F(2x2,3x3) (points 0, 1, -1, inf), for compile-time indices.
constexpr float kAt2[2][4] = {{1, 1, 1, 0}, {0, 1, -1, -1}};

// (a kernel body must not name the descriptor type: the host stub would be lost)
__device__ __forceinline__ v4i load_codes(const int8_t* uq, unsigned bytes, unsigned off, unsigned plane) {
  const __amdgpu_buffer_rsrc_t res =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uq), 0, bytes, 0x00020000);
  return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(res, off, plane, 0));
}
// The scalar offset stays the constant 0: with a register there the compiler takes a 16-byte store
// to be free of the rule that the instruction behind it must not overwrite its data, and on gfx950
// it is not (first words of stored rows came from the next row).
// STREAM: non-temporal (store_rule.h says when).
template <bool STREAM>
__device__ __forceinline__ void store_row(float* y, unsigned bytes, unsigned off, float a, float b,
                                          float c, float d) {
  const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(y, 0, bytes, 0x00020000);
  const v4u v = {__float_as_uint(a), __float_as_uint(b), __float_as_uint(c), __float_as_uint(d)};
  __builtin_amdgcn_raw_buffer_store_b128(v, res, off, 0, STREAM ? 2 : 0);
}

// What a workgroup's constants are formed from, requested before the first pixels: loads return in
// order, and behind the pixels these small ones from L2 would wait for memory.
struct EarlyLoads {
  static constexpr int kRecords = 4;  // records per thread (256 in a workgroup)
  v4f rec[kRecords];                  // {min, max} of positions 2*piece, 2*piece + 1
  float ur[2], vr[2];                 // threads 0..15: filter range, caller's input range of position tid
};

// Ranges of the input (Eq. 7's T) and the constants of Eq. 7 and of the expanded Eq. 8, by all 512
// threads; ends in a barrier.  With ou = min_u + su*h, ov = min_v + sv*h:
//   M[e,k,p] = su*sv*ACC + (su*ov*rowsum[e][k] + C*ou*ov) + sv*ou*colsum[e][p].
struct Constants {
  float *sc, *gc;           // [E] su*sv, sv*ou
  float *qp;                // [E][2] = {min, inv} of Eq. 7
  double *rmul, *kconst;    // [E] su*ov, C*ou*ov
  float *red;               // scratch: [8 waves][E][2], then [E][2]

  __device__ __forceinline__ static void request(const CpArgs& a, int tid, EarlyLoads& l) {
    constexpr int E = 16;
    const int e = tid & 15;
#pragma unroll
    for (int i = 0; i < 2; i++) l.ur[i] = a.u_range[2 * e + i];
    if (a.is_static) {
#pragma unroll
      for (int i = 0; i < 2; i++) l.vr[i] = a.v_range[2 * e + i];
    } else {
#pragma unroll
      for (int u = 0; u < EarlyLoads::kRecords; u++)  // (past the last record: the last one again)
        l.rec[u] = *reinterpret_cast<const v4f*>(
            a.partial + (size_t)min((tid >> 3) + u * (kThreads / 8), a.count - 1) * (2 * E) + 4 * (tid & 7));
    }
  }

  __device__ __forceinline__ void form(const CpArgs& a, int tid, EarlyLoads& l) const {
    constexpr int E = 16;
    float lo = l.vr[0], hi = l.vr[1];
    if (!a.is_static) {
      v4f v = l.rec[0];
      auto merge = [&](const v4f& x) {
        v[0] = fminf(v[0], x[0]); v[1] = fmaxf(v[1], x[1]);
        v[2] = fminf(v[2], x[2]); v[3] = fmaxf(v[3], x[3]);
      };
#pragma unroll
      for (int u = 1; u < EarlyLoads::kRecords; u++) merge(l.rec[u]);
      for (int row = (tid >> 3) + EarlyLoads::kRecords * (kThreads / 8); row < a.count; row += kThreads / 8)
        merge(*reinterpret_cast<const v4f*>(a.partial + (size_t)row * (2 * E) + 4 * (tid & 7)));
#pragma unroll
      for (int o = 8; o < 64; o <<= 1) {  // lanes of the same piece
        const v4f x = {__shfl_xor(v[0], o, 64), __shfl_xor(v[1], o, 64), __shfl_xor(v[2], o, 64), __shfl_xor(v[3], o, 64)};
        merge(x);
      }
      if ((tid & 63) < 8) *reinterpret_cast<v4f*>(red + (tid >> 6) * 2 * E + 4 * (tid & 7)) = v;
      __syncthreads();
    }
    if (tid < E) {
      if (!a.is_static) {
        lo = red[2 * tid]; hi = red[2 * tid + 1];
#pragma unroll
        for (int w = 1; w < kThreads / 64; w++) {
          lo = fminf(lo, red[w * 2 * E + 2 * tid]);
          hi = fmaxf(hi, red[w * 2 * E + 2 * tid + 1]);
        }
        if (a.per_tensor) {
#pragma unroll
          for (int o = 1; o < E; o <<= 1) {
            lo = fminf(lo, __shfl_xor(lo, o, 64));
            hi = fmaxf(hi, __shfl_xor(hi, o, 64));
          }
        }
        if (blockIdx.x == 0) { a.v_range[2 * tid] = lo; a.v_range[2 * tid + 1] = hi; }
      }
      float iu, su, inv, sv;
      dev::quant_params(l.ur[0], l.ur[1], a.bits_w, &iu, &su);
      dev::quant_params(lo, hi, a.g.bits, &inv, &sv);
      const double ou = (double)l.ur[0] + (double)su * (double)(1 << (a.bits_w - 1));
      const double ov = (double)lo + (double)sv * (double)(1 << (a.g.bits - 1));
      qp[2 * tid] = lo;
      qp[2 * tid + 1] = inv;
      sc[tid] = (float)((double)su * (double)sv);
      gc[tid] = (float)((double)sv * ou);
      rmul[tid] = (double)su * ov;
      kconst[tid] = (double)a.g.C * ou * ov;
    }
    __syncthreads();
  }
};

// LDS of a workgroup but the filter-side terms; two workgroups share a compute unit's 160 KB.
template <int NB>
constexpr int fixed_lds() {
  return kCodeBytes + 16 * (64 / NB) * (int)sizeof(int) + (16 + 16 + 32) * (int)sizeof(float) +
         2 * 16 * (int)sizeof(double);
}
constexpr int kMaxLds = 80 * 1024;

// Pixels in flight: of the next channels (NCHW), or columns of the lane's windows (NHWC).
template <class Phase, int AHEAD, bool NHWC>
struct PixelsOf {
  typename Phase::Pixels buf[AHEAD + 1];
};
template <class Phase, int AHEAD>
struct PixelsOf<Phase, AHEAD, true> {
  v4f buf[Phase::kBuffers][4];
};

// NB: channel blocks.  B8: 8-bit codes.  FULL: all channels of the blocks exist (NCHW).  STREAM (NHWC): Y is stored
// past the caches; NCHW asks a.stream.  ANY (NHWC): pairs of any two consecutive tiles.
template <int NB, bool B8, bool FULL, bool NHWC, bool STREAM = false, bool ANY = false>
__device__ __forceinline__ void conv_body(const CpArgs& a) {
  constexpr int M = 2, A = 4, E = 16;
  constexpr int kPairs = 32 / NB, kTiles = 2 * kPairs, kPlane = kTiles * 64;
  constexpr int kFilters = 64 * NB;  // filters of a block
  constexpr int kMostBlocks = (kMaxLds - fixed_lds<NB>()) / (kFilters * 16);  // 704 and 768 filters
  constexpr int kFragsAhead = 3;     // positions whose A fragments are in flight ahead of the products
  constexpr int kStepsAhead = 1;     // channels whose pixels are in flight ahead of the transform
  using Phase = std::conditional_t<NHWC, dev::PairPhaseNhwc<B8, kPairs, ANY>, dev::PairPhase<B8, FULL, kPairs>>;
  extern __shared__ char smem[];
  char* ring = smem;                                            // [NB][E][kTiles rows][64 B]
  int* cs_s = reinterpret_cast<int*>(smem + kCodeBytes);         // [E][kTiles] column sums (signed codes)
  float* sc_s = reinterpret_cast<float*>(cs_s + E * kTiles);    // [E] s_e = scale_u * scale_v
  float* gc_s = sc_s + E;                                       // [E] scale_v * offset_u
  float* qp_s = gc_s + E;                                       // [E][2] = {min, inv} of Eq. 7
  double* rmul_s = reinterpret_cast<double*>(qp_s + 2 * E);     // [E] scale_u * offset_v
  double* kconst_s = rmul_s + E;                                // [E] C * offset_u * offset_v
  float* rk_s = reinterpret_cast<float*>(kconst_s + E);         // [K, whole blocks][M*M]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K;
  // the workgroup's blocks of filters: all, or (NHWC, more of them than LDS has room for the terms of) its share
  const int kb0 = NHWC ? (int)blockIdx.y * kMostBlocks : 0;
  const int nkb = NHWC ? min((K + kFilters - 1) / kFilters, kb0 + kMostBlocks) : (K + kFilters - 1) / kFilters;
  const int kbase = kb0 * kFilters;
  const int blk = dev::xcd_contiguous(blockIdx.x, gridDim.x);

  // ============================ phase T ============================
  // wave & 3: 16-byte chunk of the code rows; wave >> 2: channel block, or half of the chunk
  const int chunk = wave & 3, upper = wave >> 2;
  Phase ph;
  PixelsOf<Phase, kStepsAhead, NHWC> px;
  auto request_rowsums = [&](int k0, int32_t (&rowsum)[E]) {
#pragma unroll
    for (int e = 0; e < E; e++) rowsum[e] = a.u_rowsum[(size_t)e * K + min(k0 + lane, K - 1)];
  };
  // filter-side terms rk_s[4*filter + ab] = sum_e A^T[a][i] A^T[b][j] (su*ov*rowsum[e][k] + C*ou*ov):
  // wave & 3 = ab, lane = filter; rowsum: of the first turn's filters
  auto filter_terms = [&](int32_t (&rowsum)[E]) {
    const int aa = (wave >> 1) & 1, b = wave & 1;
    for (int k0 = kbase + 64 * upper; k0 < nkb * kFilters; k0 += 128) {
      if (k0 >= kbase + 128) request_rowsums(k0, rowsum);
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < A; j++) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < A; i++)
          s = __builtin_fma((double)dev::at_coef(M, aa, i),
                            __builtin_fma(rmul_s[4 * i + j], (double)rowsum[4 * i + j], kconst_s[4 * i + j]), s);
        acc = __builtin_fma((double)dev::at_coef(M, b, j), s, acc);
      }
      rk_s[4 * (k0 - kbase + lane) + (wave & 3)] = (float)acc;
    }
  };
  {
    EarlyLoads early;
    Constants::request(a, tid, early);
    [[maybe_unused]] int32_t rowsum[E];
    if constexpr (NHWC) {  // four pairs per wave
      ph.setup(a.g, blk, 4 * (NB == 2 ? chunk : wave) + (lane >> 4), NB == 2 ? upper : 0, lane,
               ring + (NB == 2 ? upper * (E * kPlane) : 0));
#pragma unroll
      for (int s = 0; s < Phase::kEarly; s++) ph.issue(a.g, s, px.buf[s]);
    } else {
      request_rowsums(64 * upper, rowsum);
      ph.setup(a.g, blk, (NB == 2 ? 64 * upper : 2 * upper) + 4 * chunk, lane);
#pragma unroll
      for (int k = 0; k < kStepsAhead; k++) ph.issue(a.g, k, px.buf[k]);
    }
    // (the code rows are free until the first codes are written)
    const Constants cst{sc_s, gc_s, qp_s, rmul_s, kconst_s, reinterpret_cast<float*>(ring)};
    cst.form(a, tid, early);
    if constexpr (!NHWC) filter_terms(rowsum);
  }
  const unsigned plane_px = (unsigned)a.g.H * (unsigned)a.g.W;
  {
    float qmn[E], qinv[E];  // Eq. 7 parameters as wave-uniform scalars
#pragma unroll
    for (int e = 0; e < E; e++) {
      qmn[e] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(qp_s[2 * e])));
      qinv[e] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(qp_s[2 * e + 1])));
    }
    if constexpr (NHWC) {
      int32_t rowsum[E];
      ph.run(a.g, px.buf, qmn, qinv, [&]() { request_rowsums(kbase + 64 * upper, rowsum); });
      filter_terms(rowsum);
    } else {
      const float L = (float)((1 << a.g.bits) - 1);
      unsigned codes[2][E];
#pragma unroll
      for (int k = 0; k < Phase::kSteps; k++) {
        if (k + kStepsAhead < Phase::kSteps)
          ph.issue(a.g, k + kStepsAhead, px.buf[(k + kStepsAhead) % (kStepsAhead + 1)]);
        ph.quantize(px.buf[k % (kStepsAhead + 1)], qmn, qinv, L, k, codes);
      }
      ph.store(a.g, chunk, (NB == 2 ? 0 : 2 * upper) + lane / kPairs, lane,
               ring + (NB == 2 ? upper * (E * kPlane) : 0), codes);
    }
  }

  // ============================ phase G ============================
  // The index arithmetic of this phase starts from a lane number the compiler cannot see
  // through: otherwise it is hoisted above phase T and held in registers (or spilled) across it.
  int lane_g = lane;
  asm volatile("" : "+v"(lane_g)::"memory");
  const int col = lane_g & 15, kq = lane_g >> 4;  // fragment row; 16-byte piece of the 64 channels
  // wave: 16 filters of a block; with one channel block also one half of the 32 pairs
  const int kwave = NB == 2 ? wave * 16 : (wave >> 1) * 16;
  const int pair = NB == 2 ? col : (wave & 1) * 16 + col;
  unsigned f_off[2];  // B fragment offsets of the pair's two tiles inside a position plane
#pragma unroll
  for (int s = 0; s < 2; s++) {
    const int row = kPairs * s + pair;
    f_off[s] = (unsigned)row * 64u + (unsigned)((kq ^ dev::row_swizzle_mfma32(row)) * 16);
  }
  // uq fragments of position e, one per channel block
  auto load_afrags = [&](int kb, int e, v4i (&af)[NB]) {
    const unsigned off = (unsigned)min(kb * kFilters + kwave + col, K - 1) * 64u + 16u * (unsigned)kq;
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
      af[nb] = load_codes(a.uq, a.uq_bytes, off, (unsigned)(e * NB + nb) * (unsigned)K * 64u);
  };
  v4i afrag[kFragsAhead + 1][NB];  // ring over positions (16 positions = four turns)
#pragma unroll
  for (int e = 0; e < kFragsAhead; e++) load_afrags(kb0, e, afrag[e]);
  dev::lds_barrier();  // the codes of all waves are in LDS
  // Column sums: one more matrix instruction per fragment, with an operand of ones; wave w takes the
  // positions 2w and 2w + 1 of all tiles.  (v_sad_u8 and LDS atomics, in phase T: 89.3 / 88.1 us on N64 128 ->
  // 128 56x56 with the other barrier, 44.8 / 42.6 on N64 100 -> 100 36x36.)
  {
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
#pragma unroll
    for (int e2 = 0; e2 < 2; e2++)
#pragma unroll
      for (int t = 0; t < kTiles / 16; t++) {
        const int e = 2 * wave + e2, row = 16 * t + col;
        const unsigned off = (unsigned)row * 64u + (unsigned)((kq ^ dev::row_swizzle_mfma32(row)) * 16);
        v4i sum = {0, 0, 0, 0};
#pragma unroll
        for (int nb = 0; nb < NB; nb++)
          sum = __builtin_amdgcn_mfma_i32_16x16x64_i8(
              ones, *reinterpret_cast<const v4i*>(ring + (nb * E + e) * kPlane + off), sum, 0, 0, 0);
        if (kq == 0) cs_s[e * kTiles + row] = sum[0];  // every row of the product is the same
      }
  }
  dev::lds_barrier();

  float gp[2][M * M];  // input-side terms of the lane's tiles through A^T . A
#pragma unroll
  for (int s = 0; s < 2; s++) {
#pragma unroll
    for (int ab = 0; ab < M * M; ab++) gp[s][ab] = 0.0f;
#pragma unroll
    for (int e = 0; e < E; e++) {
      const float ge = gc_s[e] * (float)cs_s[e * kTiles + kPairs * s + pair];
#pragma unroll
      for (int ab = 0; ab < M * M; ab++) {
        const float coef = kAt2[ab >> 1][e / A] * kAt2[ab & 1][e % A];
        if (coef != 0.0f) gp[s][ab] = __builtin_fmaf(coef, ge, gp[s][ab]);
      }
    }
  }
  // byte offsets of the pair's two output rows: of filter 0 (NCHW), or of their first pixels (NHWC; ANY: of each tile's)
  constexpr int kRuns = ANY ? 2 : 1;
  unsigned y_off[kRuns][2];
  int cols[kRuns];  // pixels of a row that exist
  cols[0] = 4;
  if constexpr (ANY) {
#pragma unroll
    for (int run = 0; run < 2; run++) {
      const int t = 2 * (blk * kPairs + pair) + run;
      int tx, ty, n;
      dev::locate_pair<true>(a.g, min(t, a.g.tiles - 1), &tx, &ty, &n);
      cols[run] = a.g.Wo - 2 * tx;
      const unsigned row = (unsigned)a.g.Wo * (unsigned)K * 4u;
      const unsigned base = ((unsigned)n * (unsigned)a.g.Ho + (unsigned)(2 * ty)) * row + (unsigned)(2 * tx) * (unsigned)K * 4u;
      y_off[run][0] = t < a.g.tiles ? base : kOob;
      y_off[run][1] = t < a.g.tiles && 2 * ty + 1 < a.g.Ho ? base + row : kOob;
    }
  } else {
    const int p = blk * kPairs + pair;
    int q, ty, n;
    dev::locate_pair<NHWC>(a.g, min(p, a.g.pairs - 1), &q, &ty, &n);
    unsigned base, row;
    if constexpr (NHWC) {
      cols[0] = a.g.Wo - 4 * q;
      row = (unsigned)a.g.Wo * (unsigned)K * 4u;
      base = ((unsigned)n * (unsigned)a.g.Ho + (unsigned)(2 * ty)) * row + (unsigned)(4 * q) * (unsigned)K * 4u;
    } else {
      row = (unsigned)a.g.W * 4u;
      base = ((unsigned)n * (unsigned)K * plane_px + (unsigned)(2 * ty) * (unsigned)a.g.W + 4u * (unsigned)q) * 4u;
    }
    y_off[0][0] = p < a.g.pairs ? base : kOob;
    y_off[0][1] = p < a.g.pairs && 2 * ty + 1 < (NHWC ? a.g.Ho : a.g.H) ? base + row : kOob;
  }

  for (int kb = kb0; kb < nkb; kb++) {
    v4f out[2][M * M];  // [tile of the pair][ab][accumulator register]
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
      for (int ab = 0; ab < M * M; ab++) out[s][ab] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    static_for<E>([&](auto ec) {
      constexpr int e = decltype(ec)::value;
      {  // request the A fragments kFragsAhead positions ahead (of the next filter block at the end)
        constexpr int en = (e + kFragsAhead) % E;
        const int kbn = e + kFragsAhead >= E ? kb + 1 : kb;
        if (kbn < nkb) load_afrags(kbn, en, afrag[(e + kFragsAhead) % (kFragsAhead + 1)]);
      }
      const v4i(&af)[NB] = afrag[e % (kFragsAhead + 1)];
      const char* plane = ring + e * kPlane;
      v4i acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int s = 0; s < 2; s++) {
          const v4i bf = *reinterpret_cast<const v4i*>(plane + nb * (E * kPlane) + f_off[s]);
          acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[nb], bf, acc[s], 0, 0, 0);
        }
      // Position e is complete: out[ab] += A^T[a][i] A^T[b][j] s_e ACC (coefficients +-1 or 0).
      // The empty statements tie the sums to their position (the compiler would otherwise sink
      // the folds of all positions to the first use of the outputs and keep every accumulator
      // until then).
      constexpr int gi = e / A, gj = e % A;
      const float se = sc_s[e];
#pragma unroll
      for (int s = 0; s < 2; s++) {
        v4f accf;
#pragma unroll
        for (int r = 0; r < 4; r++) accf[r] = (float)acc[s][r];
        static_for<4>([&](auto abc) {
          constexpr int ab = decltype(abc)::value;
          constexpr float coef = kAt2[ab >> 1][gi] * kAt2[ab & 1][gj];
          if constexpr (coef != 0.0f) {
            const float c = coef * se;
#pragma unroll
            for (int r = 0; r < 4; r++) out[s][ab][r] = __builtin_fmaf(c, accf[r], out[s][ab][r]);
            asm volatile("" : "+v"(out[s][ab]));
          }
        });
      }
    });

    // ---- tail: add the two separable terms, store the pair's two output rows of four pixels.
    // The lane holds filters kfirst + r (r = accumulator register).  Stores that must not happen
    // (pairs past the last, filters past K, the second row of an odd height) get an offset
    // beyond the buffer instead of a branch. ----
    const int kfirst = kb * kFilters + kwave + 4 * kq;  // first of the lane's four filters
    if constexpr (NHWC) {  // four consecutive filters of a pixel: one store
      v4f f4[4];
#pragma unroll
      for (int r = 0; r < 4; r++) f4[r] = *reinterpret_cast<const v4f*>(rk_s + 4 * (kfirst - kbase + r));
#pragma unroll
      for (int ab = 0; ab < M * M; ab++)
#pragma unroll
        for (int s = 0; s < 2; s++) {
          const int aa = ab >> 1, run = ANY ? s : 0, x = (ANY ? 0 : 2 * s) + (ab & 1);
          float o[4];
#pragma unroll
          for (int r = 0; r < 4; r++) o[r] = (out[s][ab][r] + f4[r][ab]) + gp[s][ab];
          dev::store_nhwc_k4<STREAM>(a.y, a.y_bytes, y_off[run][aa] + (unsigned)x * (unsigned)K * 4u,
                                     (unsigned)kfirst * 4u, y_off[run][aa] != kOob && x < cols[run], K - kfirst,
                                     STREAM || (K & 3) == 0, o[0], o[1], o[2], o[3]);
        }
      continue;
    }
    auto tail = [&](auto stream) {
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const unsigned koff = (unsigned)(kfirst + r) * plane_px * 4u;
        const v4f f4 = *reinterpret_cast<const v4f*>(rk_s + 4 * (kfirst + r));
        const bool k_ok = kfirst + r < K;
#pragma unroll
        for (int aa = 0; aa < M; aa++) {
          float o[4];
#pragma unroll
          for (int s = 0; s < 2; s++)
#pragma unroll
            for (int b = 0; b < M; b++)
              o[2 * s + b] = (out[s][2 * aa + b][r] + f4[2 * aa + b]) + gp[s][2 * aa + b];
          const unsigned off = k_ok && y_off[0][aa] != kOob ? y_off[0][aa] + koff : kOob;
          store_row<decltype(stream)::value>(a.y, a.y_bytes, off, o[0], o[1], o[2], o[3]);
        }
      }
    };
    if (a.stream) tail(std::true_type{}); else tail(std::false_type{});
  }
}

template <bool B8, bool FULL>
__global__ __launch_bounds__(kThreads, 4) void conv_fused_pairs_c64_kernel(const CpArgs a) {
  conv_body<1, B8, FULL, false>(a);
}
template <bool B8, bool FULL>
__global__ __launch_bounds__(kThreads, 4) void conv_fused_pairs_c128_kernel(const CpArgs a) {
  conv_body<2, B8, FULL, false>(a);
}
// The NHWC kernels of the plans of one and of two channel blocks, on pairs of a tile row and (conv_fused_any_pairs) of any
// two tiles.  STREAM is a parameter of the kernel: with both kinds of stores in one the cached ones took up to 2 %
// longer.
template <bool B8, bool STREAM>
__global__ __launch_bounds__(kThreads, 4) void conv_fused_pairs_nhwc_c64_kernel(const CpArgs a) {
  conv_body<1, B8, false, true, STREAM>(a);
}
template <bool B8, bool STREAM>
__global__ __launch_bounds__(kThreads, 4) void conv_fused_pairs_nhwc_c128_kernel(const CpArgs a) {
  conv_body<2, B8, false, true, STREAM>(a);
}
template <bool B8, bool STREAM>
__global__ __launch_bounds__(kThreads, 4) void conv_fused_any_pairs_nhwc_c64_kernel(const CpArgs a) {
  conv_body<1, B8, false, true, STREAM, true>(a);
}
template <bool B8, bool STREAM>
__global__ __launch_bounds__(kThreads, 4) void conv_fused_any_pairs_nhwc_c128_kernel(const CpArgs a) {
  conv_body<2, B8, false, true, STREAM, true>(a);
}

// LDS of a workgroup with the terms of K filters.
template <int NB>
int lds_bytes(int K) {
  return fixed_lds<NB>() + (K + 64 * NB - 1) / (64 * NB) * (64 * NB) * 16;
}

// Pairs in a tile row.
int pairs_per_row(const Geo& g) { return is_nhwc(g) ? (g.tw + 1) / 2 : g.W / 4; }

// Filters of a workgroup: those LDS has room for the terms of.
template <int NB>
constexpr int most_filters() { return (kMaxLds - fixed_lds<NB>()) / (64 * NB * 16) * (64 * NB); }

// Bytes from the first image of a block to the end of the last one that its pairs can touch; NHWC: of X.
long long reach_bytes(const Geo& g) {
  if (is_nhwc(g)) return (long long)g.N * g.C * g.H * g.W * 4;
  const int pairs = 32 / g.NB;
  const long long per_image = (long long)g.th * pairs_per_row(g);
  return ((pairs - 1) / per_image + 2) * g.C * g.H * g.W * 4LL;
}

template <int NB>
hipError_t launch_kernel(void (*kern)(CpArgs), const CpArgs& a, const char* name, hipStream_t s) {
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), kMaxLds);
  if (e != hipSuccess) return e;
  note_kernel(name);
  constexpr int kMost = most_filters<NB>();
  const dim3 grid((a.g.pairs + 32 / NB - 1) / (32 / NB), (a.K + kMost - 1) / kMost);
  kern<<<grid, kThreads, lds_bytes<NB>(a.K < kMost ? a.K : kMost), s>>>(a);
  return hipGetLastError();
}

template <int NB, bool B8, bool FULL>
hipError_t launch_variant(const CpArgs& a, hipStream_t s) {
  return NB == 1 ? launch_kernel<1>(conv_fused_pairs_c64_kernel<B8, FULL>, a, "conv_fused_pairs_c64_kernel", s)
                 : launch_kernel<2>(conv_fused_pairs_c128_kernel<B8, FULL>, a, "conv_fused_pairs_c128_kernel", s);
}

template <int NB>
hipError_t launch_blocks(const Geo& g, const CpArgs& a, hipStream_t s) {
  const bool b8 = g.bits == 8, full = g.C == 64 * NB;
  if (b8) return full ? launch_variant<NB, true, true>(a, s) : launch_variant<NB, true, false>(a, s);
  return full ? launch_variant<NB, false, true>(a, s) : launch_variant<NB, false, false>(a, s);
}

template <bool B8, bool STREAM>
hipError_t launch_nhwc(const Geo& g, const CpArgs& a, hipStream_t s) {
  if (conv_fused_any_pairs(g))
    return g.NB == 1
               ? launch_kernel<1>(conv_fused_any_pairs_nhwc_c64_kernel<B8, STREAM>, a, "conv_fused_any_pairs_nhwc_c64_kernel", s)
               : launch_kernel<2>(conv_fused_any_pairs_nhwc_c128_kernel<B8, STREAM>, a, "conv_fused_any_pairs_nhwc_c128_kernel", s);
  return g.NB == 1 ? launch_kernel<1>(conv_fused_pairs_nhwc_c64_kernel<B8, STREAM>, a, "conv_fused_pairs_nhwc_c64_kernel", s)
                   : launch_kernel<2>(conv_fused_pairs_nhwc_c128_kernel<B8, STREAM>, a, "conv_fused_pairs_nhwc_c128_kernel", s);
}

bool divisions_exact(long long pairs, long long npr, long long th) {
  return pairs * npr < 1LL << 32 && pairs * th < 1LL << 32;
}

CpArgs make_args(const Geo& g, const float* x, const int8_t* uq, const float* u_range, const int32_t* u_rowsum,
                 const float* partial, int count, float* v_range, float* y, bool stream) {
  const bool any = is_nhwc(g) && conv_fused_any_pairs(g);
  const int npr = any ? g.tw : pairs_per_row(g), pairs = any ? (g.P + 1) / 2 : g.N * g.th * npr;
  return CpArgs{{x, g.C, g.H, g.W, g.Ho, g.Wo, g.pad, g.th, npr, pairs, g.bits, g.P, div_magic(g.th), div_magic(npr),
                 divisions_exact(any ? g.P : pairs, npr, g.th) ? 1 : 0, (unsigned)reach_bytes(g)},
                uq, u_range, u_rowsum, partial, v_range, y, count,
                (g.flags & LANCE_RANGE_PER_TENSOR) ? 1 : 0, (g.flags & LANCE_INPUT_RANGE_STATIC) ? 1 : 0,
                g.bits_w, g.K, (unsigned)((size_t)g.E * g.NB * g.K * 64),
                (unsigned)((size_t)g.N * g.K * g.Ho * g.Wo * 4), stream ? 1 : 0};
}

}  // namespace

// NHWC: pairs of any two consecutive tiles, where that takes fewer rounds of one workgroup per compute unit.  With an
// odd number of tile columns every row of pairs ends in half a pair, with one column all pairs are halves; a pair of any
// two tiles costs 32 pixel loads and 8 column passes instead of 24 and 6.  Caller's ranges, pairs of a row / any pairs / four
// tiles per thread: N3571 128 -> 128 14x1 53.6 / 35.5 / 41.8 us, N96 120 -> 374 18x18 (270 and 243 workgroups) 70.4 / 44.2 / 51.0,
// N2940 128 -> 620 5x6 137.9 / 123.0 / 130.5.  Of 1500 random layers with more than two workgroups of the few-tile plan per
// compute unit 292 take this form; 0.14 % over the better form's time on average.  With the same number of rounds it
// is 2 % (300 filters and more) to 7 % (up to 16) slower.
// Filters that are no multiple of four take 4-byte stores, for which more workgroups are the better.  One channel block, one
// column of whole tiles, more than 128 filters: bound by them, pairs of a row (N17038 32 -> 1687 2x2 364 / 433 us, N20000 64 ->
// 301 2x2 87 / 101).  A last share of the filters, however small, counts as a whole one there (N1091 128 -> 798 3x5 91 / 58, N166 128 ->
// 1222 13x13 138 / 106): 0.6 % over the better form on 900 random layers with odd numbers of tile columns, 1.3 % with shares by
// their work and no such layer of more than 512 filters and three columns; none 5 % slower than four tiles per thread, before ten.
bool conv_fused_any_pairs(const Geo& g) {
  const bool whole_stores = g.K % 4 == 0;
  if (!whole_stores && g.NB == 1 && g.tw == 1 && g.Wo == 2 && g.K > 128) return false;
  // blocks of filters, and of a workgroup; the last share of the filters may be small
  const long long per_wg = 32 / g.NB, most = (g.NB == 1 ? most_filters<1>() : most_filters<2>()) / (64 * g.NB);
  const long long blocks = (g.K + 64 * g.NB - 1) / (64 * g.NB), shares = (blocks + most - 1) / most;
  const long long work = whole_stores && blocks > most ? blocks : shares * most;
  auto rounds = [&](long long pairs) { return ((pairs + per_wg - 1) / per_wg * work + 256 * most - 1) / (256 * most); };
  return rounds((g.P + 1LL) / 2) < rounds((long long)g.N * g.th * pairs_per_row(g));
}

bool conv_fused_pairs_applicable(const Geo& g) {
  if (g.m != 2 || g.CB != 64 || g.NB > 2 || is_nhwc(g) || is_packed(g)) return false;
  if (g.pad != 1 || g.W % 4 != 0) return false;
  if ((long long)g.N * g.K * g.Ho * g.Wo * 4 >= 0xFFFFFFF0LL) return false;  // 32-bit store offsets
  if ((g.NB == 1 ? lds_bytes<1>(g.K) : lds_bytes<2>(g.K)) > kMaxLds) return false;  // 704 and 768 filters
  const long long npr = pairs_per_row(g);
  return divisions_exact(g.N * g.th * npr, npr, g.th) && reach_bytes(g) < (1LL << 31);
}

hipError_t launch_conv_fused_pairs(const Geo& g, const float* x, const int8_t* uq, const float* u_range,
                                   const int32_t* u_rowsum, const float* partial, int count,
                                   float* v_range, float* y, hipStream_t s) {
  if (!conv_fused_pairs_applicable(g)) return hipErrorInvalidValue;
  const CpArgs a = make_args(g, x, uq, u_range, u_rowsum, partial, count, v_range, y, stores_past_caches(g, true));
  return g.NB == 1 ? launch_blocks<1>(g, a, s) : launch_blocks<2>(g, a, s);
}

// NHWC: 16-byte pixel loads of four channels at 32-bit offsets, 32-bit store offsets; X 16-byte aligned.
bool conv_fused_pairs_nhwc_applicable(const Geo& g) {
  return g.m == 2 && g.CB == 64 && g.NB <= 2 && is_nhwc(g) && !is_packed(g) && g.C % 4 == 0 &&
         (long long)g.N * g.K * g.Ho * g.Wo * 4 < 0xFFFFFFF0LL && (long long)g.N * g.C * g.H * g.W * 4 < 0xFFFFFFF0LL;
}

hipError_t launch_conv_fused_pairs_nhwc(const Geo& g, const float* x, const int8_t* uq, const float* u_range,
                                        const int32_t* u_rowsum, const float* partial, int count,
                                        float* v_range, float* y, bool stream, hipStream_t s) {
  if (!conv_fused_pairs_nhwc_applicable(g) || (reinterpret_cast<uintptr_t>(x) & 15) != 0) return hipErrorInvalidValue;
  const CpArgs a = make_args(g, x, uq, u_range, u_rowsum, partial, count, v_range, y, stream);
  if (g.bits == 8) return stream ? launch_nhwc<true, true>(g, a, s) : launch_nhwc<true, false>(g, a, s);
  return stream ? launch_nhwc<false, true>(g, a, s) : launch_nhwc<false, false>(g, a, s);
}

}  // namespace lance
