// The second plan for layers with few tiles: where many channels meet many filters, transforming the
// tiles again in every filter split (conv_fused_pos.h) costs more than a second kernel.
//
//   quant_pos_kernel   one workgroup of four waves per (16 tiles, channel block): range reduction,
//                      transform + quantize into LDS, the code rows from there to vq with 16-byte
//                      stores (1 KB contiguous per position).
//   gemm_pos_kernel    one workgroup per (16*TG tiles, 16*KG filters), wave w the positions w*E/NW ..,
//                      both operands straight from memory into fragments (each is used once per
//                      workgroup); column sums by matrix instructions with ones; then M to LDS, A^T M A
//                      and the stores as in conv_fused_pos.h.
//
// vq here is the workspace's own: codes below 8 bits are unsigned in it (pos_phases.h).
#include "pos_phases.h"

namespace lance {
namespace pos {

template <int M, int CPL, int LOAD, bool CLAMP>
__global__ __launch_bounds__(256, M == 2 ? 4 : 3) void quant_pos_kernel(const CpArgs a) {
  constexpr int E = (M + 2) * (M + 2), NW = 4, NT = 256;
  extern __shared__ char smem[];
  const Consts<M> cst(smem);
  char* ring = smem + kConstBytes;
  float* red = reinterpret_cast<float*>(ring);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int blk = blockIdx.x % a.NB, p0 = (blockIdx.x / a.NB) * 16;
  {
    typename Consts<M>::template Early<NT> early(a, a.is_static, tid);
    const Quantizer<M, NW, CPL, LOAD, CLAMP> qz(a, p0, lane, wave);
    qz.run(blk, 1, cst.qp, ring, [&]() { cst.template form<NT>(a, a.is_static, early, red, tid); });
  }
  dev::lds_barrier();
  const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(a.vq, 0, a.vq_bytes, 0x00020000);
  const int row = lane >> 2, chunk = lane & 3;
  const unsigned src = (unsigned)row * 64u + (unsigned)((chunk ^ swz(row)) * 16);
  const bool tile_ok = p0 + row < a.P;
  const unsigned dst = (unsigned)(p0 + row) * 64u + 16u * chunk;
  for (int e = wave; e < E; e += NW) {  // one KB of one position per wave and turn
    const v4u v = *reinterpret_cast<const v4u*>(ring + e * 1024 + src);
    // (the scalar offset stays the constant 0: see store_row in conv_fused_pairs.hip)
    const unsigned plane = ((unsigned)e * (unsigned)a.NB + (unsigned)blk) * (unsigned)a.P * 64u;
    __builtin_amdgcn_raw_buffer_store_b128(v, res, tile_ok ? plane + dst : kOobY, 0, 0);
  }
}

template <int M, int KG, int TG, bool NHWC>
__global__ __launch_bounds__(M == 2 ? 1024 : 768) void gemm_pos_kernel(const CpArgs a) {
  constexpr int E = (M + 2) * (M + 2), NW = M == 2 ? 16 : 12, NT = NW * 64, PW = E / NW;
  extern __shared__ char smem[];
  const Consts<M> cst(smem);
  float* ex = reinterpret_cast<float*>(smem + kConstBytes);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ky = blockIdx.x % a.nky, p0 = (blockIdx.x / a.nky) * 16 * TG, k0 = ky * 16 * KG;
  const int nb = a.NB, col = lane & 15, kq = lane >> 4;
  typename Consts<M>::template Early<NT> early(a, 1, tid);
  const UqReader<M, KG> uq(a, k0, col, kq);
  unsigned v_off[TG];
#pragma unroll
  for (int t = 0; t < TG; t++) v_off[t] = (unsigned)min(p0 + 16 * t + col, a.P - 1) * 64u + 16u * kq;
  const unsigned v_block = (unsigned)a.P * 64u;

  // blocks requested together, twice: one batch is multiplied while the next is in flight
  constexpr int UB = KG + TG <= 2 ? 4 : (KG + TG == 3 ? 3 : (KG + TG == 4 ? 2 : 1));
  v4i af[UB][KG], bf[UB][TG], an[UB][KG], bn[UB][TG];
  auto request = [&](v4i (&fa)[UB][KG], v4i (&fb)[UB][TG], int e, int b0) {
#pragma unroll
    for (int u = 0; u < UB; u++)
      if (b0 + u < nb) {
#pragma unroll
        for (int t = 0; t < TG; t++)
          fb[u][t] = load_code(a.vq, a.vq_bytes, v_off[t], ((unsigned)e * (unsigned)nb + (unsigned)(b0 + u)) * v_block);
#pragma unroll
        for (int kg = 0; kg < KG; kg++) fa[u][kg] = uq.load(e, b0 + u, kg);
      }
  };
  request(af, bf, wave * PW, 0);
  int rs[PW];  // row sums of filter k0 + lane
#pragma unroll
  for (int w = 0; w < PW; w++) rs[w] = load_rowsum<KG>(a, wave * PW + w, k0, lane);
  v4i acc[PW][TG][KG], csum[PW][TG];
#pragma unroll
  for (int w = 0; w < PW; w++)
#pragma unroll
    for (int t = 0; t < TG; t++) {
      csum[w][t] = v4i{0, 0, 0, 0};
#pragma unroll
      for (int kg = 0; kg < KG; kg++) acc[w][t][kg] = v4i{0, 0, 0, 0};
    }
  cst.template form<NT>(a, 1, early, ex, tid);
#pragma unroll
  for (int w = 0; w < PW; w++) {
    const int e = wave * PW + w;
    for (int b0 = 0; b0 < nb; b0 += UB) {
      const bool more = b0 + UB < nb;
      if (more) request(an, bn, e, b0 + UB);
      else if (w + 1 < PW) request(an, bn, e + 1, 0);
#pragma unroll
      for (int u = 0; u < UB; u++)
        if (b0 + u < nb) {
#pragma unroll
          for (int t = 0; t < TG; t++) {
            csum[w][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(uq.ones(), bf[u][t], csum[w][t], 0, 0, 0);
#pragma unroll
            for (int kg = 0; kg < KG; kg++)
              acc[w][t][kg] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[u][kg], bf[u][t], acc[w][t][kg], 0, 0, 0);
          }
        }
      if (more || w + 1 < PW) {
#pragma unroll
        for (int u = 0; u < UB; u++) {
#pragma unroll
          for (int t = 0; t < TG; t++) bf[u][t] = bn[u][t];
#pragma unroll
          for (int kg = 0; kg < KG; kg++) af[u][kg] = an[u][kg];
        }
      }
    }
  }
#pragma unroll
  for (int w = 0; w < PW; w++) sums_to_lds<KG, TG, NHWC>(a, cst, wave * PW + w, lane, rs[w], acc[w], csum[w], ex);
  dev::lds_barrier();
  store_patches<M, KG, TG, NT, NHWC>(a, ex, k0, p0, tid);
}

template <int M, bool CLAMP>
static hipError_t launch_quant(const CpArgs& a, int load, hipStream_t s) {
  const unsigned grid = (unsigned)((a.P + 15) / 16) * (unsigned)a.NB;
  constexpr int lds = kConstBytes + (M + 2) * (M + 2) * 1024;
  auto go = [&](auto kern) -> hipError_t {
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    note_kernel("quant_pos_kernel");
    kern<<<grid, 256, lds, s>>>(a);
    return hipGetLastError();
  };
  switch (load) {
    case kRowsEdge: return go(quant_pos_kernel<M, 4, kRowsEdge, CLAMP>);
    case kRowsAny: return go(quant_pos_kernel<M, 4, kRowsAny, CLAMP>);
    case kNhwc1: return go(quant_pos_kernel<M, 1, kNhwc1, CLAMP>);
    default:
      if constexpr (M == 2) return go(quant_pos_kernel<M, 4, kNhwc4, CLAMP>);
      return hipErrorInvalidValue;
  }
}

template <int M, int KG, int TG>
static hipError_t launch_gemm(const CpArgs& a, bool nhwc, hipStream_t s) {
  constexpr int E = (M + 2) * (M + 2);
  constexpr size_t lds = kConstBytes + (size_t)E * KG * TG * 1024;
  const unsigned grid = (unsigned)((a.P + 16 * TG - 1) / (16 * TG)) * (unsigned)a.nky;
  auto go = [&](auto kern) -> hipError_t {
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), (int)lds);
    if (e != hipSuccess) return e;
    note_kernel("gemm_pos_kernel");
    kern<<<grid, M == 2 ? 1024 : 768, lds, s>>>(a);
    return hipGetLastError();
  };
  return nhwc ? go(gemm_pos_kernel<M, KG, TG, true>) : go(gemm_pos_kernel<M, KG, TG, false>);
}
}  // namespace pos

// How the product kernel's work is cut: 16*tg tiles x 16*kg filters per workgroup.
struct PosGemmShape {
  int kg, tg;
  long long groups;
};

// The shape with the smallest (rounds of one workgroup per compute unit) x (relative time of a
// workgroup), the times from sweeps over 208 to 512 channels with F(4x4) and 600 to 1024 with F(2x2): a
// workgroup streams its operands through the compute unit's path to L2 (512 -> 512 channels, F(4x4): 12 us
// per round with (1, 1); 448 groups of (1, 1) 45 us for the call, 224 of (2, 1) 39 us).
static PosGemmShape pos_gemm_shape(const Geo& g) {
  static constexpr struct { int kg, tg; double cost; } kShapes[] = {{1, 1, 1.0}, {2, 1, 1.45}, {2, 2, 1.85}};
  PosGemmShape best{1, 1, 0};
  double best_cost = 0.0;
  for (const auto& c : kShapes) {
    const long long groups = ((g.P + 16LL * c.tg - 1) / (16 * c.tg)) * ((g.K + 16 * c.kg - 1) / (16 * c.kg));
    const double cost = (double)((groups + 255) / 256) * c.cost;
    if (best_cost == 0.0 || cost < best_cost) { best = PosGemmShape{c.kg, c.tg, groups}; best_cost = cost; }
  }
  return best;
}

// Layers with more channel blocks than conv_fused_pos keeps in LDS, while one round of workgroups
// covers them (us per call with dynamic ranges, the general plan against this one): F(4x4), 512 -> 512
// channels: N4 14x14 59 -> 31, N8 28x28 57 -> 51, N16 40x40 99 against 142; 208 -> 40: N16 40x40 49 -> 42.
// F(2x2), 1024 -> 256: N3 31x33 45 -> 38; 600 -> 40: N16 28x28 41 against 47.
bool gemm_fused_pos_preferred(const Geo& g) {
  if (g.NB <= (g.m == 2 ? 8 : 3) || is_packed(g) || (long long)g.N * g.C * g.H * g.W * 4 >= 0x7FF00000LL) return false;
  return pos_gemm_shape(g).groups <= 256 && (g.m == 4 || g.P <= 2048);
}

hipError_t launch_quant_pos(const Geo& g, const float* x, const float* u_range, const float* partial,
                            int count, float* v_range, int8_t* vq, hipStream_t s) {
  const bool is_static = (g.flags & LANCE_INPUT_RANGE_STATIC) != 0;
  const pos::CpArgs a{x, nullptr, u_range, nullptr, partial, v_range, nullptr, vq, count,
                      (g.flags & LANCE_RANGE_PER_TENSOR) ? 1 : 0, is_static ? 1 : 0,
                      g.N, g.C, g.H, g.W, g.K, g.pad, g.P, g.th, g.tw, g.Ho, g.Wo, g.bits, g.bits_w,
                      g.NB, g.Q, 0, 1, (unsigned)((size_t)g.N * g.C * g.H * g.W * 4), 0,
                      (unsigned)((size_t)g.E * g.NB * g.P * 64)};
  int load;
  if (is_nhwc(g))
    load = g.m == 2 && g.C % 4 == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0 ? pos::kNhwc4 : pos::kNhwc1;
  else
    load = patch_edge_cols_only(g) ? pos::kRowsEdge : pos::kRowsAny;
  const bool clamp = g.bits < 8;  // as in conv_fused_pos.hip
  if (g.m == 4) return clamp ? pos::launch_quant<4, true>(a, load, s) : pos::launch_quant<4, false>(a, load, s);
  return clamp ? pos::launch_quant<2, true>(a, load, s) : pos::launch_quant<2, false>(a, load, s);
}

hipError_t launch_gemm_pos(const Geo& g, const int8_t* uq, const int8_t* vq, const float* u_range,
                           const int32_t* u_rowsum, float* v_range, float* y, hipStream_t s) {
  const PosGemmShape sh = pos_gemm_shape(g);
  const int nky = (g.K + 16 * sh.kg - 1) / (16 * sh.kg);
  const pos::CpArgs a{nullptr, uq, u_range, u_rowsum, nullptr, v_range, y, const_cast<int8_t*>(vq), 0, 0, 1,
                      g.N, g.C, g.H, g.W, g.K, g.pad, g.P, g.th, g.tw, g.Ho, g.Wo, g.bits, g.bits_w,
                      g.NB, g.Q, 0, nky, 0, (unsigned)((size_t)g.N * g.K * g.Ho * g.Wo * 4),
                      (unsigned)((size_t)g.E * g.NB * g.P * 64)};
  const bool nhwc = is_nhwc(g);
  if (sh.kg == 1) return g.m == 2 ? pos::launch_gemm<2, 1, 1>(a, nhwc, s) : pos::launch_gemm<4, 1, 1>(a, nhwc, s);
  if (sh.tg == 1) return g.m == 2 ? pos::launch_gemm<2, 2, 1>(a, nhwc, s) : pos::launch_gemm<4, 2, 1>(a, nhwc, s);
  return g.m == 2 ? pos::launch_gemm<2, 2, 2>(a, nhwc, s) : pos::launch_gemm<4, 2, 2>(a, nhwc, s);
}

}  // namespace lance
