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
// The transform is repeated by each of the ceil(K / (16*KG)) workgroups of a tile block: the plan
// is for layers that leave the chip idle otherwise (conv_fused_pos_preferred).  Every workgroup reduces
// the records of the range pass for itself, unless that is repeated too often (conv_fused_pos_can_merge).
//
// What bounds it: the chain launch - pixels and ranges from memory (about 2 us) - constants -
// transform - uq fragments - exchange - stores of one workgroup; 6 us for the smallest layers with
// caller-supplied ranges, launch included (N122 16->16 7x7; 19 us before on conv_fused_c16), 11 us
// with the range pass (one 16->16 32x32 image: 24.8 us before).  One image of the 512-channel 14x14
// layer: 21 -> 11.6 us, N13 100->72 37x29 F(4x4): 43 -> 16 us.  By the workgroups' clocks (one image, caller's
// ranges): 512->512 28x28, 208 workgroups, 9 of 14 us are phase T (each compute unit transforms all channels of its
// tiles: vector ALUs and the path from L2, about equally), 0.6 until the pixels are requested, 1 until the
// constants are formed, 1 products, 0.4 sums, 0.6 stores.  What the constants are formed from is requested before
// the pixels, and the filter-side terms are formed once per filter (pos_phases.h): 64->128
// 112x112 12.0 -> 10.1 us, 256->256 56x56 13.8 -> 12.2, 512->512 14x14 12.1 -> 11.6; 160 random layers 1.05 on average.
#pragma once
#include "pos_phases.h"

namespace lance {
namespace pos {

// channel blocks whose codes fit into LDS
template <int M> constexpr int most_blocks() { return M == 2 ? 8 : 3; }

template <int M, int NW, int CPL, int KG, int LOAD, bool CLAMP>
__global__ __launch_bounds__(NW * 64, (M == 2 ? 16 : 12) / 4) void conv_fused_pos_kernel(const CpArgs a) {
  constexpr int E = (M + 2) * (M + 2), NT = NW * 64, PW = E / NW;
  constexpr bool kNhwc = LOAD == kNhwc1 || LOAD == kNhwc4;
  extern __shared__ char smem[];
  const Consts<M> cst(smem);
  char* ring = smem + kConstBytes;
  float* ex = reinterpret_cast<float*>(ring);   // the exchange reuses the code rows
  float* red = reinterpret_cast<float*>(ring);  // so does the reduction of the records

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the filter splits of a tile block are neighbours, so that with several splits each die's L2
  // holds few of them
  const int ky = blockIdx.x % a.nky, p0 = (blockIdx.x / a.nky) * 16, k0 = ky * 16 * KG;
  const int nb = a.NB;
  const unsigned plane = (unsigned)nb * 1024u;  // code rows of one position
  {
    typename Consts<M>::template Early<NT> early(a, a.is_static, tid);
    const Quantizer<M, NW, CPL, LOAD, CLAMP> qz(a, p0, lane, wave);
    qz.run(0, nb, cst.qp, ring, [&]() { cst.template form<NT>(a, a.is_static, early, red, tid); });
  }

  // ---- products: positions wave*PW .., accumulators [position][group of 16 filters] ----
  const int col = lane & 15, kq = lane >> 4;  // fragment row; 16-byte piece of the 64 channels
  const unsigned f_off = (unsigned)col * 64u + (unsigned)((kq ^ swz(col)) * 16);
  v4i acc[PW][1][KG], csum[PW][1];
#pragma unroll
  for (int w = 0; w < PW; w++) {
    csum[w][0] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int kg = 0; kg < KG; kg++) acc[w][0][kg] = v4i{0, 0, 0, 0};
  }
  const UqReader<M, KG> uq(a, k0, col, kq);
  // blocks whose uq fragments are requested together: all that LDS holds, as far as registers go
  constexpr int UB = M == 4 ? 3 : (KG == 4 ? 4 : 8);
  v4i af[UB][KG];
  auto load_batch = [&](int e, int b0) {
#pragma unroll
    for (int u = 0; u < UB; u++)
#pragma unroll
      for (int kg = 0; kg < KG; kg++)
        if (b0 + u < nb) af[u][kg] = uq.load(e, b0 + u, kg);
  };
  load_batch(wave * PW, 0);
  int rs[PW];  // row sums of filter k0 + lane
#pragma unroll
  for (int w = 0; w < PW; w++) rs[w] = load_rowsum<KG>(a, wave * PW + w, k0, lane);
  dev::lds_barrier();  // the codes of all waves are in LDS
#pragma unroll
  for (int w = 0; w < PW; w++) {
    const int e = wave * PW + w;
    for (int b0 = 0; b0 < nb; b0 += UB) {
      if (w > 0 || b0 > 0) load_batch(e, b0);
#pragma unroll
      for (int u = 0; u < UB; u++) {
        if (b0 + u < nb) {
          const v4i bf = *reinterpret_cast<const v4i*>(ring + (unsigned)e * plane + (unsigned)(b0 + u) * 1024u + f_off);
          csum[w][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(uq.ones(), bf, csum[w][0], 0, 0, 0);
#pragma unroll
          for (int kg = 0; kg < KG; kg++)
            acc[w][0][kg] = __builtin_amdgcn_mfma_i32_16x16x64_i8(uq.codes(af[u][kg]), bf, acc[w][0][kg], 0, 0, 0);
        }
      }
    }
  }
  dev::lds_barrier();  // the code rows are free again
#pragma unroll
  for (int w = 0; w < PW; w++) sums_to_lds<KG, 1, kNhwc>(a, cst, wave * PW + w, lane, rs[w], acc[w], csum[w], ex);
  dev::lds_barrier();
  store_patches<M, KG, 1, NT, kNhwc>(a, ex, k0, p0, tid);
}

template <int M, int NW, int CPL, int KG, int LOAD, bool CLAMP>
inline hipError_t launch_one(const CpArgs& a, unsigned grid, size_t lds, hipStream_t s) {
  auto kern = conv_fused_pos_kernel<M, NW, CPL, KG, LOAD, CLAMP>;
  constexpr int kMost = kConstBytes + (KG > most_blocks<M>() ? KG : most_blocks<M>()) * (M + 2) * (M + 2) * 1024;
  const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern), kMost);
  if (e != hipSuccess) return e;
  note_kernel("conv_fused_pos_kernel");
  kern<<<grid, NW * 64, lds, s>>>(a);
  return hipGetLastError();
}

template <int M, int NW, int CPL, int LOAD, bool CLAMP>
inline hipError_t launch_kg(const CpArgs& a, int kg, unsigned grid, size_t lds, hipStream_t s) {
  switch (kg) {
    case 1: return launch_one<M, NW, CPL, 1, LOAD, CLAMP>(a, grid, lds, s);
    case 2: return launch_one<M, NW, CPL, 2, LOAD, CLAMP>(a, grid, lds, s);
    default: return launch_one<M, NW, CPL, 4, LOAD, CLAMP>(a, grid, lds, s);
  }
}

// load: kRowsEdge, kRowsAny, kNhwc1 or (m = 2) kNhwc4; kg: 1, 2 or 4 groups of 16 filters.
template <int M, int NW, bool CLAMP>
inline hipError_t launch(const CpArgs& a, int cpl, int load, int kg, hipStream_t s) {
  constexpr int E = (M + 2) * (M + 2);
  const unsigned grid = (unsigned)((a.P + 15) / 16) * (unsigned)a.nky;
  const size_t lds = kConstBytes + (size_t)(a.NB > kg ? a.NB : kg) * E * 1024;
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
