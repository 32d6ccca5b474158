// Beam cut of the evaluation kernels (kBeamBits): every kernel of a field
// derives the same cut from the beam width on the device and the field's
// cut_sig2, so that what one leaves out no other reads.
#pragma once

#include "objects.hpp"

namespace bv {

// kb of a beam of width sig, B = 2^(-theta^2 kb).  Never below 1e-27, so that the
// marker of a pixel below the horizon or of a slot without one (kBelowHorizon)
// has beam 0 at any width, and theta^2 < pi^2 / 4 beam 1; an undefined width stays so.
__device__ __forceinline__ float beam_kb(float sig) {
  const float kb = 1.0f / (2.0f * sig * sig * static_cast<float>(kLn2));
  return kb < 1e-27f ? 1e-27f : kb;
}

// Excess theta^2 beyond which a beam of width sig is cut.
__device__ __forceinline__ float beam_cut(float cut_sig2, float sig) { return cut_sig2 * sig * sig; }

// Number of leading entries of an ascending excess list up to `cut`; the same
// in every lane.  SEG 64-entry segments load at once.  An undefined cut (NaN)
// cuts nothing.
template <int SEG>
__device__ __forceinline__ int beam_prefix(const float* __restrict__ ex, int n, float cut, int lane) {
  int cnt = 0;
  for (int base = 0; base < n; base += 64 * SEG) {
    float e[SEG];
#pragma unroll
    for (int q = 0; q < SEG; ++q) e[q] = ex[min(base + 64 * q + lane, n - 1)];
    int c = 0;
#pragma unroll
    for (int q = 0; q < SEG; ++q)
      c += __popcll(__ballot(base + 64 * q + lane < n && !(e[q] > cut)));
    cnt += c;
    if (c < 64 * SEG) break;
  }
  return cnt;
}

// First and last entry up to `cut` of an excess list in any order ((n, -1) if
// there is none); the same in every lane.
__device__ __forceinline__ int2 beam_range(const float* __restrict__ ex, int n, float cut, int lane) {
  int2 r = make_int2(n, -1);
  constexpr int kSeg = 2;   // 64-entry segments loaded at once
  for (int base = 0; base < n; base += 64 * kSeg) {
    float e[kSeg];
#pragma unroll
    for (int q = 0; q < kSeg; ++q) e[q] = ex[min(base + 64 * q + lane, n - 1)];
#pragma unroll
    for (int q = 0; q < kSeg; ++q) {
      const unsigned long long in = __ballot(base + 64 * q + lane < n && !(e[q] > cut));
      if (in == 0) continue;
      if (r.y < 0) r.x = base + 64 * q + __builtin_ctzll(in);
      r.y = base + 64 * q + 63 - __builtin_clzll(in);
    }
  }
  return r;
}

// The chunks (64 slots each) within the beam of a field's widest channel, a
// prefix of the field's chunks: the slots whose sky or dL/dI any kernel needs.
struct BeamSlots {
  const float* fwhm;
  float sigr_max, cut_sig2;
  const float* chunk_ex;   // [nchunks], ascending
  int nchunks;
  __device__ __forceinline__ float cut() const { return beam_cut(cut_sig2, fwhm[0] * sigr_max); }
  __device__ __forceinline__ bool outside(int chunk) const { return chunk_ex[chunk] > cut(); }
  __device__ __forceinline__ int slots(int lane) const {
    return kChunk * beam_prefix<8>(chunk_ex, nchunks, cut(), lane);
  }
};
inline BeamSlots beam_slots(const vis_field* f, const float* fwhm) {
  return BeamSlots{fwhm, f->sigr_max, f->cut_sig2, f->tab.chunk_ex, f->n_chunks};
}

}  // namespace bv
