// Map-making: x_hat = D A^H N^-1 y (Sec. 4.3, eq. vis_to_map, eq. map_psf).
//
// A is the beam-and-fringe response with gains (eq. rime_matrix), stacked
// over times and baselines.  Re(A^H y) at the pixels above the horizon is the
// adjoint fringe pass applied to the cotangent y (unique-baseline collapse in
// the gains kernel, then the adjoint fringe kernel, unchanged).  The diagonal
// normalisation D = diag(A^H A)^-1 makes the point-spread function unit on
// its diagonal (N is proportional to the identity, so the noise level
// cancels); the diagonal has the closed form
//     (A^H A)_pp = dOmega^2 sum_t B(p, t)^2 sum_{i<j} |g_i g_j|^2,
// evaluated here per (channel, visible pixel), and
//     sum_{i<j} |g_i g_j|^2 = ((sum |g|^2)^2 - sum |g|^4) / 2.
// Where the response is negligible the ratio only amplifies noise (it grows
// like 1 / B), so pixels whose weight is below kMapWeightFloor times the
// channel's largest weight map to 0, as do pixels never above the horizon.
#include "beam.hpp"
#include "objects.hpp"

namespace bv {

constexpr float kMapWeightFloor = 1e-6f;

// w[f][k] = (A^H A)_pp for visible slot k; one wavefront per (64-pixel chunk,
// kMapChan channels), which share the loads of theta^2 (one channel per wave read
// the 12 MB table of 61 dishes and 60 times once per channel).  cmax[f][chunk] is
// the chunk's largest weight.  Slots without a pixel (k >= nv) get 0: w is the
// sky scratch, whose padding must stay finite, and an undefined width or gain
// makes every weight NaN.  Bound by the exponential's rate: 64 channels 26.5 ->
// 22.6 us.
constexpr int kMapChan = 4;

__global__ void __launch_bounds__(64)
k_map_weight(int nf, int nv, int nvp, int nant, double d_omega, const float* __restrict__ sigr,
             const float* __restrict__ TH2, const int2* __restrict__ chunk_t,
             const float2* __restrict__ gains, const float* __restrict__ fwhm, float* __restrict__ w,
             float* __restrict__ cmax) {
  const int chunk = blockIdx.x, f0 = blockIdx.y * kMapChan, lane = threadIdx.x;
  float kb2[kMapChan];
  double s2[kMapChan], s4[kMapChan];
#pragma unroll
  for (int c = 0; c < kMapChan; ++c) {
    kb2[c] = -2.0f * beam_kb(fwhm[0] * sigr[min(f0 + c, nf - 1)]);
    s2[c] = s4[c] = 0.0;
  }
  for (int a = lane; a < nant; a += 64)
#pragma unroll
    for (int c = 0; c < kMapChan; ++c) {
      const float2 g = gains[static_cast<size_t>(min(f0 + c, nf - 1)) * nant + a];
      const double m2 = static_cast<double>(g.x) * g.x + static_cast<double>(g.y) * g.y;
      s2[c] += m2;
      s4[c] += m2 * m2;
    }
  const int k = chunk * kChunk + lane;
  const int2 tr = chunk_t[chunk];
  // sum of B^2 = 2^(-2 theta^2 kb) over the visible times: four independent
  // partial sums so four loads are in flight; the hardware exponential
  // (a square below 2^-126 adds nothing to the weight)
  float sb[kMapChan][4] = {};
  int t = tr.x;
  for (; t + 3 <= tr.y; t += 4) {
    float th2[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) th2[q] = TH2[static_cast<size_t>(t + q) * nvp + k];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < kMapChan; ++c) sb[c][q] += __builtin_amdgcn_exp2f(kb2[c] * th2[q]);
  }
#pragma unroll
  for (int q = 0; q < 3; ++q)
    if (t + q <= tr.y) {
      const float th2 = TH2[static_cast<size_t>(t + q) * nvp + k];
#pragma unroll
      for (int c = 0; c < kMapChan; ++c) sb[c][q] += __builtin_amdgcn_exp2f(kb2[c] * th2);
    }
#pragma unroll
  for (int c = 0; c < kMapChan; ++c) {
    if (f0 + c >= nf) break;   // uniform
    double a2 = s2[c], a4 = s4[c];
    for (int o = 32; o >= 1; o >>= 1) {
      a2 += __shfl_xor(a2, o);
      a4 += __shfl_xor(a4, o);
    }
    const float sbt = (sb[c][0] + sb[c][1]) + (sb[c][2] + sb[c][3]);
    float wt = k < nv ? static_cast<float>(d_omega * d_omega * (0.5 * (a2 * a2 - a4)) * sbt) : 0.f;
    w[static_cast<size_t>(f0 + c) * nvp + k] = wt;
    for (int o = 32; o >= 1; o >>= 1) wt = fmaxf(wt, __shfl_xor(wt, o));
    if (lane == 0) cmax[static_cast<size_t>(f0 + c) * gridDim.x + chunk] = wt;
  }
}

// map[f][p] = dimg[f][slot] / w[f][slot] where w >= floor * the channel's largest
// weight, else 0.  Grid (ceil(npix / (256 kMapPix)), nf); every block takes the
// maximum of its channel's chunks itself (a few values per thread), which a launch
// between this one and the weights did before (10 us of the 61-dish map).
constexpr int kMapPix = 4;

__global__ void __launch_bounds__(256)
k_map_finish(int npix, int nvp, int nchunks, const int* __restrict__ vidx, const float* __restrict__ dimg,
             const float* __restrict__ w, const float* __restrict__ cmax, float* __restrict__ map,
             float* __restrict__ weight) {
  __shared__ float red[4];
  const int f = blockIdx.y, tid = threadIdx.x;
  float m = 0.f;
  for (int c = tid; c < nchunks; c += 256) m = fmaxf(m, cmax[static_cast<size_t>(f) * nchunks + c]);
  for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if ((tid & 63) == 0) red[tid >> 6] = m;
  __syncthreads();
  const float wm = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
#pragma unroll
  for (int q = 0; q < kMapPix; ++q) {
    const int p = (blockIdx.x * kMapPix + q) * 256 + tid;
    if (p >= npix) break;
    const int slot = vidx[p];
    float x = 0.f, wt = 0.f;
    if (slot >= 0) {
      wt = w[static_cast<size_t>(f) * nvp + slot];
      if (wt > 0.f && wt >= kMapWeightFloor * wm) x = dimg[static_cast<size_t>(f) * nvp + slot] / wt;
    }
    const size_t idx = static_cast<size_t>(f) * npix + p;
    map[idx] = x;
    if (weight != nullptr) weight[idx] = wt;
  }
}

void launch_map_finish(const vis_field* f, const vis_c64* gains, const float* fwhm, float* map,
                       float* weight, hipStream_t st) {
  // the sky scratch is free after the adjoint fringe pass: it holds the
  // weights; the F-gradient partials (not needed here) the chunks' maxima
  float* w = f->scr.img;
  float* cmax = f->scr.f_part;
  {
    ProfScope ps(&f->prof, "k_map_weight", st);
    k_map_weight<<<dim3(f->n_chunks, ceil_div(f->n_freq, kMapChan)), 64, 0, st>>>(
        f->n_freq, f->nv, f->nv_pad, f->n_ant, f->d_omega, f->tab.sigr, f->tab.th2,
        f->tab.chunk_t, reinterpret_cast<const float2*>(gains), fwhm, w, cmax);
    check_launch("k_map_weight");
  }
  const int npix = f->basis->n_pix;
  ProfScope ps(&f->prof, "k_map_finish", st);
  k_map_finish<<<dim3(ceil_div(npix, 256 * kMapPix), f->n_freq), 256, 0, st>>>(
      npix, f->nv_pad, f->n_chunks, f->tab.vidx, f->scr.dimg, w, cmax, map, weight);
  check_launch("k_map_finish");
}

}  // namespace bv
