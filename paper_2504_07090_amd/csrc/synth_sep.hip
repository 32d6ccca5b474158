// Separable sky synthesis on the RA x sin(dec) grid (Sec. 3.2, eq. fg_separable).
//
// Every pixel sits on a ring j (z_j = sin dec) and a column k (alpha_k), and
// the real harmonic factorises as Y(j, k; l, m) = lambda_l|m|(z_j) T_m(alpha_k)
// with T_0 = 1, T_m = sqrt 2 cos(m alpha), T_-m = sqrt 2 sin(m alpha).  Hence
//     I(j, k, nu) = sum_m T_m(alpha_k) G_m(j, nu),
//     G_m(j, nu)  = sum_{l >= |m|} lambda_l|m|(z_j) a_lm(nu),
// a Legendre stage (one GEMM per m: rings x l x channels) and an azimuthal
// stage (one GEMM per ring: columns x m x channels).  The adjoint runs the
// transposes in reverse order:
//     H_m(j, nu)   = sum_k T_m(alpha_k) dL/dI(j, k, nu),
//     dL/da_lm(nu) = sum_j lambda_l|m|(z_j) H_m(j, nu).
// At lmax 100 on 128 x 384 pixels and 64 channels this is ~0.7e9 MACs per
// direction against 1.7e10 for the dense product with the visible rows of Y,
// and the factor tables take ~3 MB instead of 2 GB.  The Legendre stages run
// every ring; the azimuthal stages run only the 32-column batches of a ring
// that hold a pixel above the horizon at some time.  The forward writes the
// visible pixels into the sky scratch; the adjoint reads dL/dI on the full
// grid, where the adjoint fringe pass writes it (zero at the other pixels).
// All stages run only the rings and batches that hold a pixel of a chunk within
// the beam of the field's widest channel (beam.hpp): the sky elsewhere is not
// read by the forward fringe pass and dL/dI is zero there.
//
// Every GEMM is a grid of 16 x 16 output tiles, one wavefront each, on
// v_mfma_f32_16x16x4_f32: A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k,
// D[i][j] in lane j + 16 (i / 4), register i % 4.  Operands come straight
// from the small, cache-resident tables; K is unrolled so the loads of
// several MFMAs are in flight together.  The azimuthal stages, whose K runs
// over 2 lmax + 1 or nphi, also issue the next batch's loads into a second
// register set before the current batch's MFMAs (the loop is unrolled by two so
// the sets swap roles without copies, and a scheduling barrier keeps the
// batch's loads together); those loads use indices clamped into the tables and
// are always issued (a load under a divergent branch is waited for where the
// branch ends), and terms past the end of K are removed by zeroing one operand
// at the MFMA.
#include "batch.hpp"
#include "beam.hpp"
#include "objects.hpp"

namespace bv {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 sep_mfma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Blocks are dealt round-robin over the 8 XCDs (block b to XCD b % 8).  The
// block's linear index is mapped to a logical one such that each XCD runs one
// contiguous range of logical blocks (the tail that does not fill all eight
// keeps its index): a bijection on [0, blocks).  The adjoint Legendre stage
// decodes it with the blocks of one m adjacent, so that m's table rows come
// from one XCD's L2 instead of being fetched once per XCD.
__device__ __forceinline__ int sep_xcd_logical(const Blk& B) {
  const int total = B.nx * B.ny * B.nz;
  const int b = B.x + B.nx * (B.y + B.ny * B.z);
  const int per = total / 8;
  return b >= 8 * per ? b : (b % 8) * per + b / 8;
}

// (x, y, z) block coordinates of logical block L with y and z fastest.
__device__ __forceinline__ int3 sep_blocks_m_major(int L, const Blk& B) {
  const int nyz = B.ny * B.nz, yz = L % nyz;
  return make_int3(L / nyz, yz % B.ny, yz / B.ny);
}

constexpr int kSepBatch = 8;              // MFMAs whose operand loads are issued together
static_assert(kSepStep == 4 * kSepBatch, "K covered per batch");

// What the stages need to find the rings and batches within the beam.
struct SepBeam {
  const float* fwhm;
  float sigr_max, cut_sig2;
  const float* ring_ex;   // [nz]
  __device__ float cut() const { return beam_cut(cut_sig2, fwhm[0] * sigr_max); }
};

// G[j][c][nu] = sum_{l=|m|}^{lmax} lambda_l|m|(z_j) a[nu][l^2 + l + m],  c = m + lmax,
// for the rings between the first and the last within the beam.  One block per
// (|m|, 16-channel tile), grid (lmax + 1, ceil(nf / 16)): it gathers the
// coefficients of +m and -m into LDS, kLegL degrees at a time, and each wave
// takes 16-ring tiles in turn, one Legendre operand feeding both signs (D rows =
// rings, columns = channels).  In MFMA step q the lanes of group kk = lane / 16
// take l = l0 + 8 kk + q, so every lane reads eight consecutive l of its ring's
// Legendre row (two 16-byte loads), all issued before the gather is waited for.
// Bound by the latency of the gather.  It replaces a transpose of the
// coefficients and a stage reading its rows, one wave per (m, ring tile, channel
// tile): 61 dishes, lmax 100, 64 channels 17.9 -> 15.8 us over two and one
// launches, 19 dishes, lmax 45, 33 channels 13.0 -> 8.9 us.
constexpr int kLegL = 128, kLegWaves = 8;
struct SepLegFwdArgs {
  int nz;
  int nf;
  int nm;
  int lmax;
  int blmax;
  int kaz;
  const float* lam;
  const int* loff;
  const float* alm;
  float* G;
  SepBeam beam;
};

struct KSepLegFwd {
  using Args = SepLegFwdArgs;
  static constexpr int kThreads = 64 * kLegWaves, kWaves = 1;
  static __device__ void run(const SepLegFwdArgs& args_, const Blk& B_);
};

// Row of degree l0 + d of one sign in LDS: 16 channels, every eighth row
// followed by 16 floats so that the four lane groups (rows 8 apart) read
// different banks.
__device__ __forceinline__ int leg_row(int d) { return 16 * (d + (d >> 3)); }

__device__ void KSepLegFwd::run(const SepLegFwdArgs& args_, const Blk& B_) {
  const int nz = args_.nz, nf = args_.nf, lmax = args_.lmax, kaz = args_.kaz;
  const float* __restrict__ alm = args_.alm;
  float* __restrict__ G = args_.G;
  constexpr int kRows = 16 * (kLegL + kLegL / 8);
  __shared__ float as[2][kRows];

  const int am = B_.x, f0 = B_.y * 16, nsign = am > 0 ? 2 : 1;
  const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, kk = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int2 rng = beam_range(args_.beam.ring_ex, nz, args_.beam.cut(), lane);
  const int t0 = rng.x / 16, t1 = rng.y < 0 ? t0 : rng.y / 16 + 1;   // ring tiles
  const int lp = sep_lpad(args_.blmax, am);
  // one round of the block's waves over the ring tiles per pass
  for (int tb = t0; tb < t1; tb += kLegWaves) {
    const int jt = tb + wv, j = min(16 * jt + i, nz - 1);
    const float* lrow = args_.lam + args_.loff[am] + static_cast<size_t>(j) * lp;
    f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
    for (int lb = am; lb <= lmax; lb += kLegL) {
      const int nl = min(kLegL, lmax + 1 - lb);
      // this lane's Legendre operands of every batch, in flight beside the gather
      f4 av[kLegL / kSepStep][2];
#pragma unroll
      for (int h = 0; h < kLegL / kSepStep; ++h) {
        const int dl = lb - am + kSepStep * h + 8 * kk;   // this lane's l - am = dl .. dl + 7
        const bool in = kSepStep * h < nl && dl < lp;     // lp is a multiple of 8: all eight in the row or none
#pragma unroll
        for (int q = 0; q < 2; ++q)
          av[h][q] = in ? *reinterpret_cast<const f4*>(lrow + dl + 4 * q) : f4{0.f, 0.f, 0.f, 0.f};
      }
      if (tb == t0 || lmax + 1 - am > kLegL) {
        // thread (d, q): degree lb + d of slab after slab of 32, channel and sign
        // q, q + 16; all loads issue before the first is stored
        constexpr int kQ = 2 * kLegWaves;   // threads per degree
        const int d = tid & 31, q0 = tid >> 5;
        float v[kLegL / 32][32 / kQ];
#pragma unroll
        for (int h = 0; h < kLegL / 32; ++h)
#pragma unroll
          for (int it = 0; it < 32 / kQ; ++it) {
            const int q = q0 + kQ * it, l = lb + 32 * h + d, f = f0 + (q & 15);
            v[h][it] = 32 * h + d < nl && f < nf && (q >> 4) < nsign
                           ? alm[static_cast<size_t>(f) * args_.nm + l * l + l + ((q >> 4) ? -am : am)] : 0.f;
          }
        __syncthreads();   // the previous contents are read
#pragma unroll
        for (int h = 0; h < kLegL / 32; ++h)
#pragma unroll
          for (int it = 0; it < 32 / kQ; ++it) {
            const int q = q0 + kQ * it;
            as[q >> 4][leg_row(32 * h + d) + (q & 15)] = v[h][it];
          }
        __syncthreads();
      }
      if (jt >= t1) continue;   // uniform over the wave
#pragma unroll
      for (int h = 0; h < kLegL / kSepStep; ++h) {
        if (kSepStep * h >= nl) break;   // uniform
#pragma unroll
        for (int q = 0; q < kSepBatch; ++q) {
          const int o = leg_row(kSepStep * h + 8 * kk + q) + i;
          acc[0] = sep_mfma(av[h][q >> 2][q & 3], as[0][o], acc[0]);
          if (nsign == 2) acc[1] = sep_mfma(av[h][q >> 2][q & 3], as[1][o], acc[1]);
        }
      }
    }
    const int fo = f0 + (lane & 15);
    if (jt >= t1 || fo >= nf) continue;
#pragma unroll
    for (int sg = 0; sg < 2; ++sg) {
      if (sg >= nsign) break;
      const int c = lmax + (sg ? -am : am);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int jo = 16 * jt + 4 * kk + r;
        if (jo < nz) G[(static_cast<size_t>(jo) * kaz + c) * nf + fo] = acc[sg][r];
      }
    }
  }
}

// img[nu][slot(j, k)] = sum_{c < nc} G[j][c][nu] Tt[c + toff][k] for visible pixels
// (nc = 2 lmax + 1 rows of G per ring are used).
// grid (column batches, 1, ceil(nf / 32)): block x takes the batch of x-th
// smallest excess, so those within the beam are a prefix dealt evenly to the
// XCDs; each wave computes a 2 x 2 block of 16 x 16 tiles
// (rows = channels, columns = pixels), so every operand load feeds two MFMAs.
// Wave w of the block takes every fourth batch of K from batch w on; the four
// partial tiles are added in wave order through LDS, one tile by each wave.  The
// batches within the beam are fewer than the SIMDs, so a single wave per block
// waited out its K alone: 61 dishes, lmax 100, 64 channels 18.4 -> 15.5 us, 19
// dishes, lmax 45, 33 channels 11.7 -> 10.1 us.
constexpr int kAzWaves = 4;
struct SepAzFwdArgs {
  int nphi;
  int nf;
  int kaz;
  int nc;
  int toff;
  int tstride;        // row length of Tt (nphi rounded up to whole batches)
  const float* Tt;
  const float* G;
  const int* vidx;
  const int* sorted;
  const float* sorted_ex;
  int nvp;
  float* img;
  SepBeam beam;
};

struct KSepAzFwd {
  using Args = SepAzFwdArgs;
  static constexpr int kThreads = 64 * kAzWaves, kWaves = 1;
  static __device__ void run(const SepAzFwdArgs& args_, const Blk& B_);
};

__device__ void KSepAzFwd::run(const SepAzFwdArgs& args_, const Blk& B_) {
  int nphi = args_.nphi;
  int nf = args_.nf;
  int kaz = args_.kaz;
  int nc = args_.nc;
  int toff = args_.toff;
  const float* Tt = args_.Tt;
  const float* G = args_.G;
  const int* __restrict__ vidx = args_.vidx;
  int nvp = args_.nvp;
  float* __restrict__ img = args_.img;

  __shared__ f4 part[kAzWaves][4][64];
  if (args_.sorted_ex[B_.x] > args_.beam.cut()) return;   // the whole block
  const int first = args_.sorted[B_.x], j = first / nphi, k0 = first - j * nphi, f0 = B_.z * 32;
  const int lane = threadIdx.x & 63, i = lane & 15, kk = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this wave's tile of the sum: rows 16 (wv / 2), columns 16 (wv % 2)
  const int ko = k0 + 16 * (wv & 1) + i;
  const int slot = ko < nphi ? vidx[j * nphi + ko] : -1;
  const bool two = f0 + 16 < nf;   // the second channel tile holds a channel
  const float* grow[2];
  const float* tcol[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    grow[h] = G + static_cast<size_t>(j) * kaz * nf + min(f0 + 16 * h + i, nf - 1);
    tcol[h] = Tt + static_cast<size_t>(toff) * args_.tstride + min(k0 + 16 * h + i, nphi - 1);
  }
  f4 acc[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int g = 0; g < 2; ++g) acc[h][g] = f4{0.f, 0.f, 0.f, 0.f};
  struct Batch {
    float a[kSepBatch][2], b[kSepBatch][2];
  };
  auto load = [&](int c0, Batch& B) {
#pragma unroll
    for (int q = 0; q < kSepBatch; ++q) {
      const int c = min(c0 + 4 * q + kk, nc - 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        B.a[q][h] = grow[h][static_cast<size_t>(c) * nf];
        B.b[q][h] = tcol[h][static_cast<size_t>(c) * args_.tstride];
      }
    }
  };
  auto mma = [&](int c0, const Batch& B) {
#pragma unroll
    for (int q = 0; q < kSepBatch; ++q) {
      const bool ok = c0 + 4 * q + kk < nc;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 1 && !two) break;
        const float av = ok ? B.a[q][h] : 0.f;
#pragma unroll
        for (int g = 0; g < 2; ++g) acc[h][g] = sep_mfma(av, B.b[q][g], acc[h][g]);
      }
    }
  };
  constexpr int kStride = kAzWaves * kSepStep;
  if (wv * kSepStep < nc) {
    Batch B0, B1;
    load(wv * kSepStep, B0);
    for (int c0 = wv * kSepStep; c0 < nc; c0 += 2 * kStride) {
      load(c0 + kStride, B1);
      __builtin_amdgcn_sched_barrier(0);
      mma(c0, B0);
      if (c0 + kStride >= nc) break;
      load(c0 + 2 * kStride, B0);
      __builtin_amdgcn_sched_barrier(0);
      mma(c0 + kStride, B1);
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int g = 0; g < 2; ++g) part[wv][2 * h + g][lane] = acc[h][g];
  __syncthreads();
  if (slot < 0) return;
  f4 v = part[0][wv][lane];
#pragma unroll
  for (int w = 1; w < kAzWaves; ++w) v += part[w][wv][lane];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int fo = f0 + 16 * (wv >> 1) + 4 * kk + r;
    if (fo < nf) img[static_cast<size_t>(fo) * nvp + slot] = v[r];
  }
}

// H[j][c][nu] = sum_k T[k][c + toff] dL/dI[j][nu][k] for c < nc = 2 lmax + 1,
// over the ring's column batches within the beam (dL/dI is zero elsewhere), for
// the rings within it and those between them.  Block b runs on XCD b % 8; ring r
// (in ascending order of excess, so that the rings within the beam are dealt
// evenly) goes to XCD r % 8 with all its c and channel tiles, which share its
// rows; grid 8 ceil(nz / 8) ceil(nc / 32) ceil(nf / 32), each wave computes a 2 x 2 block of 16 x 16 tiles (rows = c, columns =
// channels).  In a group of four MFMA steps, lane group kk supplies columns
// k0 + 4 kk .. + 3 (one per step): the transposed table Tt[c][k] and the
// channel's dL/dI row are both contiguous in k, so each operand value of the
// four steps comes with one 16-byte load.  Rows are tstride (whole batches)
// long and zero beyond nphi in both, so no column needs masking.
struct SepAzAdjArgs {
  int nf;
  int kaz;
  int nc;
  int tstride;
  int toff;
  const float* Tt;
  const float* dfull;
  const int* kb_off;
  const int* kb;
  const float* kb_ex;
  const int* ring;
  int nz;
  int ctiles;         // ceil(nc / 32)
  int per_ring;       // blocks per ring
  float* H;
  SepBeam beam;
};

struct KSepAzAdj {
  using Args = SepAzAdjArgs;
  static constexpr int kThreads = 64, kWaves = 1;
  static __device__ void run(const SepAzAdjArgs& args_, const Blk& B_);
};

__device__ void KSepAzAdj::run(const SepAzAdjArgs& args_, const Blk& B_) {
  const int nf = args_.nf, kaz = args_.kaz, nc = args_.nc, tstride = args_.tstride;
  float* __restrict__ H = args_.H;

  const int lane = threadIdx.x, i = lane & 15, kk = lane >> 4;
  const int s = B_.x >> 3, g8 = s / args_.per_ring, within = s - g8 * args_.per_ring;
  const int r = 8 * g8 + (B_.x & 7);
  if (r >= args_.nz) return;
  const int j = args_.ring[r], ft = within / args_.ctiles;
  const int c0 = (within - ft * args_.ctiles) * 32, f0 = ft * 32;
  const float cut = args_.beam.cut();
  const int kb0 = args_.kb_off[j];
  const int nkb = beam_prefix<1>(args_.kb_ex + kb0, args_.kb_off[j + 1] - kb0, cut, lane);
  if (nkb == 0) {
    const int2 rng = beam_range(args_.beam.ring_ex, args_.nz, cut, lane);
    if (j < rng.x || j > rng.y) return;   // not read by the Legendre stage
  }
  const bool two = f0 + 16 < nf;   // the second channel tile holds a channel
  const float* trow[2];
  const float* drow[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    trow[h] = args_.Tt + static_cast<size_t>(min(c0 + 16 * h + i, nc - 1) + args_.toff) * tstride + 4 * kk;
    drow[h] = args_.dfull + (static_cast<size_t>(j) * nf + min(f0 + 16 * h + i, nf - 1)) * tstride + 4 * kk;
  }
  f4 acc[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int g = 0; g < 2; ++g) acc[h][g] = f4{0.f, 0.f, 0.f, 0.f};
  // one batch: two groups of 16 columns, per group a 16-byte load of each row
  // (h) and each channel (g)
  struct Batch {
    f4 a[2][2], b[2][2];
  };
  auto load = [&](int k0, Batch& B) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        B.a[s][h] = *reinterpret_cast<const f4*>(trow[h] + k0 + 16 * s);
        B.b[s][h] = *reinterpret_cast<const f4*>(drow[h] + k0 + 16 * s);
      }
  };
  auto mma = [&](const Batch& B) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int g = 0; g < 2; ++g)
            if (g == 0 || two) acc[h][g] = sep_mfma(B.a[s][h][q], B.b[s][g][q], acc[h][g]);
  };
  const int* kb = args_.kb + kb0;
  if (nkb > 0) {
    // the batch after the last re-reads the last (always issued, never used)
    auto kb_at = [&](int q) { return kb[min(q, nkb - 1)]; };
    Batch B0, B1;
    load(kb[0], B0);
    for (int q = 0; q < nkb; q += 2) {
      load(kb_at(q + 1), B1);
      __builtin_amdgcn_sched_barrier(0);
      mma(B0);
      if (q + 1 >= nkb) break;
      load(kb_at(q + 2), B0);
      __builtin_amdgcn_sched_barrier(0);
      mma(B1);
    }
  }
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int fo = f0 + 16 * g + (lane & 15);
    if (fo >= nf) continue;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int co = c0 + 16 * h + 4 * kk + r;
        if (co < nc) H[(static_cast<size_t>(j) * kaz + co) * nf + fo] = acc[h][g][r];
      }
  }
}

// grad[nu][l^2 + l + m] = sum_j lambda_l|m|(z_j) H[j][m + lmax][nu], l = |m| .. lmax,
// over the rings between the first and the last within the beam;
// 16 lanes read 16 consecutive l of one ring row of the m-major Legendre table.
// grid (2 lmax + 1, ceil((lmax + 1) / 16), ceil(nf / 16)); D rows = l, columns = channels.
struct SepLegAdjArgs {
  int nz;
  int nf;
  int nm;
  int lmax;
  int blmax;
  int kaz;
  const float* lam;
  const int* loff;
  const float* H;
  float* grad;
  SepBeam beam;
};

struct KSepLegAdj {
  using Args = SepLegAdjArgs;
  static constexpr int kThreads = 64, kWaves = 1;
  static __device__ void run(const SepLegAdjArgs& args_, const Blk& B_);
};

__device__ void KSepLegAdj::run(const SepLegAdjArgs& args_, const Blk& B_) {
  int nz = args_.nz;
  int nf = args_.nf;
  int nm = args_.nm;
  int lmax = args_.lmax;
  int blmax = args_.blmax;
  int kaz = args_.kaz;
  const float* __restrict__ lam = args_.lam;
  const int* __restrict__ loff = args_.loff;
  const float* __restrict__ H = args_.H;
  float* __restrict__ grad = args_.grad;

  const int3 bk = sep_blocks_m_major(sep_xcd_logical(B_), B_);
  const int m = bk.x - lmax, am = m < 0 ? -m : m;
  const int l0 = am + 16 * bk.y, f0 = bk.z * 16;
  if (l0 > lmax) return;
  const int lane = threadIdx.x, i = lane & 15, kk = lane >> 4;
  const int l = min(l0 + i, lmax), f = min(f0 + i, nf - 1);
  const int c = m + lmax;
  const int lp = sep_lpad(blmax, am);
  const float* lcol = lam + loff[am] + (l - am);   // 16 lanes: 16 consecutive l of one ring
  const float* hcol = H + static_cast<size_t>(c) * nf + f;
  f4 acc = f4{0.f, 0.f, 0.f, 0.f};
  const int2 rng = beam_range(args_.beam.ring_ex, nz, args_.beam.cut(), lane);
  for (int jb = rng.x; jb <= rng.y; jb += kSepStep) {
    float a[kSepBatch], b[kSepBatch];
#pragma unroll
    for (int q = 0; q < kSepBatch; ++q) {
      const int j = jb + 4 * q + kk;
      const bool ok = j <= rng.y;
      a[q] = ok ? lcol[static_cast<size_t>(j) * lp] : 0.f;
      b[q] = ok ? hcol[static_cast<size_t>(j) * kaz * nf] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kSepBatch; ++q) acc = sep_mfma(a[q], b[q], acc);
  }
  const int fo = f0 + (lane & 15);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int lo = l0 + 4 * kk + r;
    if (lo <= lmax && fo < nf) grad[static_cast<size_t>(fo) * nm + lo * lo + lo + m] = acc[r];
  }
}

void launch_synth_fwd_sep(const vis_field* f, const float* alm, const float* fwhm, float* img,
                          hipStream_t st) {
  const vis_basis* b = f->basis;
  BV_REQUIRE(b->sep_lam != nullptr, VIS_EINVAL, "basis has no separable factor tables");
  const int L = f->lmax;
  const int toff = b->lmax + kSepPad - L;   // T column of c = 0 (m = -L)
  const SepBeam beam{fwhm, f->sigr_max, f->cut_sig2, f->tab.sep_ring_ex};
  {
    ProfScope ps(&f->prof, "k_sep_leg_fwd", st);
    launch_k<KSepLegFwd>(dim3(L + 1, ceil_div(f->n_freq, 16)), 0,
                         SepLegFwdArgs{b->nz, f->n_freq, f->n_modes, L, b->lmax, f->kaz, b->sep_lam,
                                       b->sep_loff, alm, f->scr.sep_g, beam}, st, "k_sep_leg_fwd");
  }
  ProfScope ps(&f->prof, "k_sep_az_fwd", st);
  dim3 grid(f->sep_nkb, 1, ceil_div(f->n_freq, 32));
  launch_k<KSepAzFwd>(grid, 0, SepAzFwdArgs{b->nphi, f->n_freq, f->kaz, 2 * L + 1, toff, b->nphi_b, b->sep_tt, f->scr.sep_g,
                                    f->tab.vidx, f->tab.sep_sorted, f->tab.sep_sorted_ex, f->nv_pad, img, beam},
                      st, "k_sep_az_fwd");
}

// dL/dI comes in the full-grid scratch sep_dfull, written there by the
// adjoint fringe pass (zero at pixels never above the horizon).
void launch_synth_adj_sep(const vis_field* f, const float* fwhm, float* grad_alm, hipStream_t st) {
  const vis_basis* b = f->basis;
  BV_REQUIRE(b->sep_lam != nullptr, VIS_EINVAL, "basis has no separable factor tables");
  const int L = f->lmax;
  const int toff = b->lmax + kSepPad - L;
  const SepBeam beam{fwhm, f->sigr_max, f->cut_sig2, f->tab.sep_ring_ex};
  {
    ProfScope ps(&f->prof, "k_sep_az_adj", st);
    const int ctiles = ceil_div(2 * L + 1, 32), per_ring = ctiles * ceil_div(f->n_freq, 32);
    launch_k<KSepAzAdj>(dim3(static_cast<unsigned>(round_up(b->nz, 8) * per_ring)), 0,
                        SepAzAdjArgs{f->n_freq, f->kaz, 2 * L + 1, b->nphi_b, toff, b->sep_tt, f->scr.sep_dfull,
                                     f->tab.sep_kb_off, f->tab.sep_kb, f->tab.sep_kb_ex, f->tab.sep_ring, b->nz,
                                     ctiles, per_ring, f->scr.sep_g, beam},
                        st, "k_sep_az_adj");
  }
  ProfScope ps(&f->prof, "k_sep_leg_adj", st);
  dim3 grid(2 * L + 1, ceil_div(L + 1, 16), ceil_div(f->n_freq, 16));
  launch_k<KSepLegAdj>(grid, 0, SepLegAdjArgs{b->nz, f->n_freq, f->n_modes, L, b->lmax, f->kaz, b->sep_lam,
                                     b->sep_loff, f->scr.sep_g, grad_alm, beam}, st, "k_sep_leg_adj");
}

}  // namespace bv
