// Forward and adjoint fringe contractions of the discrete RIME on MFMA.
//
// Sec. 2.1, eq. rime_discrete: V_u(nu, t) = sum_p S_p exp(-2 pi i nu b_u . s_p(t) / c)
// with S = dOmega B I, evaluated once per redundant baseline u (Sec. 3.1).
//
// Lattice factorisation.  Antennas sit on a lattice, so every unique baseline
// is b_u = n1 e1 + n2 e2 with integers 0 <= n1 <= D, |n2| <= D, and the fringe
// factorises exactly:
//     exp(-2 pi i nu b_u . s / c) = alpha^n1 beta^n2,
//     alpha = exp(-2 pi i x1), x1 = nu (e1 . s) / c,  beta likewise with e2.
// Writing beta^m S = c + i d and alpha^n = a_r + i a_i, the four real sums
//     P1 = sum a_r c,  P2 = sum a_i d,  P3 = sum a_r d,  P4 = sum a_i c
// give both signs of n2 at once:
//     V(n, +m) = (P1 - P2) + i (P3 + P4),   V(n, -m) = (P1 + P2) + i (P4 - P3).
// For each (nu, t) the P's for n, m in 1..D form one real GEMM
//     P[2D x 2D] = A[2D x pixels] Bm[pixels x 2D]
// (rows (n, Re/Im alpha^n), columns (m, Re/Im beta^m S)), run on MFMA with
// the pixels as the contraction dimension; the axis baselines n = 0 or m = 0
// are plain sums taken on the vector ALU.  The fringe x beam tiles exist only
// in registers and LDS; nothing of size pixels x baselines touches HBM.
//
// Phase accuracy: x = nu (e . s) / c comes from tables reduced modulo one cycle
// in FP64 (phase_cycles), and the powers alpha^n, n <= D, from two chains of the
// three-term recurrence (lattice_powers).  A rounding error made at step k of a
// chain reaches step j multiplied by sin((j - k) 2t) / sin(2t), at most j - k in
// size, so the error of alpha^n stays below about n^2 / 8 FP32 roundings (8 at
// n = 8).  The split kernels take one chain (StepChain): n^2 / 2, 72 roundings
// or 4e-6 at n = 12 and 8e-6 at n = 16, against bounds of 1e-4 on what they form.
//
// The adjoint (transpose over the reals) of the same map, for coefficients
// omega_u = dL/dRe V_u - i dL/dIm V_u (formed by the gains pass), is
//     Z_p = sum_u Re[omega_u alpha^n1 beta^n2]
//         = sum_{r,c} A[r][p] G[r][c] Bb[p][c] + axis terms,
// with G built from omega(n, +m), omega(n, -m); it runs as the GEMM
// T[r][p] = sum_c G[r][c] Bb[c][p] on MFMA followed by a per-pixel dot with A.
// dL/dI(p, nu) = dOmega sum_t B Z and dL/dF = dOmega sum (dB/dF) I Z follow.
#pragma once

#include "batch.hpp"
#include "beam.hpp"
#include "objects.hpp"

namespace bv {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// sin and cos of 2 pi x on the hardware units, which take their argument in
// turns; BV_ACCURATE_TRIG selects the correctly-rounded library routine instead.
__device__ __forceinline__ void sincos_rev(float x, float& s, float& c) {
#ifdef BV_ACCURATE_TRIG
  sincospif(2.0f * (x - __builtin_rintf(x)), &s, &c);
#else
  s = __builtin_amdgcn_sinf(x);
  c = __builtin_amdgcn_cosf(x);
#endif
}

// 2^x on the hardware exponential unit (no denormal-range rescaling: the
// beam factors it forms are only ever weights, and one below 2^-126 adds
// nothing to a sum of beam-weighted terms).
__device__ __forceinline__ float beam_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Element k of a per-wave array through a 32-bit byte offset (the base is
// uniform over the wave, so the load takes the scalar-base form and no
// per-lane 64-bit address arithmetic is needed).
template <class V>
__device__ __forceinline__ V at_u32(const V* base, int k) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) +
                                     static_cast<uint32_t>(k) * static_cast<uint32_t>(sizeof(V)));
}

// A lane's elements of (uniform) rows in a loop over rows.  ROW: the byte
// offsets look changed in every iteration (`touch` issues no instruction), so
// that the row's address is formed on the scalar unit; otherwise the optimizer
// adds the lane to the array's base once, outside, and pays a 64-bit vector add
// per load.  The vector adds cost more than the scalar ones where the vector
// unit is the shorter chain (extents up to 6: 8 of 57 vector instructions per
// chunk of a 37-dish forward pass, 205 -> 196 us; the adjoint 210 -> 207 us),
// less above (91 dishes, adjoint 334 us against 339 us with ROW).
template <bool ROW>
struct LaneOffset {
  uint32_t o4, o8;
  __device__ explicit LaneOffset(int lane) : o4(4u * lane), o8(8u * lane) {}
  __device__ __forceinline__ void touch(int row) {
    if constexpr (ROW) asm("" : "+v"(o4), "+v"(o8) : "s"(row));
  }
  __device__ __forceinline__ float at(const float* row) const {
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + o4);
  }
  __device__ __forceinline__ float2 at(const float2* row) const {
    return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(row) + o8);
  }
};

// Phase of nu_f p in cycles, modulo whole cycles, in FP32 from the table entry
// q = (y, p), y = nu_c p reduced modulo 1 on the host in FP64, and dnu = nu_f -
// nu_c: x = y + dnu p, one fma.  The hardware sine and cosine take an argument
// of up to 256 turns and reduce it exactly (errors on [-2, 2] as on [-1/2, 1/2],
// measured; at 30, 150 and 230 turns the visibilities follow the rounding of x
// itself, as they do reduced at 400), so only fields whose |x| may exceed kMaxTurns
// (WRAP: a lattice step of a kilometre over a half band of 75 MHz) reduce it here;
// the two instructions per axis cost 3% of both passes.
constexpr float kMaxTurns = 240.0f;
template <bool WRAP>
__device__ __forceinline__ float phase_cycles(float dnu, float2 q) {
  const float x = __builtin_fmaf(dnu, q.y, q.x);
  return WRAP ? x - __builtin_rintf(x) : x;
}

// Block index -> logical index so that consecutive logical indices share an
// XCD (the dispatcher deals blocks round-robin over the 8 XCDs; consecutive
// logical work items reuse the same geometry rows from that XCD's L2).
__device__ __forceinline__ int xcd_logical(int bid, int nblocks) {
  const int per = (nblocks + 7) >> 3;
  return (bid & 7) * per + (bid >> 3);
}

// Logical index L -> (outer o, inner i) of an n_o x n_i grid, visited in
// tiles of to outers x ti inners (outer-major inside a tile), so that the
// blocks resident on one XCD at a time share few outer and few inner rows
// (geometry rows per outer, image or coefficient rows per inner) and both fit
// its L2.  A bijection for L < n_o n_i.
__device__ __forceinline__ void tile_map(int L, int n_o, int n_i, int to, int ti, int& o, int& i) {
  const int og = L / (to * n_i), o0 = og * to, tog = min(to, n_o - o0);
  int local = L - og * to * n_i;
  const int ig = local / (tog * ti), i0 = ig * ti, tig = min(ti, n_i - i0);
  local -= ig * tog * ti;
  o = o0 + local / tig;
  i = i0 + local % tig;
}

template <int D>
struct Tile {
  static constexpr int RT = (2 * D + 15) / 16;  // 16-wide MFMA tiles per side
  static constexpr int W = 16 * RT;             // padded side = LDS row length (floats)
};

// LDS layout of the per-pixel operand rows: row px holds W floats as W/4
// groups of 4; logical group g sits at physical group g ^ swz(px).  The
// swizzle makes a wavefront's 128-bit row writes hit every bank group evenly
// and keeps the MFMA operand reads (16 consecutive columns of one row per
// 16 lanes, the next row in the next 16 lanes) free of bank conflicts.
template <int W>
__device__ __forceinline__ int swz(int px) {
  return W == 16 ? ((px >> 1) & 3) : (((px & 1) << 2) | ((px >> 1) & 3));
}
template <int W>
__device__ __forceinline__ int lds_at(int px, int col) {
  return px * W + ((((col >> 2) ^ swz<W>(px))) << 2) + (col & 3);
}

// w a^n, n = 1..D, of a = exp(-i t) from c = cos t, s = sin t, into re[n], im[n]:
// two interleaved chains of step a^2, u_{n+2} = 2 cos(2t) u_n - u_{n-2} (the
// three-term recurrence of cos(n t) and sin(n t)), one FMA per component.  A
// rounding error grows over n / 2 steps instead of the n of a chain of step a.
// cos(2t) comes from the smaller of |s| and |c|, which the hardware unit gives
// with the smaller absolute error (2.3e-8 against 4.6e-8 rms, measured) and
// whose square damps it further.
template <int D>
__device__ __forceinline__ void lattice_powers(float c, float s, float w, float* re, float* im) {
  const bool small_s = fabsf(s) < fabsf(c);
  const float m = small_s ? s : c;
  const float h = __builtin_fmaf(-2.f * m, m, 1.f), c2 = small_s ? h : -h, t = 2.f * c2;
  re[1] = c * w;
  im[1] = -s * w;
  re[2] = c2 * w;
  im[2] = -2.f * s * re[1];
#pragma unroll
  for (int n = 3; n <= D; ++n) {
    // u_{-1} = conj(u_1), u_0 = w
    re[n] = t * re[n - 2] - (n == 3 ? re[1] : n == 4 ? w : re[n - 4]);
    im[n] = t * im[n - 2] - (n == 3 ? -im[1] : n == 4 ? 0.f : im[n - 4]);
  }
}

// Powers alpha^n (n = 1..D) and beta^m w (m = 1..D) of one pixel into av, bv;
// visit(n, alpha^(n+1), beta^(n+1) w) sees every power while it is still in
// registers.
template <int D, class Visit>
__device__ __forceinline__ void powers_f32(float* av, float* bv, float c1, float s1, float c2,
                                           float s2, float w, Visit visit) {
  float ar[D + 1], ai[D + 1], br[D + 1], bi[D + 1];
  lattice_powers<D>(c1, s1, 1.f, ar, ai);
  lattice_powers<D>(c2, s2, w, br, bi);
#pragma unroll
  for (int n = 0; n < D; ++n) {
    av[2 * n] = ar[n + 1];
    av[2 * n + 1] = ai[n + 1];
    bv[2 * n] = br[n + 1];
    bv[2 * n + 1] = bi[n + 1];
    visit(n, ar[n + 1], ai[n + 1], br[n + 1], bi[n + 1]);
  }
}
template <int W>
__device__ __forceinline__ void store_rows(float* As, float* Bs, int px, const float* av, const float* bv) {
#pragma unroll
  for (int g = 0; g < W / 4; ++g) {
    const int o = px * W + ((g ^ swz<W>(px)) << 2);
    *reinterpret_cast<f4*>(As + o) = f4{av[4 * g], av[4 * g + 1], av[4 * g + 2], av[4 * g + 3]};
    *reinterpret_cast<f4*>(Bs + o) = f4{bv[4 * g], bv[4 * g + 1], bv[4 * g + 2], bv[4 * g + 3]};
  }
}
// ------------------------------------------------- split-precision helpers --
// Split-precision fields run the fringe products on FP16 MFMA as hi + lo
// pairs (x ~ hi + lo, hi = fp16(x), lo = fp16(x - hi)), three products
// hi hi + hi lo + lo hi accumulated in FP32: about 22 significant bits per
// product instead of FP32's 24, at a sixth of the matrix-core time.
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma_h32(h8 a, h8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma_h16(h4 a, h4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
}

// hi halves of (x0, x1) packed into one register (round toward zero; the lo
// half carries the rest exactly enough either way)
__device__ __forceinline__ uint32_t split_hi2(float x0, float x1) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(x0, x1));
}
// lo halves fp16(x0 - hi0), fp16(x1 - hi1): one mixed-precision FMA each
// (hi read as FP16 from its half of `hi`, the difference rounded once to
// FP16 into the low or high half of the result)
__device__ __forceinline__ uint32_t split_lo2(float x0, float x1, uint32_t hi) {
  uint32_t r;
  asm("v_fma_mixlo_f16 %0, %2, -1.0, %1 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(x0), "v"(hi));
  asm("v_fma_mixhi_f16 %0, %2, -1.0, %1 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
      : "+v"(r) : "v"(x1), "v"(hi));
  return r;
}

// LDS layout of the split B operand of the adjoint (32-bit words).  The hi
// halves: rows of W halves padded to BH words, so that the 16-byte operand
// reads of consecutive pixel rows fall on distinct banks.  The lo halves: W/4
// planes of 64 rows x 8 bytes (plane q = halves 4q .. 4q + 3 of every row),
// planes BLP words apart; a K = 16 operand read takes one plane per 16 lanes
// (128 contiguous bytes), and BLP = 128 + 32 words puts the next plane on the
// other half of the banks.
template <int W> struct SplitRows {
  static constexpr int BH = W / 2 + 4;
  static constexpr int BLP = 64 * 2 + 32;
  static constexpr int BL_WORDS = (W / 4) * BLP;
};

// The split kernels, whose operands keep 22 bits, take the plain recurrence of
// step a, a^(n+1) = 2 cos(t) a^n - a^(n-1), which needs only the last two powers
// in registers (lattice_powers there measured 8% slower at D = 12, every chunk
// within the beam: 91 dishes, 106 channels, 12 times 432 against 400 us
// forward, 490 against 479 us adjoint).
struct StepChain {
  float re0, im0, re, im, t;
  __device__ StepChain(float c, float s, float w) : re0(w), im0(0.f), re(c * w), im(-s * w), t(2.f * c) {}
  __device__ void next() {
    const float nr = t * re - re0, ni = t * im - im0;
    re0 = re; im0 = im; re = nr; im = ni;
  }
};

// Powers of one pixel for the split adjoint: alpha^n in FP32 (as powers_f32),
// beta^m as FP16 hi + lo pairs.
template <int D, class Visit>
__device__ __forceinline__ void powers_split_adj(float* av, uint32_t* bh, uint32_t* bl, float c1,
                                                 float s1, float c2, float s2, Visit visit) {
  StepChain a(c1, s1, 1.f), b(c2, s2, 1.f);
#pragma unroll
  for (int n = 0; n < D; ++n) {
    av[2 * n] = a.re;
    av[2 * n + 1] = a.im;
    bh[n] = split_hi2(b.re, b.im);
    bl[n] = split_lo2(b.re, b.im, bh[n]);
    visit(n, a.re, a.im, b.re, b.im);
    a.next();
    b.next();
  }
}
template <int W>
__device__ __forceinline__ void store_rows_split_adj(float* As, uint32_t* Bh, uint32_t* Bl, int px,
                                                     const float* av, const uint32_t* bh,
                                                     const uint32_t* bl) {
  using R = SplitRows<W>;
#pragma unroll
  for (int g = 0; g < W / 4; ++g) {
    const int o = px * W + ((g ^ swz<W>(px)) << 2);
    *reinterpret_cast<f4*>(As + o) = f4{av[4 * g], av[4 * g + 1], av[4 * g + 2], av[4 * g + 3]};
  }
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int g = 0; g < W / 8; ++g)
    *reinterpret_cast<u4*>(Bh + px * R::BH + 4 * g) = u4{bh[4 * g], bh[4 * g + 1], bh[4 * g + 2], bh[4 * g + 3]};
#pragma unroll
  for (int g = 0; g < W / 4; ++g)
    *reinterpret_cast<u2*>(Bl + g * R::BLP + 2 * px) = u2{bl[2 * g], bl[2 * g + 1]};
}
// Forward split rows: each pixel row holds W halves (W / 2 words, pairs
// (Re, Im) of one power) in 16-byte groups, group g stored at g ^ swz_h(px)
// so that a wavefront's 16-byte row writes spread over the banks; four
// consecutive rows (4 aligned to 4) share the swizzle, which is what the
// transposing operand reads below assume.
template <int W>
__device__ __forceinline__ int swz_h(int px) {
  return W == 16 ? ((px >> 2) & 1) : ((px >> 2) & 3);
}
// Physical row of pixel row px.  A transposing operand read takes four whole
// consecutive rows per 16 lanes; with 32-byte rows (W = 16) the next 16 lanes'
// rows lie 256 bytes further, on the same banks.  Swapping the two halves of
// every odd 8-row block puts those rows on the other half of the banks (for
// W = 32 the swizzle above already separates them).  With it, the 16-byte
// row writes of rows px and px + 4 (and of a row and its swapped partner)
// land in different halves of their 32-byte rows through swz_h.
template <int W>
__device__ __forceinline__ int row_h(int px) {
  return W == 16 ? (px ^ (((px >> 3) & 1) << 2)) : px;
}

// Powers of one pixel for the split forward: alpha^n and beta^m w as FP16
// hi + lo pairs (one word per complex power) into ah, al (alpha) and bh, bl
// (beta); visit(n, ...) sees the FP32 values (beta^m w as generated, w
// already scaled).  store_rows_split writes a pixel's words to its rows of
// Ah, Al, Bh, Bl.
template <int D, class Visit>
__device__ __forceinline__ void powers_split_fwd(uint32_t* ah, uint32_t* al, uint32_t* bh, uint32_t* bl,
                                                 float c1, float s1, float c2, float s2, float w,
                                                 Visit visit) {
  StepChain a(c1, s1, 1.f), b(c2, s2, w);
#pragma unroll
  for (int n = 0; n < D; ++n) {
    ah[n] = split_hi2(a.re, a.im);
    al[n] = split_lo2(a.re, a.im, ah[n]);
    bh[n] = split_hi2(b.re, b.im);
    bl[n] = split_lo2(b.re, b.im, bh[n]);
    visit(n, a.re, a.im, b.re, b.im);
    a.next();
    b.next();
  }
}
template <int W>
__device__ __forceinline__ void store_rows_split(uint32_t* Ah, uint32_t* Al, uint32_t* Bh, uint32_t* Bl,
                                                 int px, const uint32_t* ah, const uint32_t* al,
                                                 const uint32_t* bh, const uint32_t* bl) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int g = 0; g < W / 8; ++g) {
    const int o = row_h<W>(px) * (W / 2) + ((g ^ swz_h<W>(px)) << 2);
    *reinterpret_cast<u4*>(Ah + o) = u4{ah[4 * g], ah[4 * g + 1], ah[4 * g + 2], ah[4 * g + 3]};
    *reinterpret_cast<u4*>(Al + o) = u4{al[4 * g], al[4 * g + 1], al[4 * g + 2], al[4 * g + 3]};
    *reinterpret_cast<u4*>(Bh + o) = u4{bh[4 * g], bh[4 * g + 1], bh[4 * g + 2], bh[4 * g + 3]};
    *reinterpret_cast<u4*>(Bl + o) = u4{bl[4 * g], bl[4 * g + 1], bl[4 * g + 2], bl[4 * g + 3]};
  }
}

// One K = 32 FP16 MFMA operand (eight consecutive pixels of one row or
// column per lane) of 16-column tile `tile` from rows stored pixel-major:
// lane l (index j = l & 15 in its group, group g = l >> 4) needs values
// [pix0 + 8 g .. + 7][16 tile + j].  ds_read_b64_tr_b16 gives lane j of a
// 16-lane group element (j & 3) of the 4-half chunk addressed by lane
// 4 k + (j >> 2), for k = 0..3; so lane j addresses row pix0 + 8 g + 4 h +
// (j >> 2), halves 16 tile + 4 (j & 3) .. + 3, and the two reads (h = 0, 1)
// give its eight pixels in order.
typedef short s4 __attribute__((ext_vector_type(4)));
template <int W>
__device__ __forceinline__ h8 tr_operand(const uint32_t* base, int pix0, int tile, int lane) {
  const int j = lane & 15, g = lane >> 4;
  const int row0 = pix0 + 8 * g + (j >> 2);
  const int col = 16 * tile + 4 * (j & 3);                 // halves
  const int grp = col >> 3, within = (col & 7) >> 1;       // 16-byte group, word in group
  s4 v[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = row0 + 4 * h;
    const uint32_t* a = base + row_h<W>(row) * (W / 2) + ((grp ^ swz_h<W>(row)) << 2) + within;
    v[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s4*)(reinterpret_cast<uintptr_t>(a)));
  }
  typedef short s8 __attribute__((ext_vector_type(8)));
  const s8 c = s8{v[0][0], v[0][1], v[0][2], v[0][3], v[1][0], v[1][1], v[1][2], v[1][3]};
  return __builtin_bit_cast(h8, c);
}

// Per-channel power-of-two scale of the split forward's beam-weighted sky.
// k_chan_scale writes the maximum |I| of each of kScaleParts segments of a
// channel's row; the forward kernel turns the channel's maxima into
// scale = 2^(13 - e) with dOmega max |I| < 2^e (B <= 1), so that every
// |dOmega B I scale| < 2^13 and its FP16 lo part stays a normal number.
struct ChanScaleArgs {
  int nvp;
  BeamSlots beam;
  const float* img;
  float* part;   // [n_freq][kScaleParts]
};

struct KChanScale {
  using Args = ChanScaleArgs;
  static constexpr int kThreads = 256, kWaves = 1;
  static __device__ void run(const ChanScaleArgs& a, const Blk& B) {
    __shared__ float red[4];
    // the slots the forward pass visits (the sky elsewhere is not current)
    const int ns = a.beam.slots(threadIdx.x & 63);
    const int seg = (ns + kScaleParts - 1) / kScaleParts;
    const int k0 = B.y * seg, k1 = min(ns, k0 + seg);
    const float* row = a.img + static_cast<size_t>(B.x) * a.nvp;
    float m = 0.f;
    for (int k = k0 + threadIdx.x; k < k1; k += 256) m = fmaxf(m, fabsf(row[k]));
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0)
      a.part[B.x * kScaleParts + B.y] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  }
};

__device__ __forceinline__ float chan_scale(const float* part, int f, float d_omega) {
  float mx = 0.f;
#pragma unroll
  for (int q = 0; q < kScaleParts; ++q) mx = fmaxf(mx, part[f * kScaleParts + q]);
  mx *= d_omega;
  float sc = 1.0f;
  if (mx > 0.f && isfinite(mx)) {
    int e;
    frexpf(mx, &e);   // mx < 2^e
    sc = ldexpf(1.0f, max(-100, min(100, 13 - e)));
  }
  return sc;
}

// ------------------------------------------------------------------ forward --
// One block of kFwdWaves wavefronts per (t, nu) (per (t, group of stacked
// channels) for D <= 4, see fwd_channels_per_tile); wave w takes every
// kFwdWaves-th pixel chunk within the beam at t (kBeamBits), starting at chunk
// w, and the block adds the waves' partial tiles in a fixed order at the end.  Splitting a
// (t, nu) over the four SIMDs of a CU balances the SIMDs: with one wave per
// (t, nu), a 61-dish field's 3840 waves over 1024 SIMDs leave a quarter of
// the SIMDs with 4 waves and the rest with 3, and the kernel lasts as long
// as the busiest.  Software pipeline per chunk: the MFMA operands of chunk k
// are read from LDS into registers, then the 16 MFMAs of chunk k are
// interleaved with the vector-ALU generation of the wave's next chunk
// (written to LDS); geometry is loaded two of the wave's chunks ahead.  Four
// resident waves per SIMD (<= 128 VGPRs) for extents up to 8.  Bound by issue
// (FP32 MFMA and vector ALU take turns).  Visiting only the chunks within the
// beam leaves 27% of the (chunk, time) pairs above the horizon at 61 dishes, 64
// channels, 60 times, a 10 deg beam: 0.606 -> 0.178 ms (0.162 at the same time
// per chunk; the rest is the start and end of each block).  With a 35 deg beam,
// where every chunk is within it, the pass is about as fast as without the cut
// (37 dishes, 40 channels, 30 times: 0.200 and 0.195 ms).
constexpr int kFwdWaves = 4;

struct FwdArgs {
  int nf, nt, nvp, nubl;
  float d_omega, cut_sig2;
  const float* dnu;
  const float* sigr;
  const float2* Q1;
  const float2* Q2;
  const float* TH2;
  const int* tchunk_off;
  const int* tchunk;
  const float* tchunk_ex;
  const int2* ubl_nm;
  const float* img;
  const float* fwhm;
  float2* vu;
  const float* cscale;   // SPLIT: [n_freq][kScaleParts] segment maxima of |I|
};

// Channels that share one 16 x 16 tile: a lattice extent D fills 2D of the
// tile's rows and columns, so for D <= 4 the rows and columns of 16 / (2D)
// channels are stacked and the tile's diagonal blocks are their P matrices
// (the off-diagonal blocks pair one channel's alpha with another's beta and
// are not read).  The MFMA work is shared; the generation is per channel.
__host__ __device__ constexpr int fwd_channels_per_tile(int D) { return 2 * D <= 8 ? 16 / (2 * D) : 1; }
// Extents whose 2 D operand rows leave a one-channel tile a free row and
// column (D = 6, 12): a row of ones in A and a column of the pixel weight w in
// B make the tile form the axis sums sum_p w beta^m (row 2 D) and
// sum_p w alpha^n (column 2 D) in the padding the MFMAs compute anyway.
__host__ __device__ constexpr bool fwd_axis_in_tile(int D) {
  return fwd_channels_per_tile(D) == 1 && 2 * D < 16 * ((2 * D + 15) / 16);
}

// SPLIT: the P tile runs on FP16 MFMA (K = 32) as three products of hi + lo
// pairs, A_hi B_hi + A_lo B_hi + A_hi B_lo, accumulated in FP32; the beam-
// weighted sky carries the channel's power-of-two scale, undone at the end.
template <int D, bool SPLIT, bool WRAP>
struct KFringeFwd {
  using Args = FwdArgs;
  static constexpr int kThreads = 64 * kFwdWaves, kWaves = D <= 8 ? 4 : 2;
  static __device__ void run(const FwdArgs& args, const Blk& B);
};

template <int D, bool SPLIT, bool WRAP>
__device__ void KFringeFwd<D, SPLIT, WRAP>::run(const FwdArgs& args, const Blk& B) {
  const int nf = args.nf, nt = args.nt, nvp = args.nvp, nubl = args.nubl;
  const float d_omega = args.d_omega;
  const float2* Q1 = args.Q1;
  const float2* Q2 = args.Q2;
  const float* TH2 = args.TH2;
  const int* __restrict__ tchunk_off = args.tchunk_off;
  const int* __restrict__ tchunk = args.tchunk;
  const int2* __restrict__ ubl_nm = args.ubl_nm;
  const float* img = args.img;
  const float* __restrict__ fwhm = args.fwhm;
  float2* __restrict__ vu = args.vu;
  using T = Tile<D>;
  constexpr int RT = T::RT, W = T::W;
  __shared__ __attribute__((aligned(16))) float As_all[kFwdWaves][64 * W];
  __shared__ __attribute__((aligned(16))) float Bs_all[kFwdWaves][64 * W];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
  float* As = As_all[wv];   // this wave's operand rows
  float* Bs = Bs_all[wv];
  // SPLIT: the same LDS as FP16 hi and lo row sets (64 rows of W halves each)
  uint32_t* Ah = reinterpret_cast<uint32_t*>(As);
  uint32_t* Al = Ah + 32 * W;
  uint32_t* Bh = reinterpret_cast<uint32_t*>(Bs);
  uint32_t* Bl = Bh + 32 * W;
  constexpr int NCH = fwd_channels_per_tile(D);
  static_assert(NCH == 1 || RT == 1, "stacked channels share one 16 x 16 tile");
  constexpr bool AXT = fwd_axis_in_tile(D);
  const int nfg = (nf + NCH - 1) / NCH;   // channel groups
  const int L = xcd_logical(B.x, B.nx);
  if (L >= nfg * nt) return;   // uniform over the block
  int t, fgrp;
  tile_map(L, nt, nfg, 4, 32, t, fgrp);   // 128 resident blocks per XCD: 4 times x 32 channel groups
  // channel c of the group: f = NCH fgrp + c; one past the band (an odd
  // channel count) runs with zero weight and is not written
  float dnu[NCH], csc[NCH], kb[NCH], chan_on[NCH], cut = 0.f;
  const float* imf[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int fc = NCH * fgrp + c, fl = min(fc, nf - 1);
    chan_on[c] = fc < nf ? 1.0f : 0.0f;
    dnu[c] = args.dnu[fl];
    csc[c] = SPLIT ? chan_scale(args.cscale, fl, d_omega) : 1.0f;   // power of two
    const float sig = fwhm[0] * args.sigr[fl];
    kb[c] = beam_kb(sig);
    cut = c == 0 ? beam_cut(args.cut_sig2, sig) : fmaxf(cut, beam_cut(args.cut_sig2, sig));
    imf[c] = img + static_cast<size_t>(fl) * nvp;
  }

  // NACC independent accumulator sets (consecutive MFMAs of a chunk go to
  // different sets); one set measured fastest at 61 dishes
  constexpr int NACC = 1;
  f4 acc[NACC][RT][RT];
#pragma unroll
  for (int h = 0; h < NACC; ++h)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < RT; ++j) acc[h][i][j] = f4{0.f, 0.f, 0.f, 0.f};
  // per-lane partial sums of alpha^n S and beta^m S (the axis baselines;
  // unused where they ride in the tile)
  constexpr int DX = AXT ? 1 : D;
  float axr[NCH][DX], axi[NCH][DX], bxr[NCH][DX], bxi[NCH][DX];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int n = 0; n < DX; ++n) axr[c][n] = axi[c][n] = bxr[c][n] = bxi[c][n] = 0.f;

  // the chunks of this time within the beam of the group's widest channel,
  // visited from the furthest to the nearest: the sums take the small terms
  // first (nearest first, their rounding errors measured 1.2 to 2 times larger)
  const int cbeg = tchunk_off[t];
  const int cend = cbeg + beam_prefix<8>(args.tchunk_ex + cbeg, tchunk_off[t + 1] - cbeg, cut, lane);
  const float2* q1t = Q1 + static_cast<size_t>(t) * nvp;
  const float2* q2t = Q2 + static_cast<size_t>(t) * nvp;
  const float* tht = TH2 + static_cast<size_t>(t) * nvp;

  struct G { float2 q1, q2; float th, iv[NCH]; };
  // this wave's chunks: entry j is the list's (wv + kFwdWaves j)-th from its end
  constexpr int S = kFwdWaves;
  constexpr bool ROW = D <= 6;   // scalar row addresses (LaneOffset) and chunk indices
  const int mine = max(0, (cend - cbeg - wv + S - 1) / S);
  auto chunk_at = [&](int j) {   // uniform
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (ROW) {   // through the constant address space: a scalar load
      typedef const int __attribute__((address_space(4))) ConstInt;
      return ((const ConstInt*)(reinterpret_cast<uintptr_t>(tchunk)))[cend - 1 - wv - S * j];
    }
#endif
    return tchunk[cend - 1 - wv - S * j];
  };
  LaneOffset<ROW> lo(lane);
  auto load = [&](int chunk) {
    G g;
    if constexpr (ROW) {
      const int k0 = chunk * kChunk;
      lo.touch(k0);
      g.q1 = lo.at(q1t + k0);
      g.q2 = lo.at(q2t + k0);
      g.th = lo.at(tht + k0);
#pragma unroll
      for (int c = 0; c < NCH; ++c) g.iv[c] = lo.at(imf[c] + k0);
    } else {
      const int k = chunk * kChunk + lane;
      g.q1 = at_u32(q1t, k);
      g.q2 = at_u32(q2t, k);
      g.th = at_u32(tht, k);
#pragma unroll
      for (int c = 0; c < NCH; ++c) g.iv[c] = at_u32(imf[c], k);
    }
    return g;
  };
  // powers of one chunk into LDS, channel c in rows and columns 2D c ..
  auto generate = [&](const G& g) {
    float av[SPLIT ? 1 : W], bv[SPLIT ? 1 : W];
    uint32_t ah[SPLIT ? W / 2 : 1], al[SPLIT ? W / 2 : 1], bh[SPLIT ? W / 2 : 1], bl[SPLIT ? W / 2 : 1];
    float wlast = 0.f;   // the weight (times its scale) of the last channel
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const float x1 = phase_cycles<WRAP>(dnu[c], g.q1);
      const float x2 = phase_cycles<WRAP>(dnu[c], g.q2);
      const float s = chan_on[c] * d_omega * beam_exp2(-g.th * kb[c]) * g.iv[c];
      float s1, c1, s2, c2;
      sincos_rev(x1, s1, c1);
      sincos_rev(x2, s2, c2);
      auto visit = [&](int n, float ar, float ai, float br, float bi) {
        if constexpr (!AXT) {
          axr[c][n] += ar * s;
          axi[c][n] += ai * s;
          bxr[c][n] += br;   // SPLIT: scaled by csc, undone after the loop
          bxi[c][n] += bi;
        }
      };
      wlast = SPLIT ? s * csc[c] : s;
      if constexpr (SPLIT)
        powers_split_fwd<D>(ah + D * c, al + D * c, bh + D * c, bl + D * c, c1, s1, c2, s2,
                            wlast, visit);
      else
        powers_f32<D>(av + 2 * D * c, bv + 2 * D * c, c1, s1, c2, s2, s, visit);
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (int n = NCH * D; n < W / 2; ++n) ah[n] = al[n] = bh[n] = bl[n] = 0u;
      if constexpr (AXT) {   // row 2 D: (1, 0); column 2 D: (w, 0), as hi + lo
        ah[D] = split_hi2(1.f, 0.f);
        bh[D] = split_hi2(wlast, 0.f);
        bl[D] = split_lo2(wlast, 0.f, bh[D]);
      }
      store_rows_split<W>(Ah, Al, Bh, Bl, lane, ah, al, bh, bl);
    } else {
#pragma unroll
      for (int r = 2 * NCH * D; r < W; ++r) av[r] = bv[r] = 0.f;
      if constexpr (AXT) {
        av[2 * D] = 1.f;
        bv[2 * D] = wlast;
      }
      store_rows<W>(As, Bs, lane, av, bv);
    }
  };
  float a[SPLIT ? 1 : 16][RT], b[SPLIT ? 1 : 16][RT];
  // SPLIT operands of the two K = 32 steps of a chunk: hi and lo of A and B
  h8 oah[SPLIT ? 2 : 1][RT], oal[SPLIT ? 2 : 1][RT], obh[SPLIT ? 2 : 1][RT], obl[SPLIT ? 2 : 1][RT];
  // MFMA step q reads row px = 4 q + (lane >> 4); the swizzle of row px
  // depends on q only through q & 1, so two per-lane offsets per column tile
  // plus a constant 8 W per step pair address every read (the constant goes
  // into the instruction's offset field instead of an address register)
  int ofs[2][RT];
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int i = 0; i < RT; ++i) ofs[e][i] = lds_at<W>(4 * e + (lane >> 4), 16 * i + (lane & 15));
  auto operands = [&]() {
    if constexpr (SPLIT) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          oah[ks][i] = tr_operand<W>(Ah, 32 * ks, i, lane);
          oal[ks][i] = tr_operand<W>(Al, 32 * ks, i, lane);
          obh[ks][i] = tr_operand<W>(Bh, 32 * ks, i, lane);
          obl[ks][i] = tr_operand<W>(Bl, 32 * ks, i, lane);
        }
    } else {
#pragma unroll
      for (int q = 0; q < 16; ++q) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const int o = ofs[q & 1][i] + (q >> 1) * 8 * W;
          a[q][i] = As[o];
          b[q][i] = Bs[o];
        }
      }
    }
  };
  auto products = [&]() {
    if constexpr (SPLIT) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < RT; ++j) {
            acc[0][i][j] = mfma_h32(oah[ks][i], obh[ks][j], acc[0][i][j]);
            acc[0][i][j] = mfma_h32(oal[ks][i], obh[ks][j], acc[0][i][j]);
            acc[0][i][j] = mfma_h32(oah[ks][i], obl[ks][j], acc[0][i][j]);
          }
    } else {
#pragma unroll
      for (int q = 0; q < 16; ++q)
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < RT; ++j)
            acc[q % NACC][i][j] = mfma4(a[q][i], b[q][j], acc[q % NACC][i][j]);
    }
  };
  // one chunk but the wave's last: the MFMAs of chunk j (register operands)
  // interleaved with the generation of the next chunk from `cur`, while the
  // geometry of the one after it loads into `nxt` (ROW: its chunk `ahead` was
  // read a step earlier); the loop below is unrolled by two so the two geometry
  // sets swap roles without register copies
  int ahead = 0;
  auto chunk_step = [&](int j, const G& cur, G& nxt) {
    if constexpr (ROW) {
      nxt = load(ahead);
      ahead = chunk_at(min(j + 3, mine - 1));
    } else {
      nxt = load(chunk_at(min(j + 2, mine - 1)));
    }
    // keep the prefetch here: the sources are read-only, so the optimizer
    // would otherwise re-issue the loads right before their use
    asm volatile("" ::: "memory");
    products();
    generate(cur);
    if constexpr (SPLIT) {
#pragma unroll
      for (int q = 0; q < 6 * RT * RT; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 16 / (RT * RT), 0);  // vector ALU
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // one LDS write (128-bit)
      }
    } else {
#pragma unroll
      for (int q = 0; q < 16 * RT * RT; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 8 / (RT * RT), 0);  // vector ALU
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // one LDS write (128-bit)
      }
    }
    wave_sync();
    operands();
    wave_sync();
  };
  if (mine > 0) {   // uniform over the wave
    ahead = chunk_at(min(2, mine - 1));
    generate(load(chunk_at(0)));
    G ga = load(chunk_at(min(1, mine - 1))), gb;
    wave_sync();
    operands();
    wave_sync();
    int j = 0;
    if ((mine - 1) & 1) {   // an odd number of steps before the last chunk
      chunk_step(j, ga, gb);
      ga = gb;
      ++j;
    }
    for (; j + 1 < mine; j += 2) {
      chunk_step(j, ga, gb);
      chunk_step(j + 1, gb, ga);
    }
    products();
  }
  float inv_csc[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) inv_csc[c] = 1.0f / csc[c];   // exact: a power of two
  // Axis sums over the lanes of all waves: every lane's NAX partial sums go to
  // the operand rows value by value, and eight threads per value add them in a
  // fixed order (a butterfly over the lanes, 6 NAX cross-lane moves per wave,
  // costs as much as two chunks).
  constexpr int NAX = AXT ? 0 : 4 * D * NCH;
  constexpr int NAXT = (NAX + 31) / 32;   // values per thread group
  float axs[NAXT > 0 ? NAXT : 1];
  if constexpr (!AXT) {
    static_assert(NAX == 2 * W, "axis sums fill the operand rows");
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int n = 0; n < D; ++n) {
        const float v[4] = {axr[c][n], axi[c][n], bxr[c][n] * inv_csc[c], bxi[c][n] * inv_csc[c]};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int e = 4 * (D * c + n) + q;
          (e < W ? As + 64 * e : Bs + 64 * (e - W))[lane] = v[q];
        }
      }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < NAXT; ++g) {
      const int e = 32 * g + (threadIdx.x >> 3), part = threadIdx.x & 7;
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < kFwdWaves; ++w) {
        const float* x = (e < W ? As_all[w] + 64 * e : Bs_all[w] + 64 * (e - W)) + 8 * part;
        const f4 x0 = *reinterpret_cast<const f4*>(x), x1 = *reinterpret_cast<const f4*>(x + 4);
        sum += ((x0[0] + x0[1]) + (x0[2] + x0[3])) + ((x1[0] + x1[1]) + (x1[2] + x1[3]));
      }
      for (int o = 1; o < 8; o <<= 1) sum += __shfl_xor(sum, o);
      axs[g] = sum;
    }
    __syncthreads();
  }
  // this wave's P tile to its LDS rows (reused as a W x W matrix)
  {
    float* Pw = As;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < RT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float sum = acc[0][i][j][r];
#pragma unroll
          for (int h = 1; h < NACC; ++h) sum += acc[h][i][j][r];
          // column 16 j + (lane & 15) belongs to channel (lane & 15) / 2D
          if constexpr (SPLIT) {
            float isc = inv_csc[0];
#pragma unroll
            for (int c = 1; c < NCH; ++c)
              if ((lane & 15) >= 2 * D * c) isc = inv_csc[c];
            sum *= isc;
          }
          Pw[(16 * i + 4 * (lane >> 4) + r) * W + 16 * j + (lane & 15)] = sum;
        }
  }
  __syncthreads();
  // the block's totals, waves added in index order, into the last wave's rows
  float* P = Bs_all[kFwdWaves - 1];
  float* AX = P + W * W;   // [NCH][D][4]: axr, axi, bxr, bxi
  static_assert(NAX + W * W <= 64 * W, "tile totals exceed one wave's rows");
  for (int e = threadIdx.x; e < W * W; e += 64 * kFwdWaves) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kFwdWaves; ++w) sum += As_all[w][e];
    P[e] = sum;
  }
  if constexpr (!AXT) {
#pragma unroll
    for (int g = 0; g < NAXT; ++g)
      if ((threadIdx.x & 7) == 0) AX[32 * g + (threadIdx.x >> 3)] = axs[g];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int fc = NCH * fgrp + c;
    if (fc >= nf) break;   // uniform over the block
    float2* out = vu + (static_cast<size_t>(t) * nf + fc) * nubl;
    const float* AXc = AX + 4 * D * c;
    const int off = 2 * D * c;   // the channel's diagonal block
    for (int u = threadIdx.x; u < nubl; u += 64 * kFwdWaves) {
      const int2 nm = ubl_nm[u];
      float2 v;
      if (AXT && nm.x == 0) {   // row 2 D: sum_p of the B columns of beta^m w
        v = make_float2(P[2 * D * W + 2 * (nm.y - 1)], P[2 * D * W + 2 * (nm.y - 1) + 1]);
      } else if (AXT && nm.y == 0) {   // column 2 D: sum_p of alpha^n w
        v = make_float2(P[2 * (nm.x - 1) * W + 2 * D], P[(2 * (nm.x - 1) + 1) * W + 2 * D]);
      } else if (nm.x == 0) {
        v = make_float2(AXc[4 * (nm.y - 1) + 2], AXc[4 * (nm.y - 1) + 3]);
      } else if (nm.y == 0) {
        v = make_float2(AXc[4 * (nm.x - 1)], AXc[4 * (nm.x - 1) + 1]);
      } else {
        const int m = nm.y > 0 ? nm.y : -nm.y;
        const int r0 = off + 2 * (nm.x - 1), c0 = off + 2 * (m - 1);
        const float p1 = P[r0 * W + c0], p3 = P[r0 * W + c0 + 1];
        const float p4 = P[(r0 + 1) * W + c0], p2 = P[(r0 + 1) * W + c0 + 1];
        v = nm.y > 0 ? make_float2(p1 - p2, p3 + p4) : make_float2(p1 + p2, p4 - p3);
      }
      out[u] = v;
    }
  }
}

// ------------------------------------------------------------------ adjoint --
// One block per (nu, chunk of 64 visible pixels) (per pair of channels
// for D = 4, see adj_channels_per_tile); its wavefronts loop over the times at
// which the chunk is above the horizon and within the beam (kBeamBits).
// gco[t][nu] holds the coefficient matrix in MFMA A-operand order, then the
// alpha-axis accumulator inputs of every (row tile, lane group), then the axis
// coefficients (and, SPLIT, the inverse of the power-of-two scale of the FP16
// coefficients).
//
// Bound by issue, like the forward.  61 dishes, 64 channels, 60 times, 10 deg
// beam: 0.660 -> 0.212 ms for 27% of the (chunk, time) pairs.  What is left
// over the 0.176 ms of the same time per pair is each wave's start and end
// (about 200 vector instructions, two steps' worth).  Tried: one wave per item
// (0.245 ms: 8400 items within the beam in 4096 resident waves of unequal length
// leave CUs idle at the end, 72% of the CU cycles busy), two waves (0.215 ms), and
// resident blocks that take items in rounds (0.236 ms).  Chunks dealt to the XCDs
// with all their channels, so that a chunk's geometry is read into one L2 only,
// change nothing (0.99 to 1.01 times over beams of 10 to 37 deg).
//
// SPLIT: T = G Bb runs on FP16 MFMA, per 16 x 16 tile one K = 32 product
// [G_hi | G_lo] [B_hi; B_hi] and one K = 16 product G_hi B_lo; the coefficient
// operands come ready from the gains pass, only beta^m is split here.
template <int RT, bool SPLIT> struct AdjCoef { f4 gv[RT][RT]; };
template <int RT> struct AdjCoef<RT, true> { h8 ga[RT][RT]; h4 gb[RT][RT]; };

struct AdjArgs {
  int nf, nt, nvp, nchunks, gstride;
  float d_omega, cut_sig2;
  const float* dnu;
  const float* sigr;
  const float2* Q1;
  const float2* Q2;
  const float* TH2;
  const float* chunk_ex;
  float sigr_max;
  int split_chunks;
  int shared_items;     // items of the first split_chunks chunks
  unsigned nfg_magic;   // ceil(2^32 / channel groups)
  const int4* chunk_times;
  const int* ctime;
  const float* ctime_ex;
  const float* img;
  const float* fwhm;
  const float* gco;
  const float* gco_lane;
  float* dimg;
  float* f_part;
  // non-null: dL/dI of visible slot k < nv goes to dfull[voff[k] + nu fstride]
  // (the full-grid rows of the separable adjoint synthesis), not dimg[nu][k]
  float* dfull;
  const int* voff;
  int nv, fstride;
};

// Wavefronts per block.
__host__ __device__ constexpr int adj_waves(int D) { return D <= 8 ? 4 : 2; }

// Items within the beam up to which a block's waves share one item's times:
// rounds of `resident` waves, more of them the more times an item may have.  A
// wave that takes items of its own leaves its SIMD idle for part of the last
// item's times; sharing costs every item its set-up in each wave and the
// reduction over them.  With `n` rounds of items, microseconds whole / shared:
//   61 dishes, 15 times  n = 0.2: 19.1 / 14.6   0.6: 30.7 / 30.4   1.1: 45.7 / 50.2   3.8 (24 deg): 120 / 132
//   61 dishes, 30 times  n = 0.5: 40.8 / 35.9   1.6: 101 / 101     1.9: 124 / 120     3.1 (14 deg): 181 / 187
//   61 dishes, 60 times  n = 0.7: 102 / 87      1.3: 159 / 139     4.0 (24 deg): 437 / 405
//   61 dishes,  5 times  n = 0.2: 10.3 / 10.1   0.6: 15.0 / 19.2
//   91 dishes, 30 times  n = 1.4: 156 / 123     3.1: 288 / 258     4.7: 372 / 363     7.8 (24 deg): 587 / 591
//   91 dishes,  5 times  n = 2.1: 44 / 48       4.5: 82 / 89
inline double adj_shared_items(int D, int n_time, int resident) {
  const double t = n_time;
  return resident * (D <= 8 ? std::max(t / 25.0, t * t / 350.0) : t / 4.0);
}

template <int D, bool SPLIT, bool WRAP>
struct KFringeAdj {
  using Args = AdjArgs;
  // four waves per SIMD, where the compiler would take one register too many
  static constexpr int kThreads = 64 * adj_waves(D), kWaves = D == 4 && SPLIT ? 4 : 1;
  static __device__ void run(const AdjArgs& args, const Blk& B);
};

template <int D, bool SPLIT, bool WRAP>
__device__ void KFringeAdj<D, SPLIT, WRAP>::run(const AdjArgs& args, const Blk& B) {
  const int nf = args.nf, nvp = args.nvp, nchunks = args.nchunks, gstride = args.gstride;
  const float d_omega = args.d_omega;
  const float2* Q1 = args.Q1;
  const float2* Q2 = args.Q2;
  const float* TH2 = args.TH2;
  const float* __restrict__ img = args.img;
  const float* __restrict__ fwhm = args.fwhm;
  const float* __restrict__ gco = args.gco;
  const float* gco_lane = args.gco_lane;
  float* __restrict__ dimg = args.dimg;
  float* __restrict__ f_part = args.f_part;
  using T = Tile<D>;
  using R = SplitRows<T::W>;
  constexpr int RT = T::RT, W = T::W;
  constexpr int NMAT = RT * RT * (SPLIT ? 384 : 256);
  constexpr int NW = adj_waves(D);
  __shared__ __attribute__((aligned(16))) float As_all[NW][64 * W];
  // FP32 B operand rows, or (SPLIT) the hi rows followed by the lo rows
  __shared__ __attribute__((aligned(16))) float Bs_all[NW][SPLIT ? 64 * R::BH + R::BL_WORDS : 64 * W];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
  float* As = As_all[wv];
  float* Bs = Bs_all[wv];
  uint32_t* Bh = reinterpret_cast<uint32_t*>(Bs);
  uint32_t* Bl = Bh + 64 * R::BH;
  const int lane = threadIdx.x & 63;
  constexpr int NCH = adj_channels_per_tile(D);
  static_assert(NCH == 1 || (D == 4 && RT == 1), "two stacked channels: D = 4 only");
  // beta-axis terms in the tile's row 2 D (the gains pass put omega(0, m)
  // there) against a row of ones in the pixel operand
  constexpr bool AXT = adj_axis_in_tile(D);
  // the beam weights of two channels in the padding of the split B rows: with an
  // array of their own a block's LDS fits a CU three times instead of four (19
  // dishes, 120 channels, 30 times: 128 -> 107 us with a 10 deg beam, 355 -> 315 us
  // with 37 deg; where four fit either way the array's reads are 2% faster)
  constexpr bool BW_PAD = SPLIT && NCH == 2;
  static_assert(!BW_PAD || 2 * NCH <= R::BH - W / 2, "beam weights in the padding of the split rows");
  const int nfg = (nf + NCH - 1) / NCH;   // channel groups
  // dL/dI of this lane's pixel of a chunk
  auto put = [&](int chunk, int f, float v) {
    const int k = chunk * kChunk + lane;
    if (args.dfull != nullptr) {        // uniform over the wave
      if (k < args.nv)
        args.dfull[static_cast<size_t>(args.voff[k]) + static_cast<size_t>(f) * args.fstride] = v;
    } else {
      dimg[static_cast<size_t>(f) * nvp + k] = v;
    }
  };
  const float fw = fwhm[0];
  const float cut_w = beam_cut(args.cut_sig2, fw * args.sigr_max);   // the field's widest channel
  // Items are (chunk, channel group) pairs, chunk-major.  The chunks come
  // sorted by their nearest approach to the beam centre: those within the beam
  // of the field's widest channel are a prefix, the longest time loops start
  // first, and the grid ends on items that only write zeros.  With few items
  // within the beam (at most split_chunks chunks) the block's waves share one
  // item's times; with many, each wave takes an item of its own, and so it does
  // of the items that are then sure to be outside.
  const bool few = args.split_chunks >= nchunks || args.chunk_ex[args.split_chunks] > cut_w;
  const bool shared = few && B.x < args.shared_items;
  const int first = few ? args.shared_items : 0;   // of the items taken by waves
  const int item = shared ? B.x : first + (B.x - first) * NW + wv;
  if (item >= nfg * nchunks) return;
  // item / nfg through the host's ceil(2^32 / nfg) (at most one too large), on
  // the scalar unit
  int chunk = nfg == 1 ? item : static_cast<int>(__umulhi(static_cast<unsigned>(item), args.nfg_magic));
  if (chunk * nfg > item) --chunk;
  const int fgrp = item - chunk * nfg;
  const int4 ct = args.chunk_times[chunk];
  if (__int_as_float(ct.x) > cut_w) {   // uniform over the wave
    if (!shared || wv == 0)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int f = NCH * fgrp + c;
        if (f >= nf) break;
        put(chunk, f, 0.f);
        if (lane == 0) f_part[static_cast<size_t>(f) * nchunks + chunk] = 0.f;
      }
    return;
  }
  const int w0 = shared ? wv : 0, nw = shared ? NW : 1;   // this wave's share of the times
  const int k = chunk * kChunk + lane;
  // channel c of the group: f = NCH fgrp + c (one past the band, for an odd
  // channel count, gets zero coefficients and is not written)
  int fch[NCH];
  float dnu[NCH], kb[NCH], acc_i[NCH], acc_f[NCH], chan_on[NCH], cut = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int fc = NCH * fgrp + c;
    fch[c] = min(fc, nf - 1);
    chan_on[c] = fc < nf ? 1.0f : 0.0f;
    dnu[c] = args.dnu[fch[c]];
    const float sig = fw * args.sigr[fch[c]];
    kb[c] = beam_kb(sig);
    cut = c == 0 ? beam_cut(args.cut_sig2, sig) : fmaxf(cut, beam_cut(args.cut_sig2, sig));
    acc_i[c] = acc_f[c] = 0.f;
  }
  // NCH > 1: the tile's row block r / 2D and column block belong to one
  // channel each; a lane's coefficient operand is channel c's own operand of
  // lane `lane - src_shift c` on the diagonal blocks and zero elsewhere, and
  // its output rows 4 (lane >> 4) .. + 3 belong to channel (lane >> 4) / 2
  const int c_row = NCH > 1 ? (lane & 15) / (2 * D) : 0;
  const int c_out = NCH > 1 ? (lane >> 4) / (D / 2) : 0;
  // the times at which this chunk is within the beam of the group's widest
  // channel; where that is all of them, nothing waits for the list's excesses
  // (nor, in a wave that takes them all, the first step for the list)
  const int tall = ct.z;
  const size_t trow = static_cast<size_t>(chunk) * args.nt;
  const int* __restrict__ tlist = args.ctime + trow;
  int tl = tlist[min(lane, args.nt - 1)], tl_blk = 0;   // 64 entries of the list in the lanes
  const bool all_in = __int_as_float(ct.y) <= cut;
  int ntl = tall;
  if (!all_in) ntl = beam_prefix<1>(args.ctime_ex + trow, tall, cut, lane);
  const int mine = shared ? max(0, (ntl - wv + NW - 1) / NW) : ntl;   // entries w0, w0 + nw, ..
  // Partial sums, over this lane's four rows of every row tile, of the core and
  // alpha-axis terms of the pixels of the four 16-pixel groups, weighted by B
  // and by B theta^2; reduced across the row groups once, after the time loop.
  float pz_i[4] = {0.f, 0.f, 0.f, 0.f}, pz_f[4] = {0.f, 0.f, 0.f, 0.f};
  // (B, B theta^2) of every pixel of the chunk at this t and channel
  __shared__ float2 BW_all[BW_PAD ? 1 : NW][NCH][BW_PAD ? 1 : 64];
  auto bw_at = [&](int c, int px) -> float2& {
    if constexpr (BW_PAD) return *reinterpret_cast<float2*>(Bh + px * R::BH + W / 2 + 2 * c);
    else return BW_all[wv][c][px];
  };
  const size_t gst = static_cast<size_t>(nf) * gstride;
  // gco feeds the wave-uniform (scalar) loads of the axis coefficients;
  // gco_lane, the same table, the per-lane loads of the prefetch below: a
  // pointer not marked read-only-unaliased keeps the optimizer from moving
  // those loads to their use in the next step (as it does for Q1, Q2, TH2)
  auto gco_at = [&](int t, int c) { return gco + t * gst + static_cast<size_t>(fch[c]) * gstride; };
  // Software pipeline over t, unrolled by two so that the two register sets
  // swap roles without copies: the geometry and this lane's coefficients of
  // the next time load while one is processed.
  struct Step : AdjCoef<RT, SPLIT> {
    int t;
    float2 q1, q2;
    float th2;
    // alpha-axis coefficients of this lane's rows 16 i + 4 (lane >> 4) + 0..3:
    // (Re, -Im) of omega(n, 0) for the two powers n of those rows, stored in
    // this order by the gains pass.  As the first MFMA's accumulator input
    // they put sum_n Re[omega(n, 0) alpha^n] into the per-pixel dot with A.
    f4 g1[RT];
  };
  // per-lane channel selection (NCH <= 2)
  auto chan_of = [&](const int* arr, int c) { return NCH == 1 || c == 0 ? arr[0] : arr[NCH - 1]; };
  // entry i of this wave's share, from its end (the weakest beam first, as in
  // the forward)
  auto time_at = [&](int i) {   // uniform
    const int e = ntl - 1 - w0 - i * nw;
    if ((e >> 6) != tl_blk) {
      tl_blk = e >> 6;
      tl = tlist[min(64 * tl_blk + lane, tall - 1)];
    }
    return __builtin_amdgcn_readlane(tl, e & 63);
  };
  LaneOffset<(D <= 6)> lo(lane);
  auto load_step = [&](Step& S, int t) {   // t uniform
    lo.touch(t);
    S.t = t;
    const size_t row = static_cast<size_t>(t) * nvp + chunk * kChunk;   // uniform over the wave
    S.q1 = lo.at(Q1 + row);
    S.q2 = lo.at(Q2 + row);
    S.th2 = lo.at(TH2 + row);
    const size_t tbase = static_cast<size_t>(t) * gst;
    // the coefficient operand: this lane's row channel's slice; zero off the
    // diagonal blocks and for a channel past the band
    const float* Gr = gco_lane + tbase + static_cast<size_t>(chan_of(fch, c_row)) * gstride;
    const float* Go = gco_lane + tbase + static_cast<size_t>(chan_of(fch, c_out)) * gstride;
    const bool row_on = NCH == 1 || (c_row == 0 ? chan_on[0] : chan_on[NCH - 1]) != 0.f;
    const bool on_blk = NCH == 1 || (row_on && c_row == c_out);
    const bool on_k32 = NCH == 1 || (row_on && c_row == ((lane >> 4) & 1));
    const int src = lane - 40 * c_row;          // FP32 and K = 16 operands
    const int src32 = lane - 24 * c_row;        // K = 32 operand
#pragma unroll
    for (int i = 0; i < RT; ++i) {
#pragma unroll
      for (int kt = 0; kt < RT; ++kt) {
        if constexpr (SPLIT) {
          const h8 va = *reinterpret_cast<const h8*>(Gr + ((i * RT + kt) * 64 + (on_k32 ? src32 : lane)) * 4);
          const h4 vb = *reinterpret_cast<const h4*>(Gr + RT * RT * 256 + ((i * RT + kt) * 64 + (on_blk ? src : lane)) * 2);
          S.ga[i][kt] = on_k32 ? va : h8{};
          S.gb[i][kt] = on_blk ? vb : h4{};
        } else {
          const f4 v = at_u32(reinterpret_cast<const f4*>(Gr), (i * RT + kt) * 64 + (on_blk ? src : lane));
          S.gv[i][kt] = on_blk ? v : f4{0.f, 0.f, 0.f, 0.f};
        }
      }
      S.g1[i] = *reinterpret_cast<const f4*>(Go + NMAT + 16 * i + 4 * ((lane >> 4) - (D / 2) * c_out));
    }
  };
  auto step = [&](int i, const Step& S, Step& next) {
    const int t = S.t;
    const float2 q1 = S.q1, q2 = S.q2;
    const float th2 = S.th2;
    // unconditional (the last step re-reads its own time) so that the waits
    // for this step's operands never cover the loads just issued
    load_step(next, time_at(min(i + 1, mine - 1)));
    float av[W], bv[SPLIT ? 1 : W];
    uint32_t bh[SPLIT ? W / 2 : 1], bl[SPLIT ? W / 2 : 1];
    float bm[NCH], zax[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const float* G = gco_at(t, c);
      bm[c] = beam_exp2(-th2 * kb[c]);
      const float x1 = phase_cycles<WRAP>(dnu[c], q1);
      const float x2 = phase_cycles<WRAP>(dnu[c], q2);
      float s1, c1, s2, c2;
      sincos_rev(x1, s1, c1);
      sincos_rev(x2, s2, c2);
      // beta-axis terms of this lane's pixel: sum_n Re[omega(0, n) beta^n]
      zax[c] = 0.f;
      auto visit = [&](int n, float ar, float ai, float br, float bi) {
        if constexpr (!AXT) {
          const f4 ax = *reinterpret_cast<const f4*>(G + NMAT + 16 * RT + 4 * n);
          zax[c] = __builtin_fmaf(ax[2], br, zax[c]);   // two FMAs, no separate add
          zax[c] = __builtin_fmaf(-ax[3], bi, zax[c]);
        }
      };
      if constexpr (SPLIT) {
        powers_split_adj<D>(av + 2 * D * c, bh + D * c, bl + D * c, c1, s1, c2, s2, visit);
        // T comes out scaled by the coefficients' power of two: the weights undo it
        const float isc = G[NMAT + 16 * RT + 4 * D];
        bw_at(c, lane) = make_float2(bm[c] * isc, bm[c] * th2 * isc);
      } else {
        powers_f32<D>(av + 2 * D * c, bv + 2 * D * c, c1, s1, c2, s2, 1.0f, visit);
        bw_at(c, lane) = make_float2(bm[c], bm[c] * th2);
      }
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (int r = 2 * D * NCH; r < W; ++r) av[r] = 0.f;
#pragma unroll
      for (int n = D * NCH; n < W / 2; ++n) bh[n] = bl[n] = 0u;
      if constexpr (AXT) av[2 * D] = 1.f;
      store_rows_split_adj<W>(As, Bh, Bl, lane, av, bh, bl);
    } else {
#pragma unroll
      for (int r = 2 * D * NCH; r < W; ++r) av[r] = bv[r] = 0.f;
      if constexpr (AXT) av[2 * D] = 1.f;
      store_rows<W>(As, Bs, lane, av, bv);
    }
    wave_sync();
    float2 bw[4];
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) bw[pg] = bw_at(NCH == 1 ? 0 : c_out, 16 * pg + (lane & 15));
    // T = G Bb + alpha-axis rows for the four 16-pixel groups: the four MFMA
    // chains are interleaved (pixel group innermost) so consecutive MFMAs are
    // independent
    // B operand: lane l supplies column 4 (l >> 4) + s of the 16-column block kt
    // in MFMA step s (the coefficient layout uses the same order), so its four
    // steps' values are one 16-byte read of group l >> 4 of its pixel's row
    // (conflict-free; four scalar reads of rows 16 apart would share banks)
    // SPLIT: lane l supplies, for pixel 16 pg + (l & 15), the hi halves of
    // columns 16 kt + 8 ((l >> 4) & 1) + 0..7 (K = 32 product: lane groups 0, 1
    // meet G_hi, groups 2, 3 meet G_lo) and the lo halves of columns
    // 16 kt + 4 (l >> 4) + 0..3 (K = 16 product)
    f4 bq[SPLIT ? 1 : RT][4];
    h8 bh8[SPLIT ? RT : 1][4];
    h4 bl4[SPLIT ? RT : 1][4];
#pragma unroll
    for (int kt = 0; kt < RT; ++kt)
#pragma unroll
      for (int pg = 0; pg < 4; ++pg) {
        const int px = 16 * pg + (lane & 15);
        if constexpr (SPLIT) {
          bh8[kt][pg] = *reinterpret_cast<const h8*>(Bh + px * R::BH + 8 * kt + 4 * ((lane >> 4) & 1));
          bl4[kt][pg] = *reinterpret_cast<const h4*>(Bl + (4 * kt + (lane >> 4)) * R::BLP + 2 * px);
        } else {
          bq[kt][pg] = *reinterpret_cast<const f4*>(Bs + lds_at<W>(px, 16 * kt + 4 * (lane >> 4)));
        }
      }
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      f4 tacc[4];
      if constexpr (SPLIT) {
#pragma unroll
        for (int kt = 0; kt < RT; ++kt) {
#pragma unroll
          for (int pg = 0; pg < 4; ++pg)
            tacc[pg] = mfma_h32(S.ga[i][kt], bh8[kt][pg], kt == 0 ? S.g1[i] : tacc[pg]);
#pragma unroll
          for (int pg = 0; pg < 4; ++pg) tacc[pg] = mfma_h16(S.gb[i][kt], bl4[kt][pg], tacc[pg]);
        }
      } else {
#pragma unroll
        for (int kt = 0; kt < RT; ++kt)
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int pg = 0; pg < 4; ++pg)
              tacc[pg] = mfma4(S.gv[i][kt][s], bq[kt][pg][s], (kt == 0 && s == 0) ? S.g1[i] : tacc[pg]);
      }
#pragma unroll
      for (int pg = 0; pg < 4; ++pg) {
        const int px = 16 * pg + (lane & 15);
        const f4 av = *reinterpret_cast<const f4*>(As + lds_at<W>(px, 16 * i + 4 * (lane >> 4)));
        float zp = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) zp += av[r] * tacc[pg][r];
        pz_i[pg] += bw[pg].x * zp;
        pz_f[pg] += bw[pg].y * zp;
      }
    }
    wave_sync();
    if constexpr (!AXT) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        acc_i[c] += bm[c] * zax[c];
        acc_f[c] += bm[c] * th2 * zax[c];
      }
    }
  };
  if (mine > 0) {   // uniform over the wave
    Step sa, sb;
    int t_first = ct.w;
    if (!all_in || shared) t_first = time_at(0);
    load_step(sa, t_first);
    for (int i = 0; i < mine; i += 2) {
      step(i, sa, sb);
      if (i + 1 >= mine) break;
      step(i + 1, sb, sa);
    }
  }
  // The partial sums of each pixel sit in the lanes of its four row groups (two
  // per channel for NCH = 2) of every wave that shares the item, the beta-axis
  // terms in its own lane: all go to LDS, and the last wave (the one with the
  // fewest times) adds them for its lane's pixel in a fixed order.
  wave_sync();
  float2* pz = reinterpret_cast<float2*>(As);   // [4][64] by pixel group and lane, then [NCH][64]
#pragma unroll
  for (int pg = 0; pg < 4; ++pg) pz[64 * pg + lane] = make_float2(pz_i[pg], pz_f[pg]);
#pragma unroll
  for (int c = 0; c < NCH; ++c) pz[64 * (4 + c) + lane] = make_float2(acc_i[c], acc_f[c]);
  if (shared) {
    __syncthreads();
    if (wv != NW - 1) return;
  } else {
    wave_sync();
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    if (NCH * fgrp + c >= nf) break;   // uniform over the wave
    float si = 0.f, sf = 0.f;
    for (int w = shared ? 0 : wv; w <= wv; ++w) {
      const float2* x = reinterpret_cast<const float2*>(As_all[w]);
      float2 v = x[64 * (4 + c) + lane];
#pragma unroll
      for (int g = c * (4 / NCH); g < (c + 1) * (4 / NCH); ++g) {
        const float2 z = x[64 * (lane >> 4) + 16 * g + (lane & 15)];
        v.x += z.x;
        v.y += z.y;
      }
      si += v.x;
      sf += v.y;
    }
    put(chunk, fch[c], d_omega * si);
    float pf = sf * img[static_cast<size_t>(fch[c]) * nvp + k];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) pf += __shfl_xor(pf, o);
    const float sig = fw * args.sigr[fch[c]], kappa = 1.0f / (sig * sig * fw);   // dB/dF = B theta^2 kappa
    if (lane == 0) f_part[static_cast<size_t>(fch[c]) * nchunks + chunk] = d_omega * kappa * pf;
  }
}

// ------------------------------------------------------------ launchers --
template <class K>
struct KernelTag {
  using Kernel = K;
};

template <int D>
static void fwd_d(const vis_field* f, const float* img, const float* fwhm, float2* vu, hipStream_t st) {
  constexpr int nch = fwd_channels_per_tile(D);
  const int nblk = static_cast<int>(round_up(static_cast<long>((f->n_freq + nch - 1) / nch) * f->n_time, 8));
  const auto& T = f->tab;
  const bool split = fringe_split(f);
  if (split) {
    ProfScope ps(&f->prof, "k_chan_scale", st);
    launch_k<KChanScale>(dim3(f->n_freq, kScaleParts), 0,
                         ChanScaleArgs{f->nv_pad, beam_slots(f, fwhm), img, f->scr.fscale}, st, "k_chan_scale");
  }
  ProfScope ps(&f->prof, "k_fringe_fwd", st);
  const FwdArgs a{f->n_freq, f->n_time, f->nv_pad, f->n_ubl, static_cast<float>(f->d_omega),
                  f->cut_sig2, T.dnu, T.sigr, T.q1, T.q2, T.th2, T.tchunk_off, T.tchunk, T.tchunk_ex, T.ubl_nm,
                  img, fwhm, vu, split ? f->scr.fscale : nullptr};
  const bool wrap = f->max_turns > kMaxTurns;
  auto launch = [&](auto k) { launch_k<typename decltype(k)::Kernel>(dim3(nblk), 0, a, st, "k_fringe_fwd"); };
  if (split)
    wrap ? launch(KernelTag<KFringeFwd<D, true, true>>{}) : launch(KernelTag<KFringeFwd<D, true, false>>{});
  else
    wrap ? launch(KernelTag<KFringeFwd<D, false, true>>{}) : launch(KernelTag<KFringeFwd<D, false, false>>{});
}

template <int D>
static void adj_d(const vis_field* f, const float* img, const float* fwhm, const float* gco,
                  float* dimg, float* dfull, float* f_part, hipStream_t st) {
  constexpr int nch = adj_channels_per_tile(D);
  const int nfg = (f->n_freq + nch - 1) / nch;
  const int waves = f->n_cu * (D <= 8 ? 16 : 8);   // resident
  const int split_chunks =
      static_cast<int>(std::min<double>(f->n_chunks, adj_shared_items(D, f->n_time, waves) / nfg));
  // blocks for either way of taking the items, the later ones of which are idle
  // in the other (a block that only finds that out holds its LDS for a quarter
  // of a microsecond)
  const int items = nfg * f->n_chunks, shared_items = nfg * split_chunks;
  const int nblk = static_cast<int>(round_up(shared_items + ceil_div(items - shared_items, adj_waves(D)), 8));
  const auto& T = f->tab;
  ProfScope ps(&f->prof, "k_fringe_adj", st);
  BV_REQUIRE(f->dtile == D, VIS_EINVAL, "internal: adjoint tile mismatch");
  BV_REQUIRE((dimg == nullptr) != (dfull == nullptr), VIS_EINVAL, "internal: one adjoint output");
  const AdjArgs a{f->n_freq, f->n_time, f->nv_pad, f->n_chunks, f->gstride,
                  static_cast<float>(f->d_omega), f->cut_sig2, T.dnu, T.sigr, T.q1, T.q2, T.th2,
                  T.chunk_ex, f->sigr_max, split_chunks, shared_items,
                  static_cast<unsigned>(((1ull << 32) + nfg - 1) / nfg), T.chunk_times, T.ctime, T.ctime_ex, img, fwhm, gco, gco, dimg, f_part, dfull, T.sep_voff, f->nv,
                  f->basis->nphi_b};
  const bool wrap = f->max_turns > kMaxTurns;
  auto launch = [&](auto k) { launch_k<typename decltype(k)::Kernel>(dim3(nblk), 0, a, st, "k_fringe_adj"); };
  if (fringe_split(f))
    wrap ? launch(KernelTag<KFringeAdj<D, true, true>>{}) : launch(KernelTag<KFringeAdj<D, true, false>>{});
  else
    wrap ? launch(KernelTag<KFringeAdj<D, false, true>>{}) : launch(KernelTag<KFringeAdj<D, false, false>>{});
}

#define BV_DISPATCH_EXTENT(ext, CALL)          \
  do {                                         \
    const int e_ = (ext);                      \
    if (e_ <= 2) { CALL(2); }                  \
    else if (e_ <= 4) { CALL(4); }             \
    else if (e_ <= 6) { CALL(6); }             \
    else if (e_ <= 8) { CALL(8); }             \
    else if (e_ <= 12) { CALL(12); }           \
    else { CALL(16); }                         \
  } while (0)

}  // namespace bv
