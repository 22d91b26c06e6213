// Wave-per-site hop kernels of libdwa: one wavefront computes one site on all slices
// (L_s = 2 .. 16: there is room for 16 slices), with the fifth-dimension matrices before and
// after the hop applied together on the matrix cores.
//
// Field layout of these kernels ("site-major"): element (site, colour, s, spin) of a half
// field sits at ((site * 3 + colour) * Ls + s) * 4 + spin, so a site is one contiguous run
// (3 KB in FP64, 768 B in BF16 at L_s = 16) and a wave's gather of one neighbour and colour
// is one contiguous read.  The strides are launch arguments, so a kernel can also read or
// write the library's SoA layout.  Links are gathered per output site: [parity][site][8][9],
// the backward ones daggered, the boundary phase folded in.
#pragma once

#include <type_traits>

#include "kcommon.h"

namespace dwa {

// wave-local LDS exchange: LDS operations of one wave complete in order, so only the
// compiler has to be kept from moving them
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ unsigned fast_div(unsigned n, unsigned d, unsigned magic) {
  return d == 1 ? n : __umulhi(n, magic);
}

// The site at position i of the walk (x/2, y, z in its group, t, z group) and its eight
// neighbours, as checkerboard indices of the output parity and of the other one.
struct WaveSite {
  unsigned cb, xh, odd;
  unsigned nb[8];
};
__device__ __forceinline__ WaveSite wave_site(const WaveGeo& g, unsigned i, unsigned parity) {
  const unsigned q1 = fast_div(i, g.Lxh, g.mLxh), xh = i - q1 * g.Lxh;
  const unsigned q2 = fast_div(q1, g.Ly, g.mLy), y = q1 - q2 * g.Ly;
  const unsigned q3 = fast_div(q2, g.ZB, g.mZB), zb = q2 - q3 * g.ZB;
  const unsigned zo = fast_div(q3, g.Lt, g.mLt), t = q3 - zo * g.Lt;
  const unsigned z = zo * g.ZB + zb;
  const unsigned sy = g.Lxh, sz = g.Lxh * g.Ly, st = sz * g.Lz;
  WaveSite w;
  w.cb = t * st + z * sz + y * sy + xh;
  const unsigned odd = (y + z + t + parity) & 1u;  // x = 2 xh + odd
  w.xh = xh;
  w.odd = odd;
  w.nb[0] = odd ? (xh + 1 == g.Lxh ? w.cb + 1 - g.Lxh : w.cb + 1) : w.cb;
  w.nb[4] = odd ? w.cb : (xh == 0 ? w.cb + g.Lxh - 1 : w.cb - 1);
  w.nb[1] = y + 1 == g.Ly ? w.cb - (g.Ly - 1) * sy : w.cb + sy;
  w.nb[5] = y == 0 ? w.cb + (g.Ly - 1) * sy : w.cb - sy;
  w.nb[2] = z + 1 == g.Lz ? w.cb - (g.Lz - 1) * sz : w.cb + sz;
  w.nb[6] = z == 0 ? w.cb + (g.Lz - 1) * sz : w.cb - sz;
  w.nb[3] = t + 1 == g.Lt ? w.cb - (g.Lt - 1) * st : w.cb + st;
  w.nb[7] = t == 0 ? w.cb + (g.Lt - 1) * st : w.cb - st;
  return w;
}

// The neighbours of site xh + k of the same x row (w: the site xh, odd its row's offset).
__device__ __forceinline__ void wave_row_step(const WaveGeo& g, const WaveSite& w, unsigned k, WaveSite& o) {
  const unsigned xh = w.xh + k;
  o.cb = w.cb + k;
  o.xh = xh;
  o.odd = w.odd;
#pragma unroll
  for (int d = 0; d < 8; ++d) o.nb[d] = w.nb[d] + k;
  o.nb[0] = w.odd ? (xh + 1 == g.Lxh ? o.cb + 1 - g.Lxh : o.cb + 1) : o.cb;
  o.nb[4] = w.odd ? o.cb : (xh == 0 ? o.cb + g.Lxh - 1 : o.cb - 1);
}

// Blocks are dealt to the 8 XCDs round robin: give each XCD one contiguous range of n chunks.
__device__ __forceinline__ unsigned xcd_range(unsigned b, unsigned n) {
  const unsigned q = n >> 3, r = n & 7u, x = b & 7u;
  return x * q + (x < r ? x : r) + (b >> 3);
}
typedef float dwa_f4 __attribute__((ext_vector_type(4)));
typedef double dwa_d4 __attribute__((ext_vector_type(4)));
typedef short dwa_s4 __attribute__((ext_vector_type(4)));
template <typename R> struct AccT;
template <> struct AccT<float> { using type = dwa_f4; };
template <> struct AccT<double> { using type = dwa_d4; };
template <typename R>
using acc4 = typename AccT<R>::type;

// The type of the mix and its matrices.  FP32 fields are mixed in FP64: a dense product of 16
// terms in FP32 would round more than the sweeps of hop_mix_kernel do.
template <typename S>
using WaveMix = std::conditional_t<S::prec == DWA_BF16, float, double>;

// acc += V M^T: V (12 reals of one chirality x slices) comes as a matrix-core result, lane l
// holding column l % 16 and the slices 4 (l / 16) + i, which is also the layout of a left
// operand; M[s'][s] comes as M[l % 16][4 (l / 16) + i].  In the result lane l holds slice
// l % 16 and the reals mix_col^-1 of rows 4 (l / 16) + i (FP64: 4 i + l / 16).
__device__ __forceinline__ void mix_mfma(dwa_f4& acc, const dwa_f4& V, const float* M) {
#pragma unroll
  for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(V[i], M[i], acc, 0, 0, 0);
}
__device__ __forceinline__ void mix_mfma(dwa_d4& acc, const dwa_d4& V, const double* M) {
#pragma unroll
  for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(V[i], M[i], acc, 0, 0, 0);
}
// Column n of an operand holds the real k = spin of the chirality * 2 + (re, im) of colour
// c, such that a lane of the mixed result holds the four reals of colour lane / 16.
template <typename R>
__device__ __forceinline__ void mix_col(int n, int& c, int& k) {
  if constexpr (sizeof(R) == 8) {
    c = n & 3;
    k = n >> 2;
  } else {
    c = n >> 2;
    k = n & 3;
  }
  if (c > 2) c = 2;  // idle columns
}

template <typename R, int CTRL>
__device__ __forceinline__ R quad_perm(R v) {
  if constexpr (sizeof(R) == 8) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = __builtin_amdgcn_mov_dpp((int)(unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
  } else {
    return __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
  }
}

// T += gamma_mu x over the four spins of a quad, of which lane g holds spin g.  The factor is
// the source spin's: x: i (+, +, -, -), y: (-, +, +, -), z: i (+, -, -, +), t: 1.
template <typename R>
__device__ __forceinline__ void add_gamma(int mu, int g, const cpx<R>& x, cpx<R>& T) {
  const R e = mu == 0 ? (g < 2 ? R(1) : R(-1)) : (((g == 0 || g == 3) == (mu == 2)) ? R(1) : R(-1));
  cpx<R> y;
  if (mu == 0 || mu == 2) y = cmk<R>(-e * x.im, e * x.re);
  else if (mu == 1) y = cmk<R>(e * x.re, e * x.im);
  else y = x;
  if (mu < 2) {
    T.re += quad_perm<R, 0x1B>(y.re);
    T.im += quad_perm<R, 0x1B>(y.im);
  } else {
    T.re += quad_perm<R, 0x4E>(y.re);
    T.im += quad_perm<R, 0x4E>(y.im);
  }
}

// rows of the wave's exchange buffer: [24 = colour * 8 + spin * 2 + (re, im)][slice], padded
template <typename R>
constexpr int kWavePitch = sizeof(R) == 8 ? 18 : 20;
template <typename R>
constexpr int kWaveBuf = 24 * kWavePitch<R>;
constexpr unsigned kWaveMaxSpw = 16;  // sites of a block per wave

// FP64 / FP32 hop of one site: lane (s, spin g) = (lane / 4, lane % 4) multiplies the links
// (wave-uniform, in scalar registers) onto its own spin of each neighbour and adds them to D
// (the unit part of 1 -+ gamma_mu).
// gamma_mu of the differences goes to T: its row g is a factor +-1, +-i times spin 3 - g
// (x, y) or g ^ 2 (z, t), exchanged within the quad.
template <typename S>
__device__ __forceinline__ void wave_hop_valu(const WaveHopArgs& a, __amdgpu_buffer_rsrc_t in, const WaveSite& w,
                                              unsigned lane_off, int g, cpx<RealOf<S>> D[3],
                                              cpx<RealOf<S>> T[3]) {
  using R = RealOf<S>;
  constexpr unsigned E = sizeof(typename S::elem);
  // opaque, so that the links' addresses are not computed ahead and spilled
  unsigned lsite = w.cb;
  asm volatile("" : "+s"(lsite));
  cptr<R> L = as_const(reinterpret_cast<const R*>(a.links) + size_t(lsite) * 144);
#pragma unroll
  for (int c = 0; c < 3; ++c) D[c] = T[c] = cmk<R>(0, 0);
  cpx<R> f[4][2][3];
#pragma unroll
  for (int mu = 0; mu < 4; ++mu)
#pragma unroll
    for (int bwd = 0; bwd < 2; ++bwd) {
      const unsigned nb = w.nb[bwd * 4 + mu] * a.in_st.site;
#pragma unroll
      for (int c = 0; c < 3; ++c) f[mu][bwd][c] = ldbuf<S>(in, lane_off, (nb + unsigned(c) * a.in_st.col) * E);
    }
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    cpx<R> v[2][3];
#pragma unroll
    for (int bwd = 0; bwd < 2; ++bwd) {
      cptr<R> u = L + (bwd * 4 + mu) * 18;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        cpx<R> t;
        const cpx<R>* p = f[mu][bwd];
        t.re = u[6 * c] * p[0].re;
        t.im = u[6 * c] * p[0].im;
        t.re = fma(-u[6 * c + 1], p[0].im, t.re);
        t.im = fma(u[6 * c + 1], p[0].re, t.im);
#pragma unroll
        for (int k = 1; k < 3; ++k) {
          t.re = fma(u[6 * c + 2 * k], p[k].re, t.re);
          t.im = fma(u[6 * c + 2 * k], p[k].im, t.im);
          t.re = fma(-u[6 * c + 2 * k + 1], p[k].im, t.re);
          t.im = fma(u[6 * c + 2 * k + 1], p[k].re, t.im);
        }
        v[bwd][c] = t;
        D[c] = D[c] + t;
      }
      // the scalar registers hold the links of one or two directions at a time
      if (sizeof(R) == 8 || bwd) __builtin_amdgcn_sched_barrier(0x20);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) add_gamma<R>(mu, g, v[1][c] - v[0][c], T[c]);
  }
}

// Values of lane (s, g) to the matrix-core operand (wave_get).
template <typename R>
__device__ __forceinline__ void wave_put(R* buf, int s, int g, const cpx<R> v[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    buf[(c * 8 + g * 2) * kWavePitch<R> + s] = v[c].re;
    buf[(c * 8 + g * 2 + 1) * kWavePitch<R> + s] = v[c].im;
  }
}
// Chirality ch of them, for a mix in M.
template <typename M, typename R>
__device__ __forceinline__ acc4<M> wave_get(const R* buf, int lane, int ch) {
  const int kq = lane >> 4;
  int c, k;
  mix_col<M>(lane & 15, c, k);
  const R* p = buf + (c * 8 + ch * 4 + k) * kWavePitch<R> + 4 * kq;
  acc4<M> v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = (M)p[i];
  return v;
}

// Lane constants of the BF16 hop's link operands.  Column lane % 16 is (colour, spin of the
// chirality al, re / im ri), and chunk j of the contraction gives the lane group kq = lane / 16
// the group idx = 4 j + kq = direction * 3 + input colour.  An operand word pair serves two
// input spins, one of which has a zero: the LDS table holds each word between two zeros, and a
// lane reads (word, 0) or (0, word) by its offset.
constexpr unsigned kLinkWord = 8;   // bytes from one form of a link to the next
constexpr unsigned kLinkStep = 48;  // from one link to the next (padded against bank conflicts)
struct WaveLinkLane {
  unsigned d0;     // unit part at chunk 0 (chunks are 12 links apart)
  unsigned su[3];  // gamma_mu part, upper rows, forward chunks
  unsigned sl[3];  // the same of the lower rows
  unsigned bu[3], bl[3];  // of the backward chunks (36 links on, the opposite sign)
};
__device__ __forceinline__ WaveLinkLane wave_link_lane(int lane) {
  const int n = lane & 15, kq = lane >> 4;
  const int co = n < 12 ? n >> 2 : 2, al = (n >> 1) & 1, ri = n & 1;
  WaveLinkLane w;
  w.d0 = unsigned(kq * 3 + co) * kLinkStep + unsigned(ri) * kLinkWord + (al ? 0u : 4u);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int idx = 4 * j + kq, mu = idx / 3;
    // exponent k of gamma_mu's factor i^k in the upper and the lower row al; the forward hop
    // takes -gamma_mu
    const int ku = mu == 0 ? 3 : (mu == 1 ? (al ? 0 : 2) : (mu == 2 ? (al ? 1 : 3) : 0));
    const int kl = mu == 0 ? 1 : (mu == 1 ? (al ? 2 : 0) : (mu == 2 ? (al ? 3 : 1) : 0));
    const int in = mu < 2 ? 1 - al : al;  // input spin of the other chirality
    const unsigned base = unsigned(idx * 3 + co) * kLinkStep + (in ? 0u : 4u);
    w.su[j] = base + unsigned((ri - ku - 2) & 3) * kLinkWord;
    w.sl[j] = base + unsigned((ri - kl - 2) & 3) * kLinkWord;
    w.bu[j] = base + 36 * kLinkStep + unsigned((ri - ku) & 3) * kLinkWord;
    w.bl[j] = base + 36 * kLinkStep + unsigned((ri - kl) & 3) * kLinkWord;
  }
  return w;
}
// The two link words of a lane (lanes 0 .. 35) of one site.
__device__ __forceinline__ uint2 wave_load_links(const WaveHopArgs& a, unsigned cb, int lane) {
  uint2 v = make_uint2(0u, 0u);
  if (lane < 36) v = reinterpret_cast<const uint2*>(static_cast<const char*>(a.links) + size_t(cb) * 288)[lane];
  return v;
}
// Stage one site's 72 link words in LDS, each in the four forms that a row of the real 2x2
// block of i^k u takes: (re, -im), (im, re) and their negatives.  (The zeros between them are
// written once per block.)
__device__ __forceinline__ void wave_stage_links(uint32_t* tab, int lane, uint2 v) {
  wave_lds_sync();
  if (lane < 36) {
    uint32_t* t = tab + 2 * lane * (kLinkStep / 4) + 1;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t u = k ? v.y : v.x;
      const uint32_t v0 = u ^ 0x80000000u, v1 = (u >> 16) | (u << 16);
      t[12 * k] = v0;
      t[12 * k + 2] = v1;
      t[12 * k + 4] = v0 ^ 0x80008000u;
      t[12 * k + 6] = v1 ^ 0x80008000u;
    }
  }
  wave_lds_sync();
}
// Operands of the forward (b = 0) or backward (b = 1, opposite sign: two forms on) chunk j:
// the unit part d (either chirality) and the gamma_mu parts of the upper and lower rows.
__device__ __forceinline__ dwa_v2u wave_link_pair(const uint32_t* tab, unsigned off) {
  const uint32_t* p = reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(tab) + off);
  return dwa_v2u{p[0], p[1]};
}
typedef __bf16 dwa_b8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ dwa_f4 mfma_bf16(dwa_v4u a, dwa_v4u b, dwa_f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dwa_b8, a), __builtin_bit_cast(dwa_b8, b), c, 0, 0,
                                                 0);
}

// BF16 hop of one site on the matrix cores: rows are slices, columns the 12 reals of one
// chirality's output, and the contraction runs over (direction, colour, spin, re / im); lane
// group kq holds four spins of (direction, colour) = (idx / 3, idx % 3), idx = 4 j + kq, of
// the forward and of the backward neighbour in step j.  up / lo: spins 0, 1 / 2, 3.  The
// products of BF16 numbers are exact and summed in FP32.
struct WaveIn {
  dwa_v4u f[3], b[3];
};
template <bool SM>
__device__ __forceinline__ void wave_load_bf16(const WaveHopArgs& a, __amdgpu_buffer_rsrc_t in, const WaveSite& w,
                                               const unsigned lane_c[3], int kq, WaveIn& v) {
  const unsigned ss = a.in_st.site * 4u;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int d0 = 4 * j / 3, r = 4 * j % 3;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const unsigned n0 = w.nb[4 * b + d0] * ss, n1 = w.nb[4 * b + (d0 + 1 > 3 ? 3 : d0 + 1)] * ss;
      const unsigned off = ((kq + r >= 3) ? n1 : n0) + lane_c[j];
      dwa_v4u& q = b ? v.b[j] : v.f[j];
      if constexpr (SM) {
        // one 16-byte load: the address unit takes as long for 8 bytes a lane
        q = __builtin_bit_cast(dwa_v4u, __builtin_amdgcn_raw_buffer_load_b128(in, off, 0, 0));
      } else {
        const unsigned st = a.in_st.spin * 4u;
        q[0] = __builtin_amdgcn_raw_buffer_load_b32(in, off, 0, 0);
        q[1] = __builtin_amdgcn_raw_buffer_load_b32(in, off, st, 0);
        q[2] = __builtin_amdgcn_raw_buffer_load_b32(in, off, 2 * st, 0);
        q[3] = __builtin_amdgcn_raw_buffer_load_b32(in, off, 3 * st, 0);
      }
    }
  }
}
template <bool SPLIT>
__device__ __forceinline__ void wave_hop_bf16(const uint32_t* tab, const WaveLinkLane& ll, const WaveIn& v,
                                              dwa_f4 D[2], dwa_f4 T[2]) {
  constexpr unsigned BW = 36 * kLinkStep;
#pragma unroll
  for (int ch = 0; ch < 2; ++ch) D[ch] = T[ch] = dwa_f4{0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const unsigned dj = ll.d0 + 12 * kLinkStep * j;
    const dwa_v2u df = wave_link_pair(tab, dj), db = wave_link_pair(tab, dj + BW);
    const dwa_v2u uf = wave_link_pair(tab, ll.su[j]), lf = wave_link_pair(tab, ll.sl[j]);
    const dwa_v2u ub = wave_link_pair(tab, ll.bu[j]), lb = wave_link_pair(tab, ll.bl[j]);
    if constexpr (SPLIT) {
      const dwa_v4u up = {v.f[j][0], v.f[j][1], v.b[j][0], v.b[j][1]};
      const dwa_v4u lo = {v.f[j][2], v.f[j][3], v.b[j][2], v.b[j][3]};
      const dwa_v4u d = {df[0], df[1], db[0], db[1]};
      D[0] = mfma_bf16(up, d, D[0]);
      D[1] = mfma_bf16(lo, d, D[1]);
      T[0] = mfma_bf16(lo, dwa_v4u{uf[0], uf[1], ub[0], ub[1]}, T[0]);
      T[1] = mfma_bf16(up, dwa_v4u{lf[0], lf[1], lb[0], lb[1]}, T[1]);
    } else {
      D[0] = mfma_bf16(v.f[j], dwa_v4u{df[0], df[1], uf[0], uf[1]}, D[0]);
      D[1] = mfma_bf16(v.f[j], dwa_v4u{lf[0], lf[1], df[0], df[1]}, D[1]);
      T[0] = mfma_bf16(v.b[j], dwa_v4u{db[0], db[1], ub[0], ub[1]}, T[0]);
      T[1] = mfma_bf16(v.b[j], dwa_v4u{lb[0], lb[1], db[0], db[1]}, T[1]);
    }
  }
  if constexpr (!SPLIT) {
    D[0] += T[0];
    D[1] += T[1];
  }
}

// out = M_D D + M_T T (+ post), D and T the two parts of the hop (see wave_hop_valu).  H mixes
// the chiralities only through T, whose input has the other chirality, so a matrix applied
// before the hop can be moved behind it: with premix P and output matrix M, chirality c takes
// M_c P_c on D and M_c P_(1-c) on T (SPLIT; otherwise one matrix serves both parts and they are
// summed first).
//
// What bounds it.  BF16 on a full chip (16^3 x 32, L_s = 16): issue, not memory - 26 and 36 us
// of bytes at 5.2 TB/s (138 and 188 MB); 28 matrix instructions a site in the first hop (12 of
// the hop, 16 of the mix) and 20 in the second, and 99 and 136 vector ones for gathers,
// staging, x term and norm, take 36 and 38 us, against 47 us and a premix pass of 20 us of
// hop_mix_kernel.  Not kept: a persistent grid (50 us where this took 46), double-buffered
// neighbours (46: the registers cost a wave per SIMD), a three-way BF16 split of the mix (44
// against 44).  Five waves per SIMD; six spill (72 us).
// FP64 / FP32: on small lattices the latency of one site's chain - two hops and two updates of
// a CGLS iteration on 4^4, L_s = 8, FP64 go from 71 to 44 us, D_bb from 29 to 18 - and on a
// full chip the vector unit, which multiplies both spins of a chirality where the half-spinor
// form needs one (2x the link products; FP64 hop at 16^3 x 32, L_s = 16: 250 us against 163 of
// hop_mix_kernel), so there it serves only the L_s whose generic kernel is slower still.  More
// than one wave per site was no faster on 4^4 (44 against 42 us) and slower from 8^4 on.
//   INSM   the input is site-major (BF16 reads four spins at once); else by strides
//   OUTL   0: by strides; 1: site-major; 2: SoA through an LDS tile of the block's sites
//   CROSS  (BF16) a wave's sites go on across the ends of x rows
template <typename S, bool SPLIT, bool POST, bool INSM, int OUTL, bool CROSS>
__global__ void __launch_bounds__(256, S::prec == DWA_BF16 ? 5 : 1) wave_hop_kernel(WaveHopArgs a) {
  using R = RealOf<S>;
  using E = typename S::elem;
  constexpr bool BF = S::prec == DWA_BF16;
  constexpr unsigned EB = sizeof(E);
  constexpr int NW = 4;
  using M = WaveMix<S>;
  __shared__ __align__(16) R xbuf[BF ? 1 : NW][SPLIT ? 2 : 1][BF ? 4 : kWaveBuf<R>];
  __shared__ __align__(16) uint32_t ltab[NW][BF ? 72 * kLinkStep / 4 : 4];
  __shared__ double wsum[NW * kWaveMaxSpw];
  extern __shared__ __align__(16) char tile_raw[];
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kq = lane >> 4;
  const int Ls = (int)a.Ls;
  const int s = lane & 15, c = kq;  // slice and colour of the output
  const bool live = s < Ls && c < 3;
  M mD[2][4], mT[2][4];
#pragma unroll
  for (int ch = 0; ch < 2; ++ch)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mD[ch][i] = reinterpret_cast<const M*>(a.mixD)[(ch * 64 + lane) * 4 + i];
      if constexpr (SPLIT) mT[ch][i] = reinterpret_cast<const M*>(a.mixT)[(ch * 64 + lane) * 4 + i];
    }
  if constexpr (BF) {
    for (int i = lane; i < int(72 * kLinkStep / 16); i += 64)
      reinterpret_cast<uint4*>(ltab[wid])[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  // the tables are waited for here: left to their first use, the wait would sit in the loop
  // below and drain its loads
  __builtin_amdgcn_s_waitcnt(0x0f70);
  const unsigned sc = s < Ls ? s : Ls - 1, cc = c < 3 ? c : 2;  // idle lanes repeat others
  const unsigned post_lane = POST ? (sc * a.post_st.s + cc * a.post_st.col) * EB : 0u;
  const unsigned out_lane = (sc * a.out_st.s + cc * a.out_st.col) * EB;
  const unsigned f = blockIdx.y;  // field
  const unsigned per = NW * a.spw;  // sites of the block
  const unsigned site0 = xcd_range(blockIdx.x, gridDim.x) * per;
  const unsigned site1 = site0 + per < a.Vh ? site0 + per : a.Vh;
  const unsigned fbytes = 12u * a.Ls * a.Vh * EB;
  auto field = [&](const void* p) {
    return make_rsrc(static_cast<const char*>(p) + size_t(f) * a.rhs_stride * EB, fbytes);
  };
  constexpr bool NORM = POST && OUTL != 2;  // (the tiled store serves operators without norms)
  double nrm = 0.0;
  // Norms are summed over spg sites of a wave and then over four such terms, in an order that
  // the sites of a wave do not change.  Term i of the block is complete:
  const unsigned terms = a.spw / a.spg;  // of a wave
  auto put_norm = [&](unsigned i) {
    const double t = wave_sum(nrm);
    if (lane == 0) wsum[i] = t;
    nrm = 0.0;
  };

  // x term of one site: the spins of chirality ch of the lane's slice and colour
  auto load_post = [&](__amdgpu_buffer_rsrc_t rp, unsigned cb, int ch, cpx<R> pv[2]) {
    if constexpr (POST) {
      const unsigned off = (cb * a.post_st.site + unsigned(2 * ch) * a.post_st.spin) * EB;
#pragma unroll
      for (int k = 0; k < 2; ++k) pv[k] = ldbuf<S>(rp, post_lane, off + unsigned(k) * a.post_st.spin * EB);
    }
  };
  // the second half of a site for chirality ch: mix, x term, store.  B0 / B1 hold the hop in
  // operand form; o receives the two spins.
  auto mix = [&](int ch, const acc4<M>& B0, const acc4<M>& B1, const cpx<R> pv[2], cpx<R> o[2]) {
    acc4<M> m = acc4<M>{0, 0, 0, 0};
    mix_mfma(m, B0, mD[ch]);
    if constexpr (SPLIT) mix_mfma(m, B1, mT[ch]);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if constexpr (POST) {
        o[k] = cmk<R>((R)(m[2 * k] + (M)pv[k].re), (R)(m[2 * k + 1] + (M)pv[k].im));
        if (NORM && live) nrm += (double)norm2(o[k]);
      } else {
        o[k] = cmk<R>((R)m[2 * k], (R)m[2 * k + 1]);
      }
    }
  };
  // n spins from spin sp0 on
  auto store = [&](__amdgpu_buffer_rsrc_t ro, unsigned cb, unsigned slot, int sp0, auto n_, const cpx<R>* o) {
    constexpr int n = decltype(n_)::value;
    if (!live) return;
    if constexpr (OUTL == 2) {  // (one field per block)
      constexpr int NSB = 128 / EB;
      E* tile = reinterpret_cast<E*>(tile_raw);
#pragma unroll
      for (int k = 0; k < n; ++k) st<S>(tile, (s * 12 + (sp0 + k) * 3 + c) * (NSB + 1) + slot, o[k]);
    } else {
      const unsigned off = (cb * a.out_st.site + unsigned(sp0) * a.out_st.spin) * EB;
      // (128-bit stores with no register in the scalar offset: see stbuf)
      if constexpr (OUTL == 1 && BF && n == 4) {
        const dwa_v4u q = {pack_bf16x2(o[0].re, o[0].im), pack_bf16x2(o[1].re, o[1].im),
                           pack_bf16x2(o[2].re, o[2].im), pack_bf16x2(o[3].re, o[3].im)};
        __builtin_amdgcn_raw_buffer_store_b128(q, ro, out_lane + off, 0, 0);
      } else if constexpr (OUTL == 1 && S::prec == DWA_F32 && n == 2) {
        const dwa_f4 q = {float(o[0].re), float(o[0].im), float(o[1].re), float(o[1].im)};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(dwa_v4u, q), ro, out_lane + off, 0, 0);
      } else {
#pragma unroll
        for (int k = 0; k < n; ++k) stbuf<S>(ro, out_lane, off + unsigned(k) * a.out_st.spin * EB, o[k]);
      }
    }
  };
  if constexpr (BF) {
    const WaveLinkLane ll = wave_link_lane(lane);
    unsigned lane_c[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) lane_c[j] = (sc * a.in_st.s + unsigned((j + kq) % 3) * a.in_st.col) * EB;
    // The wave's sites are consecutive in the walk; without CROSS they are in one x row (the
    // launcher sees to it).  The next site's links are loaded ahead within a row; the
    // neighbours are not (their registers would cost a wave per SIMD, and the other waves hide
    // them).
    const unsigned first = site0 + wid * a.spw;
    const unsigned cnt = first >= site1 ? 0u : (site1 - first < a.spw ? site1 - first : a.spw);
    unsigned term = wid * terms;
    if (cnt) {
      WaveSite row = wave_site(a.geo, first, a.parity);
      const __amdgpu_buffer_rsrc_t ri = field(a.in), rp = field(POST ? a.post : a.in), ro = field(a.out);
      uint2 lk = wave_load_links(a, row.cb, lane);
      unsigned k = 0, k0 = 0;  // k0: where the row began
      do {
        const unsigned end = NORM && k + a.spg < cnt ? k + a.spg : cnt;
        for (; k < end; ++k) {
          if constexpr (CROSS) {
            if (row.xh + (k - k0) == a.geo.Lxh) {
              row = wave_site(a.geo, first + k, a.parity);
              k0 = k;
              lk = wave_load_links(a, row.cb, lane);
            }
          }
          WaveSite w;
          wave_row_step(a.geo, row, k - k0, w);
          WaveIn v;
          wave_load_bf16<INSM>(a, ri, w, lane_c, kq, v);
          cpx<R> pv[2][2];
          load_post(rp, w.cb, 0, pv[0]);
          load_post(rp, w.cb, 1, pv[1]);
          wave_stage_links(ltab[wid], lane, lk);
          if (k + 1 < cnt && (!CROSS || w.xh + 1 < a.geo.Lxh)) lk = wave_load_links(a, w.cb + 1, lane);
          dwa_f4 B0[2], B1[2];
          wave_hop_bf16<SPLIT>(ltab[wid], ll, v, B0, B1);
          cpx<R> o[4];
          mix(0, B0[0], B1[0], pv[0], o);
          mix(1, B0[1], B1[1], pv[1], o + 2);
          store(ro, w.cb, wid * a.spw + k, 0, std::integral_constant<int, 4>(), o);
        }
        if constexpr (NORM) {
          if (a.partials) put_norm(term++);
        }
      } while (k < cnt);
    }
    if constexpr (NORM) {  // (terms beyond the lattice)
      for (; term < (wid + 1) * terms; ++term)
        if (lane == 0) wsum[term] = 0.0;
    }
  } else {
    const int s4 = lane >> 2, g = lane & 3;
    const unsigned in_lane = (unsigned(s4 < Ls ? s4 : Ls - 1) * a.in_st.s + unsigned(g) * a.in_st.spin) * EB;
    R* buf = xbuf[wid][0];
    const __amdgpu_buffer_rsrc_t ri = field(a.in), rp = field(POST ? a.post : a.in), ro = field(a.out);
    unsigned term = wid, k = 0;
    do {
      const unsigned end = NORM ? k + a.spg : a.spw;
      for (; k < end; ++k) {
        const unsigned idx = site0 + k * NW + wid;
        if (idx >= site1) break;
        const WaveSite w = wave_site(a.geo, idx, a.parity);
        cpx<R> pv[2][2];
        load_post(rp, w.cb, 0, pv[0]);
        load_post(rp, w.cb, 1, pv[1]);
        cpx<R> D[3], T[3];
        wave_hop_valu<S>(a, ri, w, in_lane, g, D, T);
        if constexpr (!SPLIT) {
#pragma unroll
          for (int c = 0; c < 3; ++c) D[c] = D[c] + T[c];
        }
        wave_lds_sync();
        wave_put<R>(buf, s4, g, D);
        if constexpr (SPLIT) wave_put<R>(xbuf[wid][SPLIT ? 1 : 0], s4, g, T);
        wave_lds_sync();
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
          const acc4<M> B0 = wave_get<M>(buf, lane, ch);
          acc4<M> B1 = B0;
          if constexpr (SPLIT) B1 = wave_get<M>(buf + kWaveBuf<R>, lane, ch);
          cpx<R> o[2];
          mix(ch, B0, B1, pv[ch], o);
          store(ro, w.cb, idx - site0, 2 * ch, std::integral_constant<int, 2>(), o);
        }
      }
      k = end;
      if constexpr (NORM) {
        if (a.partials) put_norm(term);
        term += NW;
      }
    } while (k < a.spw);
  }
  if constexpr (OUTL == 2) {
    // the block's sites are consecutive checkerboard indices (the launcher sees to it)
    constexpr int NSB = 128 / EB;
    __syncthreads();
    const E* tile = reinterpret_cast<const E*>(tile_raw);
    const WaveSite w0 = wave_site(a.geo, site0, a.parity);
    E* out = reinterpret_cast<E*>(a.out) + size_t(f) * a.rhs_stride;
    for (int t = threadIdx.x; t < 12 * Ls * NSB; t += NW * 64) {
      const int row = t / NSB, j = t % NSB;
      if (site0 + j < site1) out[size_t(row) * a.Vh + w0.cb + j] = tile[row * (NSB + 1) + j];
    }
  }
  if constexpr (NORM) {
    if (a.partials) {
      __syncthreads();
      const unsigned i = site0 / (NW * a.spg) + threadIdx.x;
      if (threadIdx.x < terms && i < a.nsum) {
        double t = 0.0;
        for (int k = 0; k < NW; ++k) t += wsum[threadIdx.x * NW + k];
        a.partials[size_t(blockIdx.y) * a.nsum + i] = t;
      }
    }
  }
}

// Memory bound, at 4.5 TB/s (BF16, 16^3 x 32, L_s = 16: 22.5 us for 100 MB; with a field per
// thread and no tile the strided side moved 4 to 16 bytes a line).
// SoA -> site-major (TO_SM, with scale and precision change) or site-major -> SoA (ADD: the
// source times scale is added to the destination and then cleared), one field per blockIdx.y
// and 128 / sizeof(elem) sites per block, so that both sides move whole 128-byte lines, through
// an LDS tile.
template <typename SO, typename SI, bool TO_SM, bool ADD>
__global__ void __launch_bounds__(256) relayout_kernel(typename SO::elem* __restrict__ dst,
                                                       typename SI::elem* __restrict__ src, int Ls, unsigned Vh,
                                                       double scale, const double* __restrict__ scales) {
  using SA = std::conditional_t<TO_SM, SI, SO>;  // storage of the SoA side
  using ST = std::conditional_t<sizeof(typename SO::elem) < sizeof(typename SI::elem), SO, SI>;  // of the tile
  using E = typename ST::elem;
  constexpr int NSB = 128 / sizeof(typename SA::elem);
  constexpr int NSP = NSB + 1;
  extern __shared__ __align__(16) char tile_raw[];
  E* tile = reinterpret_cast<E*>(tile_raw);
  const unsigned site0 = xcd_range(blockIdx.x, gridDim.x) * NSB;
  const int nrow = 12 * Ls;
  const size_t foff = size_t(blockIdx.y) * nrow * Vh;
  dst += foff;
  src += foff;
  if (scales) scale = scales[blockIdx.y];
  const unsigned n = Vh - site0 < NSB ? Vh - site0 : NSB;
  auto conv = [&](cpx<RealOf<SI>> v) {
    return cmk<RealOf<SO>>((RealOf<SO>)(scale * (double)v.re), (RealOf<SO>)(scale * (double)v.im));
  };
  // thread (row group, site) on the SoA side; (site, element) on the other, whose element
  // (colour, s, spin) is row s * 12 + spin * 3 + colour
  const int j = threadIdx.x % NSB;
  if constexpr (TO_SM) {
    if (unsigned(j) < n)
      for (int row = threadIdx.x / NSB; row < nrow; row += 256 / NSB) {
        const cpx<RealOf<SI>> v = ld<SI>(src, size_t(row) * Vh + site0 + j);
        if constexpr (std::is_same_v<SO, SI>) st<ST>(tile, row * NSP + j, v);
        else st<ST>(tile, row * NSP + j, conv(v));
      }
    __syncthreads();
    for (int e = threadIdx.x; e < nrow; e += 256) {
      const int spin = e & 3, cs = e >> 2, c = cs / Ls, s = cs - c * Ls, row = s * 12 + spin * 3 + c;
      typename SO::elem* d = dst + size_t(site0) * nrow + e;
#pragma unroll 8
      for (unsigned k = 0; k < n; ++k) d[size_t(k) * nrow] = tile[row * NSP + k];
    }
  } else {
    for (int e = threadIdx.x; e < nrow; e += 256) {
      const int spin = e & 3, cs = e >> 2, c = cs / Ls, s = cs - c * Ls, row = s * 12 + spin * 3 + c;
      typename SI::elem* q = src + size_t(site0) * nrow + e;
#pragma unroll 8
      for (unsigned k = 0; k < n; ++k) {
        tile[row * NSP + k] = q[size_t(k) * nrow];
        if constexpr (ADD) st<SI>(q, size_t(k) * nrow, cmk<RealOf<SI>>(0, 0));
      }
    }
    __syncthreads();
    if (unsigned(j) < n)
      for (int row = threadIdx.x / NSB; row < nrow; row += 256 / NSB) {
        const size_t i = size_t(row) * Vh + site0 + j;
        const cpx<RealOf<SI>> v = ld<ST>(tile, row * NSP + j);
        if constexpr (ADD) {
          cpx<RealOf<SO>> x = ld<SO>(dst, i);
          x.re += (RealOf<SO>)(scale * (double)v.re);
          x.im += (RealOf<SO>)(scale * (double)v.im);
          st<SO>(dst, i, x);
        } else {
          st<SO>(dst, i, v);
        }
      }
  }
}

// 16 bytes of a field as complex numbers (BF16: 4, FP32: 2, FP64: 1), and of its accumulator
template <typename S>
constexpr int kVec = 16 / sizeof(typename S::elem);
template <typename S, bool STREAM>
__device__ __forceinline__ void ld_vec(const typename S::elem* p, size_t i, cpx<RealOf<S>>* v) {
  const dwa_v4u* q = reinterpret_cast<const dwa_v4u*>(p) + i;
  dwa_v4u u;
  if constexpr (STREAM) u = __builtin_nontemporal_load(q);
  else u = *q;
  if constexpr (S::prec == DWA_BF16) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = cmk<float>(__uint_as_float(u[k] << 16), __uint_as_float(u[k] & 0xffff0000u));
  } else if constexpr (S::prec == DWA_F32) {
#pragma unroll
    for (int k = 0; k < 2; ++k) v[k] = cmk<float>(__uint_as_float(u[2 * k]), __uint_as_float(u[2 * k + 1]));
  } else {
    const dwa_v2d d = __builtin_bit_cast(dwa_v2d, u);
    v[0] = cmk<double>(d.x, d.y);
  }
}
template <typename S, bool STREAM>
__device__ __forceinline__ void st_vec(typename S::elem* p, size_t i, const cpx<RealOf<S>>* v) {
  dwa_v4u u;
  if constexpr (S::prec == DWA_BF16) {
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = pack_bf16x2(v[k].re, v[k].im);
  } else if constexpr (S::prec == DWA_F32) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      u[2 * k] = __float_as_uint(v[k].re);
      u[2 * k + 1] = __float_as_uint(v[k].im);
    }
  } else {
    u = __builtin_bit_cast(dwa_v4u, dwa_v2d{v[0].re, v[0].im});
  }
  dwa_v4u* q = reinterpret_cast<dwa_v4u*>(p) + i;
  if constexpr (STREAM) __builtin_nontemporal_store(u, q);
  else *q = u;
}

// CGLS update 1 of site-major fields: x += a p ; r -= a q ; |r|^2, with a = gamma / |q|^2 from
// the hops' partials as in cg_update1_kernel.  The premix of r for the next operator belongs
// to its first hop here, so the update is elementwise: 16 bytes a thread and array, nvec of
// them per field, the first ones loaded before the partials are summed.  Memory bound: 67 us
// for 352 MB (5.3 TB/s) in BF16 at 16^3 x 32, L_s = 16, against 77 us of cg_update1_kernel,
// which wrote the premixed field as well.
template <typename S>
__global__ void __launch_bounds__(256) vec_update1_kernel(typename XAcc<S>::type::elem* __restrict__ x,
                                                          typename S::elem* __restrict__ r,
                                                          const typename S::elem* __restrict__ p,
                                                          const typename S::elem* __restrict__ q,
                                                          DevScalars* __restrict__ sc, size_t nvec, double* partials,
                                                          const double* __restrict__ qparts, int nq,
                                                          const double* __restrict__ zparts, int nz) {
  using R = RealOf<S>;
  using SX = typename XAcc<S>::type;
  constexpr int V = kVec<S>, XV = V / kVec<SX>;  // 16-byte words of x per word of the fields
  const size_t foff = size_t(blockIdx.y) * nvec * V;
  x += foff;
  r += foff;
  p += foff;
  q += foff;
  sc += blockIdx.y;
  size_t i = blockIdx.x * size_t(256) + threadIdx.x;
  const size_t step = size_t(gridDim.x) * 256;
  cpx<R> xv[V], rv[V], pv[V], qv[V];
  auto load = [&]() {
    if (i < nvec) {
      ld_vec<S, false>(p, i, pv);
      ld_vec<S, true>(q, i, qv);
      ld_vec<S, false>(r, i, rv);
#pragma unroll
      for (int k = 0; k < XV; ++k) ld_vec<SX, true>(x, i * XV + k, xv + k * kVec<SX>);
    }
  };
  load();
  const double qq = sum_partials_block(qparts + size_t(blockIdx.y) * nq, nq);
  const double gamma = sum_partials_block(zparts + size_t(blockIdx.y) * nz, nz);
  const bool bad = !(qq > 0.0) || !isfinite(qq);
  const double ad = (!sc->active || bad) ? 0.0 : gamma / qq;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc->qq = qq;
    sc->a = ad;
    sc->gamma = gamma;
    if (sc->active && bad) sc->flags |= 1;
  }
  const R a = (R)ad;
  double nrm = 0.0;
  while (i < nvec) {
#pragma unroll
    for (int k = 0; k < V; ++k) {
      xv[k] = xv[k] + a * pv[k];
      rv[k] = rv[k] - a * qv[k];
      nrm += (double)norm2(as_stored<S>(rv[k]));
    }
    st_vec<S, false>(r, i, rv);
#pragma unroll
    for (int k = 0; k < XV; ++k) st_vec<SX, true>(x, i * XV + k, xv + k * kVec<SX>);
    i += step;
    load();
  }
  block_sum_to(nrm, &partials[blockIdx.y * gridDim.x + blockIdx.x]);
}

// CGLS update 2: p = z + beta p, beta = |z|^2 / gamma from the partials (cg_update2_kernel).
// Memory bound: 25 us for 151 MB where cg_update2_kernel took 40 us with the premixed u.
template <typename S>
__global__ void __launch_bounds__(256) vec_update2_kernel(typename S::elem* __restrict__ p,
                                                          const typename S::elem* __restrict__ z,
                                                          DevScalars* __restrict__ sc, size_t nvec,
                                                          const double* __restrict__ zparts, int nz) {
  using R = RealOf<S>;
  constexpr int V = kVec<S>;
  const size_t foff = size_t(blockIdx.y) * nvec * V;
  p += foff;
  z += foff;
  sc += blockIdx.y;
  size_t i = blockIdx.x * size_t(256) + threadIdx.x;
  const size_t step = size_t(gridDim.x) * 256;
  cpx<R> pv[V], zv[V];
  auto load = [&]() {
    if (i < nvec) {
      ld_vec<S, false>(p, i, pv);
      ld_vec<S, true>(z, i, zv);
    }
  };
  load();
  const double zz = sum_partials_block(zparts + size_t(blockIdx.y) * nz, nz);
  const bool bad = !isfinite(zz) || !(sc->gamma > 0.0);
  const double bd = (!sc->active || bad) ? 0.0 : zz / sc->gamma;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc->zz = zz;
    sc->beta = bd;
    if (sc->active && bad) sc->flags |= 2;
  }
  const R beta = (R)bd;
  while (i < nvec) {
#pragma unroll
    for (int k = 0; k < V; ++k) pv[k] = zv[k] + beta * pv[k];
    st_vec<S, false>(p, i, pv);
    i += step;
    load();
  }
}

// canonical links -> the gathered links of both parities, [parity][cb][8][9]: the hop of
// direction dir multiplies the neighbour by E = U_mu(x) (dir = mu) or U_mu(x - mu)^dag
// (dir = 4 + mu), the antiperiodic phase folded in.  FP64 / FP32: rows E[a][b]; BF16: columns
// first, E[b][a] at [a][b] (the order in which wave_stage_links lays out the operands).
template <typename S>
__global__ void __launch_bounds__(256) gather_links_kernel(typename S::elem* __restrict__ dst,
                                                           const double2* __restrict__ src, int Lx, int Ly, int Lz,
                                                           int Lt, int apbc, unsigned V) {
  using R = RealOf<S>;
  const unsigned Vh = V / 2;
  const size_t n = size_t(8) * V;
  for (size_t t = blockIdx.x * size_t(blockDim.x) + threadIdx.x; t < n; t += size_t(gridDim.x) * blockDim.x) {
    const unsigned dir = t % 8, lex = t / 8, mu = dir & 3u;
    unsigned r = lex;
    unsigned x[4];
    const unsigned d[4] = {unsigned(Lx), unsigned(Ly), unsigned(Lz), unsigned(Lt)};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = r % d[k];
      r /= d[k];
    }
    const unsigned par = (x[0] + x[1] + x[2] + x[3]) & 1u;
    if (dir >= 4) x[mu] = x[mu] == 0 ? d[mu] - 1 : x[mu] - 1;
    const unsigned lsite = x[0] + d[0] * (x[1] + d[1] * (x[2] + d[2] * x[3]));
    const double sign = (apbc && mu == 3 && x[3] == d[3] - 1) ? -1.0 : 1.0;
    typename S::elem* o = dst + (size_t(par) * Vh + (lex >> 1)) * 72 + dir * 9;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        // E[i][j]
        const double2 v = src[(size_t(mu) * V + lsite) * 9 + (dir < 4 ? i * 3 + j : j * 3 + i)];
        const cpx<R> e = cmk<R>((R)(sign * v.x), (R)((dir < 4 ? sign : -sign) * v.y));
        st<S>(o, S::prec == DWA_BF16 ? j * 3 + i : i * 3 + j, e);
      }
  }
}

// ---------------------------------------------------------------------------
// launchers

inline FieldStrides soa_strides(const dwa_ctx* ctx) {
  const unsigned v = (unsigned)ctx->Vh;
  return {1u, 12u * v, 3u * v, v};
}
inline FieldStrides sm_strides(const dwa_ctx* ctx) {
  const unsigned L = (unsigned)ctx->Ls;
  return {12u * L, 4u, 1u, 4u * L};
}

template <typename S>
int launch_wave_hop_p(dwa_ctx* ctx, const WaveOp& op, int* nparts) {
  using R = RealOf<S>;
  constexpr unsigned EB = sizeof(typename S::elem);
  constexpr int NSB = 128 / EB;
  WaveHopArgs a;
  a.in = op.in;
  a.out = op.out;
  a.post = op.post;
  a.partials = op.partials;
  a.links = static_cast<const char*>(ctx->prec[S::prec].wlinks) + size_t(op.parity_out) * ctx->Vh * 72 * EB;
  using M = WaveMix<S>;
  const M* T = sizeof(M) == 8 ? (const M*)ctx->d_wave64 : (const M*)ctx->d_wave32;
  a.mixD = T + size_t(op.table) * 2 * 512;
  a.mixT = T + (size_t(op.table) * 2 + 1) * 512;
  a.Vh = (unsigned)ctx->Vh;
  a.Ls = (unsigned)ctx->Ls;
  a.parity = (unsigned)op.parity_out;
  a.nrhs = (unsigned)op.nrhs;
  a.rhs_stride = field_elems(ctx);
  a.in_st = op.in_soa ? soa_strides(ctx) : sm_strides(ctx);
  a.post_st = op.post_soa ? soa_strides(ctx) : sm_strides(ctx);
  a.out_st = op.out_soa ? soa_strides(ctx) : sm_strides(ctx);
  const bool split = op.table == WT_DBB1 || op.table == WT_DAG1;
  const bool tile = op.out_soa && !op.post_soa;
  a.geo = ctx->wgeo;
  // one field per block: with the links of a site shared by several, a block's fields run one
  // after the other (BF16 iteration of 12 fields of 12^3 x 24, L_s = 12: 1194 us; two fields a
  // block 1554, twelve 1359)
  const unsigned ny = a.nrhs;
  constexpr unsigned NW = 4;  // waves of a block
  // Sites per wave.  BF16: consecutive ones, whose links are loaded a site ahead, while enough
  // waves are left to fill the 256 CUs; the tiled store wants 128-byte rows (32 sites of a
  // block).  Of an x row where three or more of its sites divide it, else across row ends
  // (only rows of 8 were taken whole before, any other as 4, 2 or 1 sites: D_bb of 12 fields,
  // L_s = 12, 6 x 16^3 294 -> 216 us, 10^3 x 20 244 -> 170, 22 x 8 x 8 x 16 270 -> 187; always
  // across row ends D_bb of 8^3 x 16 takes 21.0 us instead of 18.3).  FP64 / FP32: one until
  // the chip is full, then up to 16, which repay the load of the matrices.
  auto cap = [&](size_t sites) { return tile || sites >= 32768 ? 8u : (sites >= 8192 ? 4u : 1u); };
  auto sites_per_wave = [&](size_t sites) {
    unsigned spw = 1;
    if (S::prec == DWA_BF16) {
      spw = cap(sites);
      for (unsigned d = spw; d >= 3; --d)
        if (a.geo.Lxh % d == 0) return d;
      if (a.geo.Lxh <= 2 && sites < 32768 && spw > a.geo.Lxh) spw = a.geo.Lxh;
    } else if (tile) {
      spw = NSB / NW;
    } else {
      while (spw < kWaveMaxSpw && sites / (2 * NW * spw) >= 4096) spw *= 2;
    }
    return spw;
  };
  // Norms are grouped by the lattice alone, so that a batch's field sums them as its own solve
  // does.  Its updates then sum as many terms as the single solve's, which costs a batch 0 to
  // 4% of an iteration (BF16, 12 fields of 8^3 x 16, L_s = 12: 244 -> 251 us; FP64, L_s = 9:
  // 613 -> 628) and up to 11 where few slices meet many sites (FP32, 12 of 12^3 x 24, L_s = 5:
  // 1615 -> 1795); giving every wave the sites of the single solve costs up to 10 (257, 633).
  a.spw = sites_per_wave(size_t(a.Vh) * ny);
  a.spg = sites_per_wave(a.Vh);
  if (a.spw % a.spg != 0) a.spw = cap(size_t(a.Vh) * ny) / a.spg * a.spg;
  a.nsum = (a.Vh + NW * a.spg - 1) / (NW * a.spg);
  // The walk: each XCD's range a group of Lz / 8 z-planes, walked in t, where that is two
  // planes or more (against plain order: 16^3 x 32, solves 0 to 2% and D_bb 0 to 5% less time;
  // 6 x 16^3 and 16^4 the same within 1%); of a single plane the neighbours in z are all
  // another XCD's (8^4 and 8^3 x 16: D_bb 0 to 12% more, solves 0 to 3).  The tiled store takes plain
  // order unless a plane is whole blocks, whose sites must be consecutive.
  if (ctx->dims[2] % 8 == 0 && ctx->dims[2] >= 16 && !(tile && (a.geo.Lxh * a.geo.Ly) % (NW * a.spw) != 0)) {
    a.geo.ZB = (unsigned)ctx->dims[2] / 8;
    a.geo.mZB = ctx->wgeo_mzdom;
  }
  const unsigned nblk = (a.Vh + NW * a.spw - 1) / (NW * a.spw);
  const dim3 grid(nblk, ny);
  const size_t shm = tile ? size_t(12) * a.Ls * (NSB + 1) * EB : 0;
  if (nparts) *nparts = int(a.nsum);
  const bool cross = a.geo.Lxh % a.spw != 0;
#define DWA_WAVE(SPLIT, POST, INSM, OUTL)                                                                       \
  if (S::prec == DWA_BF16 && cross)                                                                              \
    hipLaunchKernelGGL((wave_hop_kernel<S, SPLIT, POST, INSM, OUTL, S::prec == DWA_BF16>), grid, dim3(256), shm, \
                       ctx->stream, a);                                                                          \
  else                                                                                                           \
    hipLaunchKernelGGL((wave_hop_kernel<S, SPLIT, POST, INSM, OUTL, false>), grid, dim3(256), shm, ctx->stream, a)
  if (split) {
    if (op.post || op.out_soa) {
      set_error("wave hop: unsupported combination");
      return DWA_EINVAL;
    }
    if (op.in_soa) {
      DWA_WAVE(true, false, false, 1);
    } else {
      DWA_WAVE(true, false, true, 1);
    }
  } else {
    if (!op.post || op.in_soa) {
      set_error("wave hop: unsupported combination");
      return DWA_EINVAL;
    }
    if (tile) {
      DWA_WAVE(false, true, true, 2);
    } else if (op.out_soa) {
      DWA_WAVE(false, true, true, 0);
    } else {
      DWA_WAVE(false, true, true, 1);
    }
  }
#undef DWA_WAVE
  return hip_fail(hipGetLastError(), "wave hop launch");
}

template <typename SO, typename SI>
int launch_to_sm_p(dwa_ctx* ctx, void* dst, const void* src, double scale, int nrhs, const double* scales) {
  constexpr int NSB = 128 / sizeof(typename SI::elem);
  const dim3 grid((unsigned)((ctx->Vh + NSB - 1) / NSB), (unsigned)nrhs);
  constexpr size_t TE = sizeof(typename SO::elem) < sizeof(typename SI::elem) ? sizeof(typename SO::elem)
                                                                             : sizeof(typename SI::elem);
  hipLaunchKernelGGL((relayout_kernel<SO, SI, true, false>), grid, dim3(256), size_t(12) * ctx->Ls * (NSB + 1) * TE,
                     ctx->stream, (typename SO::elem*)dst, (typename SI::elem*)const_cast<void*>(src), ctx->Ls,
                     (unsigned)ctx->Vh, scale, scales);
  return hip_fail(hipGetLastError(), "relayout launch");
}
template <typename SO, typename SI, bool ADD>
int launch_from_sm_p(dwa_ctx* ctx, void* dst, void* src, double scale, int nrhs, const double* scales) {
  constexpr int NSB = 128 / sizeof(typename SO::elem);
  const dim3 grid((unsigned)((ctx->Vh + NSB - 1) / NSB), (unsigned)nrhs);
  constexpr size_t TE = sizeof(typename SO::elem) < sizeof(typename SI::elem) ? sizeof(typename SO::elem)
                                                                             : sizeof(typename SI::elem);
  hipLaunchKernelGGL((relayout_kernel<SO, SI, false, ADD>), grid, dim3(256), size_t(12) * ctx->Ls * (NSB + 1) * TE,
                     ctx->stream, (typename SO::elem*)dst, (typename SI::elem*)src, ctx->Ls, (unsigned)ctx->Vh, scale,
                     scales);
  return hip_fail(hipGetLastError(), "relayout launch");
}

// blocks of the vector updates per field: every block sums the hops' partials, so there are
// few of them for a large field
inline int vec_grid(size_t nvec) { return grid_for(nvec, 256, 2048); }

template <typename S>
int launch_vec_update1_p(dwa_ctx* ctx, void* x, void* r, const void* p, const void* q, DevScalars* s,
                         double* partials, int* nblocks, int nrhs, const double* qparts, int nq,
                         const double* zparts, int nz) {
  using E = typename S::elem;
  const size_t nvec = field_elems(ctx) / kVec<S>;
  const int grid = vec_grid(nvec);
  hipLaunchKernelGGL(vec_update1_kernel<S>, dim3(grid, nrhs), dim3(256), 0, ctx->stream,
                     (typename XAcc<S>::type::elem*)x, (E*)r, (const E*)p, (const E*)q, s, nvec, partials, qparts, nq,
                     zparts, nz);
  *nblocks = grid;
  return hip_fail(hipGetLastError(), "vector update 1 launch");
}
template <typename S>
int launch_vec_update2_p(dwa_ctx* ctx, void* p, const void* z, DevScalars* s, int nrhs, const double* zparts, int nz) {
  using E = typename S::elem;
  const size_t nvec = field_elems(ctx) / kVec<S>;
  hipLaunchKernelGGL(vec_update2_kernel<S>, dim3(vec_grid(nvec), nrhs), dim3(256), 0, ctx->stream, (E*)p, (const E*)z,
                     s, nvec, zparts, nz);
  return hip_fail(hipGetLastError(), "vector update 2 launch");
}

template <typename S>
int launch_gather_links_p(dwa_ctx* ctx, void* dst, const void* src) {
  hipLaunchKernelGGL(gather_links_kernel<S>, dim3(grid_for(size_t(8) * ctx->V, 256)), dim3(256), 0, ctx->stream,
                     (typename S::elem*)dst, (const double2*)src, ctx->dims[0], ctx->dims[1], ctx->dims[2],
                     ctx->dims[3], ctx->antiperiodic_t, (unsigned)ctx->V);
  return hip_fail(hipGetLastError(), "gather links launch");
}

#define DWA_INSTANTIATE_WAVE(S)                                                                                  \
  namespace dwa {                                                                                                \
  template int launch_wave_hop_p<S>(dwa_ctx*, const WaveOp&, int*);                                              \
  template int launch_gather_links_p<S>(dwa_ctx*, void*, const void*);                                           \
  template int launch_to_sm_p<S, S>(dwa_ctx*, void*, const void*, double, int, const double*);                   \
  template int launch_from_sm_p<S, S, false>(dwa_ctx*, void*, void*, double, int, const double*);                \
  template int launch_vec_update1_p<S>(dwa_ctx*, void*, void*, const void*, const void*, DevScalars*, double*, int*, \
                                       int, const double*, int, const double*, int);                             \
  template int launch_vec_update2_p<S>(dwa_ctx*, void*, const void*, DevScalars*, int, const double*, int);      \
  }
// FP64 SoA -> low-precision site-major
#define DWA_INSTANTIATE_WAVE_LOW(S)                                                                              \
  namespace dwa {                                                                                                \
  template int launch_to_sm_p<S, F64>(dwa_ctx*, void*, const void*, double, int, const double*);                 \
  }
// accumulated low-precision solution, site-major FP32 -> FP64 SoA
#define DWA_INSTANTIATE_WAVE_FOLD(S)                                                                             \
  namespace dwa {                                                                                                \
  template int launch_from_sm_p<F64, S, true>(dwa_ctx*, void*, void*, double, int, const double*);               \
  }

}  // namespace dwa
