// The 4D Wilson operator on canonical FP64 fields: out = (4 + M5) in - 1/2 H in
// (eq.(wilson)), straight from and to the caller's [n][V][4][3] arrays.
#include "kwave.h"

namespace dwa {
namespace {

struct DwArgs {
  const double2* in;
  double2* out;
  const double2* links;  // SoA [2][4][9][Vh], boundary phase folded
  double diag;
  unsigned Lx, Ly, Lz, Lt, ZB;
  unsigned V, n;
};

struct DwSite {
  unsigned lex, x, y, z, t;
};
// position i of the walk (x, y, z in its group of ZB planes, t, z group)
__device__ __forceinline__ DwSite dw_site(const DwArgs& a, unsigned i) {
  DwSite s;
  const unsigned q1 = i / a.Lx, q2 = q1 / a.Ly, q3 = q2 / a.ZB, q4 = q3 / a.Lt;
  s.x = i - q1 * a.Lx;
  s.y = q1 - q2 * a.Ly;
  s.t = q3 - q4 * a.Lt;
  s.z = q4 * a.ZB + (q2 - q3 * a.ZB);
  s.lex = ((s.t * a.Lz + s.z) * a.Ly + s.y) * a.Lx + s.x;
  return s;
}
// the neighbour of site lex (coordinate c of L, stride apart) one step on or back
__device__ __forceinline__ unsigned dw_next(unsigned lex, unsigned c, unsigned L, unsigned stride) {
  return c + 1 == L ? lex - (L - 1) * stride : lex + stride;
}
__device__ __forceinline__ unsigned dw_prev(unsigned lex, unsigned c, unsigned L, unsigned stride) {
  return c == 0 ? lex + (L - 1) * stride : lex - stride;
}

template <int CTRL>
__device__ __forceinline__ cpx<double> quad_pick(const cpx<double>& v) {
  return cmk<double>(quad_perm<double, CTRL>(v.re), quad_perm<double, CTRL>(v.im));
}

constexpr unsigned kDwSites = 16;  // sites of a block
constexpr unsigned kDwWaves = 4;   // its waves, one field each

// A block computes 16 sites of 4 fields: its waves share the sites' 72 link matrices in LDS,
// and lane (site q, spin g) = (lane / 4, lane % 4) multiplies its own spin of each neighbour
// by them.  gamma_mu of the difference of the two hops along mu is exchanged within the quad.
//
// 12 fields of 16^3 x 32: 295 us against 1004 us of packing both parities (4 x 90 us in runs
// of 16 bytes at 192-byte steps), the parity-wise hop (2 x 320 us) and unpacking; one field
// 40 us.  The bytes it cannot do without take 131 us at 5.2 TB/s.  In the way stand, each at
// half to three quarters of its rate: the address unit (a load of 16 bytes at 48-byte steps
// touches 32 lines), FP64 issue (763 instructions per 16 sites) and 0.9 GB of reads (each
// XCD's share of a t-slice and its neighbours' does not stay in its 4 MB L2).  What takes load
// off one of them puts it on another: spinors read in runs of 64 bytes and turned through LDS
// 318 us, through lane exchanges 314; two or three fields a wave 303 and 289 us (but 57 and
// 111 us for one field); six or twelve waves a block 311 and 292 us (52 and 69 us).
__global__ void __launch_bounds__(64 * kDwWaves) dw_kernel(DwArgs a) {
  constexpr unsigned S = kDwSites;
  __shared__ __align__(16) double2 lnk[72 * S];  // [8 directions][9][site], backward daggered
  const unsigned p0 = xcd_range(blockIdx.x, gridDim.x) * S;  // (V is a multiple of 16)
  const unsigned Vh = a.V / 2, sy = a.Lx, sz = sy * a.Ly, st = sz * a.Lz;
  {
    const unsigned j = threadIdx.x % S;
    const DwSite s = dw_site(a, p0 + j);
    const unsigned par = (s.x + s.y + s.z + s.t) & 1u;
    for (unsigned k = threadIdx.x / S; k < 72; k += 64 * kDwWaves / S) {
      const unsigned dir = k / 9, e = k - dir * 9, mu = dir & 3;
      double2 v;
      if (dir < 4) {
        v = a.links[(size_t(par * 4 + mu) * 9 + e) * Vh + (s.lex >> 1)];
      } else {
        const unsigned nb = mu == 0 ? dw_prev(s.lex, s.x, a.Lx, 1)
                                    : (mu == 1 ? dw_prev(s.lex, s.y, a.Ly, sy)
                                               : (mu == 2 ? dw_prev(s.lex, s.z, a.Lz, sz)
                                                          : dw_prev(s.lex, s.t, a.Lt, st)));
        const unsigned r = e / 3, et = (e - r * 3) * 3 + r;
        v = a.links[(size_t((1 - par) * 4 + mu) * 9 + et) * Vh + (nb >> 1)];
        v.y = -v.y;
      }
      lnk[k * S + j] = v;
    }
  }
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane & 3;
  const unsigned j = unsigned(lane) >> 2;
  const DwSite w = dw_site(a, p0 + j);
  const unsigned f = blockIdx.y * kDwWaves + unsigned(wid);
  __syncthreads();
  if (f >= a.n) return;
  const unsigned nf[4] = {dw_next(w.lex, w.x, a.Lx, 1), dw_next(w.lex, w.y, a.Ly, sy),
                          dw_next(w.lex, w.z, a.Lz, sz), dw_next(w.lex, w.t, a.Lt, st)};
  const unsigned nb[4] = {dw_prev(w.lex, w.x, a.Lx, 1), dw_prev(w.lex, w.y, a.Ly, sy),
                          dw_prev(w.lex, w.z, a.Lz, sz), dw_prev(w.lex, w.t, a.Lt, st)};
  // (a field is below 4 GB: the context's limit on a half field)
  const __amdgpu_buffer_rsrc_t ri = make_rsrc(a.in + size_t(f) * a.V * 12, a.V * 192u);
  using C = cpx<double>;
  C H[3], d[3], u0[3], u1[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) H[c] = cmk<double>(0, 0);
  auto load = [&](C(&p)[3], unsigned site) {
    const unsigned off = site * 192u + unsigned(g) * 48u;
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = ldbuf<F64>(ri, off + unsigned(c) * 16u, 0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mul = [&](const C(&p)[3], const double2* u, auto bwd) {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const double2 e0 = u[3 * r * S], e1 = u[(3 * r + 1) * S], e2 = u[(3 * r + 2) * S];
      C t;
      t.re = e0.x * p[0].re;
      t.im = e0.x * p[0].im;
      t.re = fma(-e0.y, p[0].im, t.re);
      t.im = fma(e0.y, p[0].re, t.im);
      t.re = fma(e1.x, p[1].re, t.re);
      t.im = fma(e1.x, p[1].im, t.im);
      t.re = fma(-e1.y, p[1].im, t.re);
      t.im = fma(e1.y, p[1].re, t.im);
      t.re = fma(e2.x, p[2].re, t.re);
      t.im = fma(e2.x, p[2].im, t.im);
      t.re = fma(-e2.y, p[2].im, t.re);
      t.im = fma(e2.y, p[2].re, t.im);
      H[r] = H[r] + t;
      if constexpr (decltype(bwd)::value) d[r] = t - d[r];
      else d[r] = t;
    }
    // the sums are taken here: left open, the products of all eight hops are held (168
    // registers instead of 76)
#pragma unroll
    for (int c = 0; c < 3; ++c) asm volatile("" : "+v"(H[c].re), "+v"(H[c].im), "+v"(d[c].re), "+v"(d[c].im));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // the next hop's spinors are loaded ahead of this one's products
  load(u0, nf[0]);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    load(u1, nb[mu]);
    mul(u0, lnk + mu * 9 * S + j, std::false_type());
    if (mu < 3) load(u0, nf[mu < 3 ? mu + 1 : 3]);
    mul(u1, lnk + (4 + mu) * 9 * S + j, std::true_type());
#pragma unroll
    for (int c = 0; c < 3; ++c) add_gamma<double>(mu, g, d[c], H[c]);
  }
  // the sites' own spinors and the stores in runs of 64 bytes a quad: lane g takes the
  // components 4 m + g, from lane (4 m + g) / 3 and colour (4 m + g) % 3
  const unsigned off = w.lex * 12u + unsigned(g);
  C x[3];
#pragma unroll
  for (int m = 0; m < 3; ++m) x[m] = ldbuf<F64>(ri, (off + unsigned(m) * 4u) * 16u, 0);
  const C h0[3] = {quad_pick<0x40>(H[0]), quad_pick<0x40>(H[1]), quad_pick<0x40>(H[2])};
  const C h1[3] = {quad_pick<0xA5>(H[0]), quad_pick<0xA5>(H[1]), quad_pick<0xA5>(H[2])};
  const C h2[3] = {quad_pick<0xFE>(H[0]), quad_pick<0xFE>(H[1]), quad_pick<0xFE>(H[2])};
  const int rot = g == 3 ? 0 : g;
  const C h[3] = {rot == 0 ? h0[0] : (rot == 1 ? h0[1] : h0[2]), rot == 0 ? h1[1] : (rot == 1 ? h1[2] : h1[0]),
                  rot == 0 ? h2[2] : (rot == 1 ? h2[0] : h2[1])};
  dwa_v2d* o = reinterpret_cast<dwa_v2d*>(a.out + size_t(f) * a.V * 12 + off);
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const dwa_v2d v = {a.diag * x[m].re - 0.5 * h[m].re, a.diag * x[m].im - 0.5 * h[m].im};
    __builtin_nontemporal_store(v, o + 4 * m);
  }
}

}  // namespace

int launch_dw(dwa_ctx* ctx, void* out, const void* in, int n) {
  DwArgs a;
  a.links = (const double2*)ctx->prec[DWA_F64].links;
  a.diag = 4.0 + ctx->M5;
  a.Lx = (unsigned)ctx->dims[0];
  a.Ly = (unsigned)ctx->dims[1];
  a.Lz = (unsigned)ctx->dims[2];
  a.Lt = (unsigned)ctx->dims[3];
  // each XCD a group of z-planes, walked in t, whose two neighbours in t stay in its L2
  // (295 us; plain order 310)
  a.ZB = a.Lz % 8 == 0 ? a.Lz / 8 : a.Lz;
  a.V = (unsigned)ctx->V;
  constexpr int most = 65535 * int(kDwWaves);  // grid limit
  for (int s0 = 0; s0 < n; s0 += most) {
    a.n = unsigned(n - s0 < most ? n - s0 : most);
    a.in = (const double2*)in + size_t(s0) * a.V * 12;
    a.out = (double2*)out + size_t(s0) * a.V * 12;
    const dim3 grid(a.V / kDwSites, (a.n + kDwWaves - 1) / kDwWaves);
    hipLaunchKernelGGL(dw_kernel, grid, dim3(64 * kDwWaves), 0, ctx->stream, a);
    const int rc = hip_fail(hipGetLastError(), "Wilson operator launch");
    if (rc) return rc;
  }
  return DWA_OK;
}

}  // namespace dwa
