// Field preparation: the clover term A(x) from the plaquette leaves and its
// inverse, both stored as two packed Hermitian 6x6 chirality blocks (Sec. 3:
// 6 real diagonal entries plus 15 complex upper-triangle entries per block;
// the full inverse is stored instead of an LU factorisation).  FP64.
#include "dd_internal.h"

namespace {

struct M3 {
  cx<double> a[3][3];
};

__device__ __forceinline__ M3 mul(const M3& x, const M3& y) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      cx<double> s = {0.0, 0.0};
#pragma unroll
      for (int j = 0; j < 3; ++j) cfma(s, x.a[i][j], y.a[j][k]);
      r.a[i][k] = s;
    }
  return r;
}
__device__ __forceinline__ M3 dag(const M3& x) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) r.a[i][k] = conj(x.a[k][i]);
  return r;
}

__device__ __forceinline__ SiteLoc step(const GeomDev& g, SiteLoc s, int mu, int sign) {
  int v = s.l[mu] + sign;
  if (v < 0 || v >= g.b[mu]) {
    int e = g.blk_nbr[(sign > 0 ? mu : 4 + mu) * g.Vc + s.slot];
    s.slot = e & DD_SLOT_MASK;
    v = (sign > 0) ? 0 : g.b[mu] - 1;
  }
  s.l[mu] = v;
  return s;
}

__device__ __forceinline__ M3 link(const GeomDev& g, const double2* L, const SiteLoc& s, int mu) {
  long long I = ((long long)s.slot << g.lBv) + encode_local(g, s.l);
  M3 u;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    double2 v = L[(long long)(mu * 9 + k) * g.V + I];
    u.a[k / 3][k % 3] = {v.x, v.y};
  }
  return u;
}

// sum of the four leaves of the mu-nu plane at x (same orientation; raw links,
// so the t boundary factor cancels in every closed path): closed paths of the
// steps +mu, +nu, -mu, -nu, each leaf starting one step later.  Rolled, one link
// live at a time; all sixteen at once do not fit the registers.
__device__ __forceinline__ M3 leaves(const GeomDev& g, const double2* L, const SiteLoc& x, int mu, int nu) {
  M3 q;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) q.a[i][k] = {0.0, 0.0};
#pragma unroll 1
  for (int leaf = 0; leaf < 4; ++leaf) {
    SiteLoc s = x;
    M3 p;
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
      const int d = (leaf + j) & 3, dir = d & 1 ? nu : mu;
      if (d >= 2) s = step(g, s, dir, -1);
      M3 u = link(g, L, s, dir);
      if (d >= 2) u = dag(u);
      else s = step(g, s, dir, +1);
      p = j == 0 ? u : mul(p, u);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) q.a[i][k] = q.a[i][k] + p.a[i][k];
  }
  return q;
}

// The 2x2 spin blocks of the chiral gamma matrices, gamma_mu = [[0, A_mu],
// [A_mu^dag, 0]], in whole numbers; the spin block of gamma_mu gamma_nu on
// chirality c (c = 0: A_mu A_nu^dag, c = 1: A_mu^dag A_nu) then has entries 0, +-1, +-i
// known at compile time.
struct Unit {
  int re, im;
};
__host__ __device__ constexpr Unit Amat(int mu, int r, int c) {
  return mu == 0 ? (r != c ? Unit{0, -1} : Unit{0, 0})
       : mu == 1 ? (r == c ? Unit{0, 0} : (r == 0 ? Unit{-1, 0} : Unit{1, 0}))
       : mu == 2 ? (r != c ? Unit{0, 0} : (r == 0 ? Unit{0, -1} : Unit{0, 1}))
                 : (r == c ? Unit{1, 0} : Unit{0, 0});
}
__host__ __device__ constexpr Unit mul_conj(Unit a, Unit b) { return {a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im}; }
__host__ __device__ constexpr Unit gg(int c, int mu, int nu, int r, int s) {
  Unit t{0, 0};
  for (int k = 0; k < 2; ++k) {
    const Unit u = c == 0 ? mul_conj(Amat(mu, r, k), Amat(nu, s, k)) : mul_conj(Amat(nu, k, s), Amat(mu, k, r));
    t.re += u.re;
    t.im += u.im;
  }
  return t;
}
// planes in the order (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
__host__ __device__ constexpr int plane_mu(int p) { return p < 3 ? 0 : p < 5 ? 1 : 2; }
__host__ __device__ constexpr int plane_nu(int p) { return p < 3 ? p + 1 : p < 5 ? p - 1 : 3; }

template <int Re, int Im>
__device__ __forceinline__ cx<double> unit_times(cx<double> a) {
  if (Re == 1) return a;
  if (Re == -1) return -a;
  if (Im == 1) return times_i(a);
  return times_mi(a);
}

constexpr int kSites = 64;   // sites per workgroup: one lane each, six waves (planes)

// block (al, be) of chirality C of sum_p (gamma_mu gamma_nu)(al, be) F_p, entry (a, b)
template <int C, int AL, int BE, int PL = 0>
__device__ __forceinline__ cx<double> plane_sum(const double (*F)[9][kSites], int site, int a, int b, cx<double> acc) {
  if constexpr (PL < 6) {
    constexpr Unit u = gg(C, plane_mu(PL), plane_nu(PL), AL, BE);
    if constexpr (u.re != 0 || u.im != 0) {
      cx<double> f;   // F is antihermitian: three imaginary diagonals, three upper entries
      if (a == b) f = {0.0, F[PL][a][site]};
      else {
        const int q = a + b - 1;                       // (0,1) 0, (0,2) 1, (1,2) 2
        f = {F[PL][3 + 2 * q][site], F[PL][4 + 2 * q][site]};
        if (a > b) f = {-f.re, f.im};                  // F_ba = -conj(F_ab)
      }
      acc = acc + unit_times<u.re, u.im>(f);
    }
    return plane_sum<C, AL, BE, PL + 1>(F, site, a, b, acc);
  } else {
    return acc;
  }
}

template <int C>
__device__ __forceinline__ void clover_block(const double (*F)[9][kSites], int site, double m0, double csw,
                                             double2* __restrict__ out, long long V) {
  auto entry = [&](int r, int c) -> cx<double> {   // r <= c
    const int a = r % 3, b = c % 3;
    cx<double> z = {0.0, 0.0};
    if (r < 3 && c < 3) z = plane_sum<C, 0, 0>(F, site, a, b, z);
    else if (r < 3) z = plane_sum<C, 0, 1>(F, site, a, b, z);
    else z = plane_sum<C, 1, 1>(F, site, a, b, z);
    z = (-0.5 * csw) * z;
    return r == c ? cx<double>{4.0 + m0 + z.re, 0.0} : z;
  };
#pragma unroll
  for (int k = 0; k < 3; ++k) out[k * V] = make_double2(entry(2 * k, 2 * k).re, entry(2 * k + 1, 2 * k + 1).re);
  int k = 3;
#pragma unroll
  for (int r = 0; r < 6; ++r)
#pragma unroll
    for (int c = r + 1; c < 6; ++c) {
      const cx<double> z = entry(r, c);
      out[(k++) * V] = make_double2(z.re, z.im);
    }
}

template <int PL>
__device__ __forceinline__ void plane_field(const GeomDev& g, const double2* L, const SiteLoc& x, double (*F)[kSites],
                                            int site) {
  // F = (Q_mu,nu - Q_nu,mu) / 8 with Q_nu,mu = Q_mu,nu^dagger
  const M3 Q = leaves(g, L, x, plane_mu(PL), plane_nu(PL));
#pragma unroll
  for (int a = 0; a < 3; ++a) F[a][site] = 0.25 * Q.a[a][a].im;
  int q = 3;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a + 1; b < 3; ++b) {
      F[q++][site] = 0.125 * (Q.a[a][b].re - Q.a[b][a].re);
      F[q++][site] = 0.125 * (Q.a[a][b].im + Q.a[b][a].im);
    }
}

// A(x) of 64 sites per workgroup: wave p forms the field strength of plane p (16
// link loads and 12 matrix products per site and plane), then two waves assemble
// the two chirality blocks from LDS.  Everything is indexed at compile time, so
// nothing goes through scratch memory, which is what bound the one-thread-per-site
// form (with the inverse 2.74 ms at 16^3x32, now 250 + 38 us).
__global__ void __launch_bounds__(6 * kSites) k_clover(GeomDev g, const double2* __restrict__ L, double m0, double csw,
                                                       double2* __restrict__ clov) {
  __shared__ double F[6][9][kSites];
  const int w = threadIdx.x >> 6, site = threadIdx.x & 63;
  const long long I = (long long)blockIdx.x * kSites + site;
  const bool ok = I < g.V;
  const SiteLoc x = decode_site(g, ok ? I : 0);
  if (csw != 0.0) {
    switch (w) {
      case 0: plane_field<0>(g, L, x, F[0], site); break;
      case 1: plane_field<1>(g, L, x, F[1], site); break;
      case 2: plane_field<2>(g, L, x, F[2], site); break;
      case 3: plane_field<3>(g, L, x, F[3], site); break;
      case 4: plane_field<4>(g, L, x, F[4], site); break;
      default: plane_field<5>(g, L, x, F[5], site); break;
    }
  } else {
#pragma unroll
    for (int k = 0; k < 9; ++k) F[w][k][site] = 0.0;
  }
  __syncthreads();
  if (!ok) return;
  if (w == 0) clover_block<0>(F, site, m0, csw, clov + I, g.V);
  if (w == 1) clover_block<1>(F, site, m0, csw, clov + 18 * g.V + I, g.V);
}

// Inverse of one packed Hermitian 6x6 block per thread: Gauss-Jordan with partial
// pivoting in FP64, in place in registers (row exchanges by selects, the column
// exchanges they imply undone at the end)
__global__ void __launch_bounds__(128) k_clover_inv(long long V, const double2* __restrict__ clov,
                                                    double2* __restrict__ cinv) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 2 * V) return;
  const int ch = i >= V ? 1 : 0;
  const double2* in = clov + (long long)(18 * ch) * V + (i - ch * V);
  double2* out = cinv + (long long)(18 * ch) * V + (i - ch * V);
  cx<double> M[6][6];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double2 v = in[k * V];
    M[2 * k][2 * k] = {v.x, 0.0};
    M[2 * k + 1][2 * k + 1] = {v.y, 0.0};
  }
  int e = 3;
#pragma unroll
  for (int r = 0; r < 6; ++r)
#pragma unroll
    for (int c = r + 1; c < 6; ++c) {
      const double2 v = in[(e++) * V];
      M[r][c] = {v.x, v.y};
      M[c][r] = {v.x, -v.y};
    }
  int piv[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    int p = k;
    double best = M[k][k].re * M[k][k].re + M[k][k].im * M[k][k].im;
#pragma unroll
    for (int r = k + 1; r < 6; ++r) {
      const double v = M[r][k].re * M[r][k].re + M[r][k].im * M[r][k].im;
      if (v > best) {
        best = v;
        p = r;
      }
    }
    piv[k] = p;
#pragma unroll
    for (int r = k + 1; r < 6; ++r) {
      const bool s = p == r;
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        const cx<double> a = M[k][c], b = M[r][c];
        M[k][c] = {s ? b.re : a.re, s ? b.im : a.im};
        M[r][c] = {s ? a.re : b.re, s ? a.im : b.im};
      }
    }
    const cx<double> q = M[k][k];
    const double d = q.re * q.re + q.im * q.im;
    const cx<double> inv = {q.re / d, -q.im / d};
#pragma unroll
    for (int c = 0; c < 6; ++c)
      if (c != k) M[k][c] = M[k][c] * inv;
    M[k][k] = inv;
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      if (r == k) continue;
      const cx<double> f = M[r][k];
#pragma unroll
      for (int c = 0; c < 6; ++c)
        if (c != k) M[r][c] = M[r][c] - f * M[k][c];
      M[r][k] = -(f * inv);
    }
  }
#pragma unroll
  for (int k = 5; k >= 0; --k)
#pragma unroll
    for (int c = k + 1; c < 6; ++c) {
      const bool s = piv[k] == c;
#pragma unroll
      for (int r = 0; r < 6; ++r) {
        const cx<double> a = M[r][k], b = M[r][c];
        M[r][k] = {s ? b.re : a.re, s ? b.im : a.im};
        M[r][c] = {s ? a.re : b.re, s ? a.im : b.im};
      }
    }
#pragma unroll
  for (int k = 0; k < 3; ++k) out[k * V] = make_double2(M[2 * k][2 * k].re, M[2 * k + 1][2 * k + 1].re);
  e = 3;
#pragma unroll
  for (int r = 0; r < 6; ++r)
#pragma unroll
    for (int c = r + 1; c < 6; ++c) out[(e++) * V] = make_double2(M[r][c].re, M[r][c].im);
}

}  // namespace

void launch_clover_build(const GeomDev& g, const double2* links64, double m0, double csw, double2* clover64,
                         double2* cinv64, hipStream_t st) {
  k_clover<<<(unsigned)((g.V + kSites - 1) / kSites), 6 * kSites, 0, st>>>(g, links64, m0, csw, clover64);
  k_clover_inv<<<(unsigned)((2 * g.V + 127) / 128), 128, 0, st>>>(g.V, clover64, cinv64);
}
