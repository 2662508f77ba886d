// SAP smoother for small domains (at most 128 sites), a site's work split over the
// waves of a workgroup.  Same iteration as sap.hip.
//
// A wave of the one-thread-per-site kernel has 8 of its 64 lanes busy on a 2^4
// domain, and each lane goes through eight hops, one link read after another.  Here
// the 64 lanes of a workgroup's eight waves are the sites of one or more (domain,
// right-hand side) pairs, and
//   wave d       does the hop in direction d of every lane's site (d >> 1 = mu, odd:
//                backward), its even and odd site's links in registers throughout;
//   wave w < 6   owns the rows of colour w % 3 in the chirality w / 3: it adds the
//                eight hops up, applies its two rows of A_ee or A_oo^-1 (in registers
//                as well) and keeps those rows of every vector.
// Half spinors and vectors change hands through LDS, six barriers a step, and the MR
// loop reads no memory but A_ee.  Bound by that chain of barriers and LDS round
// trips, in FP64 by the products as well.  One pair on a 2^4 domain holds every site
// eight times in a wave: its lanes then take single entries of the half spinors and
// single rows (ROWS).  us per launch (four MR steps), one thread per site / here: 4^4, 2^4
// domains, one right-hand side FP64 101 / 25, FP32 94 / 22 (45 and 28 with whole half
// spinors to a lane, idle lanes masked off 60); 16^4, FP64 one 505 / 72, FP32 twelve
// 2612 / 344.  (A_oo^-1 read in every step as well: 48 instead of 45 at 4^4; four FP32
// waves per SIMD, which spill: 37 instead of 28.)
#include "dslash.h"
#include "ktimer.h"

namespace {

// row a of the 6x6 block `half` of a packed clover-like field at site I
template <typename R, typename S>
__device__ __forceinline__ void load_row(const S* C, long long V, long long I, int half, int a, cx<R>* m) {
  const S* B = C + (long long)(18 * half) * V + I;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const int lo = a < q ? a : q, hi = a < q ? q : a;
    const cx<R> u = ld<R, S>(B + (a == q ? a >> 1 : 3 + lo * (11 - lo) / 2 + hi - lo - 1) * V);
    m[q] = a == q ? cx<R>{(a & 1) ? u.im : u.re, (R)0} : a < q ? u : conj(u);
  }
}
template <typename R>
__device__ __forceinline__ cx<R> apply_row(const cx<R>* m, const cx<R>* v) {
  cx<R> o = cmul2(m[0], v[0]);
#pragma unroll
  for (int q = 1; q < 6; ++q) cfma4(o, m[q], v[q]);
  return o;
}

// colour c of spin s of a projected spinor psi(component): psi_up + SGN A_mu psi_dn
template <int MU, int SGN, typename R, typename Psi>
__device__ __forceinline__ cx<R> project_one(Psi psi, int s, int c) {
  const cx<R> u = psi(3 * s + c), d = psi(6 + 3 * (MU < 2 ? 1 - s : s) + c);
  const R sg = s ? (R)1 : (R)-1;
  const cx<R> t = MU == 0 ? times_mi(d) : MU == 1 ? sg * d : MU == 2 ? sg * times_i(d) : d;
  return SGN > 0 ? u + t : u - t;
}

// ROWS: eight sites and one pair, and the lanes hold a site eight times: each hop lane
// takes one of the half spinor's six entries, each row lane one row (the same sums).
template <typename R, typename S, typename Tv, bool ROWS>
__global__ void __launch_bounds__(512)
k_sap_split(GeomDev g, const S* __restrict__ links, const S* __restrict__ clov, const S* __restrict__ cinv, int nrhs,
            int per, int colour, int mr_iters, const Tv* __restrict__ bvec, Tv* __restrict__ xvec) {
  __shared__ cx<R> part[8][6][64];   // scaled half spinors of the eight hops
  __shared__ cx<R> vec[12][64];      // the vector that hops read
  __shared__ cx<R> row[12][64];      // the vector that rows of A_oo^-1 read
  __shared__ R red[6][3][8];
  const int lbh = g.lBv - 1;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int j = lane & (g.Bvh - 1), copy = lane >> lbh, q = ROWS ? 0 : copy;
  // the (domain, right-hand side) pairs in order, per of them a workgroup, each XCD a contiguous eighth of the domains
  const int dom_x = g.Vch / 8, pair = (blockIdx.x >> 3) * per + q;
  const bool act = q < per && pair < dom_x * nrhs;
  const int pc = act ? pair : 0, r = pc % nrhs, slot = colour * g.Vch + (blockIdx.x & 7) * dom_x + pc / nrhs;
  const long long V = g.V;
  const Tv* b = bvec + (long long)r * 12 * V;
  Tv* x = xvec + (long long)r * 12 * V;
  const long long I[2] = {((long long)slot << g.lBv) + j, ((long long)slot << g.lBv) + g.Bvh + j};   // even, odd site

  // hops of direction w
  const int mu = w >> 1;
  const bool fwd = (w & 1) == 0;
  long long J[2];
  bool in[2];
  R coef[2];
  const int hk = copy < 6 ? copy : copy - 6, hs = hk / 3, hc = hk % 3;   // ROWS: the hop lane's entry
  const int at = ROWS ? j : lane;                                        // the site's column in LDS
  cx<R> u[2][ROWS ? 3 : 9];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    bool wrap;
    J[p] = neighbor(g, decode_site(g, I[p]), mu, fwd ? +1 : -1, wrap, in[p]);
    coef[p] = (R)(wrap ? -0.5 * g.bc_t : -0.5);
    if constexpr (!ROWS) load_link<R, S>(links, V, mu, fwd ? I[p] : J[p], u[p]);
    else
#pragma unroll
      for (int k = 0; k < 3; ++k)   // a row of U, or a column for U^dag
        u[p][k] = ld<R, S>(links + (mu * 9 + (fwd ? 3 * hc + k : 3 * k + hc)) * V + (fwd ? I[p] : J[p]));
  }
  auto hop = [&](int p, bool on, auto psi) {   // psi(c): component c of the neighbour's spinor
    if constexpr (ROWS) {
      cx<R> h[3], o;
#pragma unroll
      for (int c = 0; c < 3; ++c) switch (w) {
          case 0: h[c] = project_one<0, -1, R>(psi, hs, c); break;
          case 1: h[c] = project_one<0, +1, R>(psi, hs, c); break;
          case 2: h[c] = project_one<1, -1, R>(psi, hs, c); break;
          case 3: h[c] = project_one<1, +1, R>(psi, hs, c); break;
          case 4: h[c] = project_one<2, -1, R>(psi, hs, c); break;
          case 5: h[c] = project_one<2, +1, R>(psi, hs, c); break;
          case 6: h[c] = project_one<3, -1, R>(psi, hs, c); break;
          default: h[c] = project_one<3, +1, R>(psi, hs, c); break;
        }
      if (fwd) {
        o = cmul2(u[p][0], h[0]);
        cfma4(o, u[p][1], h[1]);
        cfma4(o, u[p][2], h[2]);
      } else {
        o = cmul2_conj(u[p][0], h[0]);
        cfma4_conj(o, u[p][1], h[1]);
        cfma4_conj(o, u[p][2], h[2]);
      }
      part[w][hk][at] = on ? coef[p] * o : cx<R>{(R)0, (R)0};
    } else {
      cx<R> v[12], h[6], uh[6];
#pragma unroll
      for (int c = 0; c < 12; ++c) v[c] = psi(c);
      switch (w) {
        case 0: project<0, -1, R>(v, h); break;
        case 1: project<0, +1, R>(v, h); break;
        case 2: project<1, -1, R>(v, h); break;
        case 3: project<1, +1, R>(v, h); break;
        case 4: project<2, -1, R>(v, h); break;
        case 5: project<2, +1, R>(v, h); break;
        case 6: project<3, -1, R>(v, h); break;
        default: project<3, +1, R>(v, h); break;
      }
      if (fwd) su3_mul_half<R>(u[p], h, uh);
      else su3_dag_mul_half<R>(u[p], h, uh);
#pragma unroll
      for (int k = 0; k < 6; ++k) part[w][k][at] = on ? coef[p] * uh[k] : cx<R>{(R)0, (R)0};
    }
  };
  auto hop_x = [&](int p) {   // from x, inside the domain and across its faces
    hop(p, true, [&](int c) { return act ? ld<R, Tv>(x + c * V + J[p]) : cx<R>{(R)0, (R)0}; });
  };
  auto hop_vec = [&](int p) {   // inside the domain, from vec (the other parity's sites)
    const int jj = (at & ~(g.Bvh - 1)) | (int)(J[p] & (g.Bvh - 1));
    hop(p, in[p], [&](int c) { return vec[c][jj]; });
  };

  // rows of waves 0 .. 5: spins 2 half and 2 half + 1 of one colour (ROWS: one of the two)
  constexpr int NR = ROWS ? 1 : 2;
  const bool own = w < 6;
  const int half = own ? w / 3 : 0, col = w % 3;
  auto spin = [&](int i) { return ROWS ? copy & 1 : i; };
  auto comp = [&](int i) { return 6 * half + 3 * spin(i) + col; };
  cx<R> mo[NR][6];   // of A_oo^-1
  if (own)
#pragma unroll
    for (int i = 0; i < NR; ++i) load_row<R, S>(cinv, V, I[1], half, 3 * spin(i) + col, mo[i]);
  // the eight hops' sum in those rows: (uh, s A_mu^dag uh), s = -1 forward, +1 backward
  auto combine = [&](cx<R>* s) {
#pragma unroll
    for (int i = 0; i < NR; ++i) s[i] = {(R)0, (R)0};
#pragma unroll
    for (int d = 0; d < 8; ++d)
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int sp = spin(i);
        if (!half) {
          s[i] = s[i] + part[d][3 * sp + col][at];
          continue;
        }
        const cx<R> h = part[d][3 * (d < 4 ? 1 - sp : sp) + col][at];
        const R sg = (sp ? (R)-1 : (R)1) * ((d & 1) ? (R)1 : (R)-1), sd = (d & 1) ? (R)1 : (R)-1;
        const cx<R> t = d >> 1 == 0 ? sd * times_i(h) : d >> 1 == 1 ? sg * h : d >> 1 == 2 ? sg * times_i(h) : sd * h;
        s[i] = s[i] + t;
      }
  };
  auto put = [&](cx<R>(*dst)[64], const cx<R>* v) {
#pragma unroll
    for (int i = 0; i < NR; ++i) dst[comp(i)][at] = v[i];
  };
  auto rows_of = [&](const cx<R>(*m)[6], const cx<R>(*src)[64], cx<R>* o) {
    cx<R> v[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = src[6 * half + k][at];
#pragma unroll
    for (int i = 0; i < NR; ++i) o[i] = apply_row<R>(m[i], v);
  };
  // b - A x in the own rows
  auto source = [&](int p, cx<R>* o) {
    cx<R> v[6], m[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = act ? ld<R, Tv>(x + (6 * half + k) * V + I[p]) : cx<R>{(R)0, (R)0};
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      load_row<R, S>(clov, V, I[p], half, 3 * spin(i) + col, m);
      o[i] = apply_row<R>(m, v);
      if (act) o[i] = ld<R, Tv>(b + comp(i) * V + I[p]) - o[i];
    }
  };
  auto minus = [&](cx<R>* a, const cx<R>* c) {
#pragma unroll
    for (int i = 0; i < NR; ++i) a[i] = a[i] - c[i];
  };

  cx<R> rho[NR], e[NR], ro[NR], s[NR], t[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) e[i] = {(R)0, (R)0};
  // r_o = b - D x
  hop_x(1);
  if (own) source(1, ro);
  __syncthreads();
  if (own) {
    combine(s);
    minus(ro, s);
    put(row, ro);
  }
  __syncthreads();
  // r_e = b - D x, and A_oo^-1 r_o
  hop_x(0);
  if (own) {
    rows_of(mo, row, t);
    put(vec, t);
    source(0, rho);
  }
  __syncthreads();
  if (own) {
    combine(s);
    minus(rho, s);
  }
  __syncthreads();
  // rho = r_e - H_eo A_oo^-1 r_o
  hop_vec(0);
  __syncthreads();
  if (own) {
    combine(s);
    minus(rho, s);
  }
#pragma unroll 1
  for (int k = 0; k < mr_iters; ++k) {
    if (own) put(vec, rho);
    __syncthreads();
    hop_vec(1);
    if (own) {   // A_ee rho; the operand comes from cache while the hops run
      cx<R> me[NR][6];
      const S* C = clov;
      asm volatile("" : "+s"(C));   // (read in every step: 48 registers kept across the loop would spill)
#pragma unroll
      for (int i = 0; i < NR; ++i) load_row<R, S>(C, V, I[0], half, 3 * spin(i) + col, me[i]);
      rows_of(me, vec, t);
    }
    __syncthreads();
    if (own) {
      combine(s);
      put(row, s);
    }
    __syncthreads();
    if (own) {
      rows_of(mo, row, s);
      put(vec, s);
    }
    __syncthreads();
    hop_vec(0);
    __syncthreads();
    R re = 0, im = 0, pp = 0;
    if (own) {
      combine(s);
      minus(t, s);   // p = A_ee rho - H_eo A_oo^-1 H_oe rho
      mr_sums(t[0], rho[0], re, im, pp);
      if constexpr (ROWS) {
        re += __shfl_xor(re, 8, 64);
        im += __shfl_xor(im, 8, 64);
        pp += __shfl_xor(pp, 8, 64);
      } else {
        R re1 = 0, im1 = 0, pp1 = 0;
        mr_sums(t[NR - 1], rho[NR - 1], re1, im1, pp1);
        re += re1;
        im += im1;
        pp += pp1;
      }
      for (int off = 1; off < g.Bvh; off <<= 1) {
        re += __shfl_xor(re, off, 64);
        im += __shfl_xor(im, off, 64);
        pp += __shfl_xor(pp, off, 64);
      }
      if (j == 0 && (!ROWS || copy == 0)) {
        red[w][0][q] = re;
        red[w][1][q] = im;
        red[w][2][q] = pp;
      }
    }
    __syncthreads();
    if (own) {
      re = im = pp = 0;
#pragma unroll
      for (int d = 0; d < 6; ++d) {
        re += red[d][0][q];
        im += red[d][1][q];
        pp += red[d][2][q];
      }
      cx<R> alpha = {(R)0, (R)0};
      if (pp > (R)0) alpha = {re / pp, im / pp};
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        cfma4(e[i], alpha, rho[i]);
        cfma4(rho[i], -alpha, t[i]);
      }
    }
  }
  // e_o = A_oo^-1 (r_o - H_oe e_e);  x += e
  if (own) put(vec, e);
  __syncthreads();
  hop_vec(1);
  __syncthreads();
  if (own) {
    combine(s);
    minus(ro, s);
    put(row, ro);
  }
  __syncthreads();
  if (own) {
    rows_of(mo, row, s);
    if (act && (!ROWS || copy < 2))
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        Tv* xe = x + comp(i) * V + I[0];
        Tv* xo = x + comp(i) * V + I[1];
        st<Tv, R>(xe, ld<R, Tv>(xe) + e[i]);
        st<Tv, R>(xo, ld<R, Tv>(xo) + s[i]);
      }
  }
}

template <typename R, typename S, typename Tv>
void run_split(const GeomDev& g, const OpSet& ops, int nrhs, int sweeps, int mr, const void* b, void* x,
               hipStream_t st) {
  // (domain, right-hand side) pairs of a workgroup: one while the CUs outnumber them, up
  // to all 64 lanes (no more instructions) on larger lattices or more right-hand sides
  const long long pairs = (long long)(g.Vch / 8) * nrhs;   // of an XCD
  int per = 1;
  while (2 * per <= 64 >> (g.lBv - 1) && (pairs + per - 1) / per > 32) per *= 2;
  const unsigned nb = (unsigned)(8 * ((pairs + per - 1) / per));
  auto* fn = per == 1 && g.Bvh == 8 ? k_sap_split<R, S, Tv, true> : k_sap_split<R, S, Tv, false>;
  // per launch, as k_sap_colour
  const double half = 0.5 * (double)g.V;
  const double bytes = half * (90.0 * sizeof(S) + 36.0 * sizeof(Tv) * nrhs);
  const double flops = half * nrhs * (mr + 2.5) * 1850.0;
  for (int s = 0; s < sweeps; ++s)
    for (int colour = 0; colour < 2; ++colour)
      DD_TIMED("k_sap_colour", st, bytes, flops,
               (fn<<<nb, 512, 0, st>>>(g, (const S*)ops.links, (const S*)ops.clover, (const S*)ops.cinv, nrhs, per,
                                       colour, mr, (const Tv*)b, (Tv*)x)));
}

}  // namespace

// By the lattice and not by the launch, as the sums round differently here.  us per
// launch, one thread per site / split: 16^3x32 with domains of 64 sites FP64 one
// right-hand side 251 / 140, FP32 one 108 / 62, twelve 1178 / 713.  Domains of 128 sites
// fill the lanes either way, and the split pays while few of them leave latency bare:
// 64 domains per colour FP64 one 94 / 52, FP32 twelve 88 / 60; 128 FP64 five right-hand
// sides 105 / 115, FP32 twelve 95 / 88; 512 FP64 five 551 / 614, FP32 twelve 610 / 748.
bool sap_split_use(const GeomDev& g) { return g.Bvh <= 32 || (g.Bvh == 64 && g.Vch <= 64); }

void launch_sap_split(const GeomDev& g, dd_dtype dt, const OpSet& ops, int nrhs, int sweeps, int mr, const void* b,
                      void* x, hipStream_t st) {
  switch (dt) {
    case DD_F64: run_split<double, double2, double2>(g, ops, nrhs, sweeps, mr, b, x, st); break;
    case DD_F32: run_split<float, float2, float2>(g, ops, nrhs, sweeps, mr, b, x, st); break;
    case DD_F16: run_split<float, __half2, float2>(g, ops, nrhs, sweeps, mr, b, x, st); break;
    case DD_BF16: run_split<float, bf16x2, float2>(g, ops, nrhs, sweeps, mr, b, x, st); break;
  }
}
