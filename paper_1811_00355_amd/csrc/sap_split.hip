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
// trips.  us per launch (four MR steps), one thread per site / here: 4^4, 2^4 domains,
// one right-hand side FP64 101 / 45, FP32 94 / 28; 16^4, FP64 one 505 / 70, FP32
// twelve 2612 / 345.  (A_oo^-1 read in every step as well: 48 and 31 at 4^4; four FP32
// waves per SIMD, which spill: 37.)
#include "dslash.h"
#include "ktimer.h"

namespace {

// rows a0 and a0 + 3 of the 6x6 block `half` of a packed clover-like field at site I
template <typename R, typename S>
__device__ __forceinline__ void load_rows(const S* C, long long V, long long I, int half, int a0, cx<R> (*m)[6]) {
  const S* B = C + (long long)(18 * half) * V + I;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const int a = a0 + 3 * i;   // uniform in a wave
      if (a == q) {
        const cx<R> d = ld<R, S>(B + (a >> 1) * V);
        m[i][q] = {(a & 1) ? d.im : d.re, (R)0};
      } else {
        const int lo = a < q ? a : q, hi = a < q ? q : a;
        const cx<R> u = ld<R, S>(B + (3 + lo * (11 - lo) / 2 + hi - lo - 1) * V);
        m[i][q] = a < q ? u : conj(u);
      }
    }
}
template <typename R>
__device__ __forceinline__ void apply_rows(const cx<R> (*m)[6], const cx<R>* v, cx<R>* o) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    o[i] = cmul2(m[i][0], v[0]);
#pragma unroll
    for (int q = 1; q < 6; ++q) cfma4(o[i], m[i][q], v[q]);
  }
}

template <typename R, typename S, typename Tv>
__global__ void __launch_bounds__(512)
k_sap_split(GeomDev g, const S* __restrict__ links, const S* __restrict__ clov, const S* __restrict__ cinv, int nrhs,
            int per, int colour, int mr_iters, const Tv* __restrict__ bvec, Tv* __restrict__ xvec) {
  __shared__ cx<R> part[8][6][64];   // scaled half spinors of the eight hops
  __shared__ cx<R> vec[12][64];      // the vector that hops read
  __shared__ cx<R> row[12][64];      // the vector that rows of A_oo^-1 read
  __shared__ R red[6][3][8];
  const int lbh = g.lBv - 1;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int j = lane & (g.Bvh - 1), q = lane >> lbh;
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
  cx<R> u[2][9];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    bool wrap;
    J[p] = neighbor(g, decode_site(g, I[p]), mu, fwd ? +1 : -1, wrap, in[p]);
    coef[p] = (R)(wrap ? -0.5 * g.bc_t : -0.5);
    load_link<R, S>(links, V, mu, fwd ? I[p] : J[p], u[p]);
  }
  auto hop = [&](int p, const cx<R>* psi, bool on) {
    cx<R> h[6], uh[6];
    switch (w) {
      case 0: project<0, -1, R>(psi, h); break;
      case 1: project<0, +1, R>(psi, h); break;
      case 2: project<1, -1, R>(psi, h); break;
      case 3: project<1, +1, R>(psi, h); break;
      case 4: project<2, -1, R>(psi, h); break;
      case 5: project<2, +1, R>(psi, h); break;
      case 6: project<3, -1, R>(psi, h); break;
      default: project<3, +1, R>(psi, h); break;
    }
    if (fwd) su3_mul_half<R>(u[p], h, uh);
    else su3_dag_mul_half<R>(u[p], h, uh);
#pragma unroll
    for (int k = 0; k < 6; ++k) part[w][k][lane] = on ? coef[p] * uh[k] : cx<R>{(R)0, (R)0};
  };
  auto hop_x = [&](int p) {   // from x, inside the domain and across its faces
    cx<R> psi[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) psi[c] = act ? ld<R, Tv>(x + c * V + J[p]) : cx<R>{(R)0, (R)0};
    hop(p, psi, true);
  };
  auto hop_vec = [&](int p) {   // inside the domain, from vec (the other parity's sites)
    const int jj = (lane & ~(g.Bvh - 1)) | (int)(J[p] & (g.Bvh - 1));
    cx<R> psi[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) psi[c] = vec[c][jj];
    hop(p, psi, in[p]);
  };

  // rows of waves 0 .. 5: spins 2 half and 2 half + 1 of one colour
  const bool own = w < 6;
  const int half = own ? w / 3 : 0, col = w % 3, R0 = 6 * half + col, R1 = R0 + 3;
  cx<R> mo[2][6];   // of A_oo^-1
  if (own) load_rows<R, S>(cinv, V, I[1], half, col, mo);
  // the eight hops' sum in those rows: (uh, s A_mu^dag uh), s = -1 forward, +1 backward
  auto combine = [&](cx<R>* s) {
    s[0] = s[1] = {(R)0, (R)0};
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      const cx<R> h0 = part[d][col][lane], h1 = part[d][3 + col][lane];
      cx<R> t0 = h0, t1 = h1;
      if (half) {
        if (d >> 1 == 0) t0 = times_i(h1), t1 = times_i(h0);
        if (d >> 1 == 1) t0 = h1, t1 = -h0;
        if (d >> 1 == 2) t0 = times_i(h0), t1 = times_mi(h1);
        if ((d & 1) == 0) t0 = -t0, t1 = -t1;
      }
      s[0] = s[0] + t0;
      s[1] = s[1] + t1;
    }
  };
  auto put = [&](cx<R>(*dst)[64], const cx<R>* v) {
    dst[R0][lane] = v[0];
    dst[R1][lane] = v[1];
  };
  auto rows_of = [&](const cx<R>(*m)[6], const cx<R>(*src)[64], cx<R>* o) {
    cx<R> v[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = src[6 * half + k][lane];
    apply_rows<R>(m, v, o);
  };
  // b - A x in the own rows
  auto source = [&](int p, cx<R>* o) {
    cx<R> v[6], m[2][6];
    load_rows<R, S>(clov, V, I[p], half, col, m);
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = act ? ld<R, Tv>(x + (6 * half + k) * V + I[p]) : cx<R>{(R)0, (R)0};
    apply_rows<R>(m, v, o);
    if (act) {
      o[0] = ld<R, Tv>(b + R0 * V + I[p]) - o[0];
      o[1] = ld<R, Tv>(b + R1 * V + I[p]) - o[1];
    }
  };

  cx<R> rho[2], e[2] = {{(R)0, (R)0}, {(R)0, (R)0}}, ro[2], s[2], t[2];
  // r_o = b - D x
  hop_x(1);
  if (own) source(1, ro);
  __syncthreads();
  if (own) {
    combine(s);
    ro[0] = ro[0] - s[0];
    ro[1] = ro[1] - s[1];
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
    rho[0] = rho[0] - s[0];
    rho[1] = rho[1] - s[1];
  }
  __syncthreads();
  // rho = r_e - H_eo A_oo^-1 r_o
  hop_vec(0);
  __syncthreads();
  if (own) {
    combine(s);
    rho[0] = rho[0] - s[0];
    rho[1] = rho[1] - s[1];
  }
#pragma unroll 1
  for (int k = 0; k < mr_iters; ++k) {
    if (own) put(vec, rho);
    __syncthreads();
    hop_vec(1);
    if (own) {   // A_ee rho; the operand comes from cache while the hops run
      cx<R> me[2][6];
      const S* C = clov;
      asm volatile("" : "+s"(C));   // (read in every step: 48 registers kept across the loop would spill)
      load_rows<R, S>(C, V, I[0], half, col, me);
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
      t[0] = t[0] - s[0];   // p = A_ee rho - H_eo A_oo^-1 H_oe rho
      t[1] = t[1] - s[1];
      mr_sums(t[0], rho[0], re, im, pp);
      mr_sums(t[1], rho[1], re, im, pp);
      for (int off = 1; off < g.Bvh; off <<= 1) {
        re += __shfl_xor(re, off, 64);
        im += __shfl_xor(im, off, 64);
        pp += __shfl_xor(pp, off, 64);
      }
      if (j == 0) {
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
      for (int i = 0; i < 2; ++i) {
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
    t[0] = ro[0] - s[0];
    t[1] = ro[1] - s[1];
    put(row, t);
  }
  __syncthreads();
  if (own) {
    rows_of(mo, row, s);
    if (act) {
      st<Tv, R>(x + R0 * V + I[0], ld<R, Tv>(x + R0 * V + I[0]) + e[0]);
      st<Tv, R>(x + R1 * V + I[0], ld<R, Tv>(x + R1 * V + I[0]) + e[1]);
      st<Tv, R>(x + R0 * V + I[1], ld<R, Tv>(x + R0 * V + I[1]) + s[0]);
      st<Tv, R>(x + R1 * V + I[1], ld<R, Tv>(x + R1 * V + I[1]) + s[1]);
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
  // per launch, as k_sap_colour
  const double half = 0.5 * (double)g.V;
  const double bytes = half * (90.0 * sizeof(S) + 36.0 * sizeof(Tv) * nrhs);
  const double flops = half * nrhs * (mr + 2.5) * 1850.0;
  for (int s = 0; s < sweeps; ++s)
    for (int colour = 0; colour < 2; ++colour)
      DD_TIMED("k_sap_colour", st, bytes, flops,
               (k_sap_split<R, S, Tv><<<nb, 512, 0, st>>>(g, (const S*)ops.links, (const S*)ops.clover,
                                                          (const S*)ops.cinv, nrhs, per, colour, mr, (const Tv*)b, (Tv*)x)));
}

}  // namespace

// By the lattice and not by the launch, as the sums round differently here.  us per
// launch, one thread per site / split: 16^3x32 with domains of 64 sites FP64 one
// right-hand side 251 / 141, FP32 one 108 / 63, twelve 1178 / 738.  Domains of 128 sites
// fill the lanes either way, and the split pays while few of them leave latency bare:
// 64 domains per colour FP64 94 / 47, FP32 twelve 88 / 61; 128 FP64 five right-hand
// sides 105 / 105, FP32 twelve 95 / 90; 512 FP64 five 551 / 614, FP32 twelve 610 / 748.
bool sap_split_use(const GeomDev& g) { return g.Bvh <= 32 || (g.Bvh == 64 && g.Vch <= 128); }

void launch_sap_split(const GeomDev& g, dd_dtype dt, const OpSet& ops, int nrhs, int sweeps, int mr, const void* b,
                      void* x, hipStream_t st) {
  switch (dt) {
    case DD_F64: run_split<double, double2, double2>(g, ops, nrhs, sweeps, mr, b, x, st); break;
    case DD_F32: run_split<float, float2, float2>(g, ops, nrhs, sweeps, mr, b, x, st); break;
    case DD_F16: run_split<float, __half2, float2>(g, ops, nrhs, sweeps, mr, b, x, st); break;
    case DD_BF16: run_split<float, bf16x2, float2>(g, ops, nrhs, sweeps, mr, b, x, st); break;
  }
}
