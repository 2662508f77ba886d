// Galerkin coarse operator D_c = P^dag D P (Eq. 2) for 4^4 aggregates, FP64 on
// matrix cores, straight from the stored test vectors (no fine vectors D lambda
// in memory).
//
// A hop has rank two in spin, so a stored block needs the two-spinor parts only.
// With f_{+,i}(x) = (upper spins of lambda_i) and f_{-,i}(x) = -A_mu (lower spins),
//   D_c(X, +mu)[(s,i), (t,j)] = coef sum_{x on the face} f_{s,i}(x)^dag U_mu(x) f_{t,j}(x+mu),
// a complex product of depth 6 x 64 instead of 12 x 256 fine entries.  The
// backward block is its conjugate transpose up to the chirality signs
// (Gamma5 D_c Gamma5 = D_c^dag, which the same links give term by term),
//   D_c(X+mu, -mu)[(t,j), (s,i)] = +- conj D_c(X, +mu)[(s,i), (t,j)]   (+ when s = t),
// and the self block is G + Gamma5 G^dag Gamma5 with G the forward hops inside the
// aggregate plus half of the clover term.
#include <type_traits>

#include "dslash.h"
#include "ktimer.h"

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kBv = 256, kBvh = 128;

// packed position inside a 4^4 block
__device__ __forceinline__ int local_of(const int l[4]) {
  return ((l[0] + l[1] + l[2] + l[3]) & 1) * kBvh + ((l[0] + 4 * (l[1] + 4 * (l[2] + 4 * l[3]))) >> 1);
}

// conj(A) W summed on matrix cores, three real products per complex one (Gauss, as
// the restriction): with conj(A) = a + ib and W = c + id, k1 += a (c + d), k2 +=
// (a + b)(-d), k3 += (b - a) c.  Element v of lane group lk holds row lk + 4 v.
// (Four products in two accumulators: 2.35 against 1.88 ms for the whole kernel at
// 16^3x32, 2n = 40, and a larger rounding error, its chains being twice as long.)
struct Acc64 {
  f64x4 k1, k2, k3;
  __device__ __forceinline__ void zero() { k1 = k2 = k3 = f64x4{0.0, 0.0, 0.0, 0.0}; }
  __device__ __forceinline__ void add(cx<double> f, cx<double> w) {
    k1 = __builtin_amdgcn_mfma_f64_16x16x4f64(f.re, w.re + w.im, k1, 0, 0, 0);
    k2 = __builtin_amdgcn_mfma_f64_16x16x4f64(f.re - f.im, -w.im, k2, 0, 0, 0);
    k3 = __builtin_amdgcn_mfma_f64_16x16x4f64(-f.im - f.re, w.re, k3, 0, 0, 0);
  }
  __device__ __forceinline__ cx<double> get(int v) const { return {k1[v] + k2[v], k1[v] + k3[v]}; }
};

// two-spinor part of one chirality for a forward hop: upper spins as they are, lower spins as -A_mu d
template <int MU>
__device__ __forceinline__ void half_part(bool lower, cx<double>* f) {
  cx<double> o[6];
  A_mul<MU, double>(f, f + 3, o, o + 3);
#pragma unroll
  for (int k = 0; k < 6; ++k) f[k] = lower ? -o[k] : f[k];
}

// One workgroup per (aggregate, 16 columns of its blocks), one wave per direction.
// Lane (li, lk) of a wave holds, for the site lk of a group of four, the six
// entries of row 16 rt + li (A operand) and of column li (B operand): it loads the
// latter at x + mu, multiplies them by the link itself, and every entry is one k
// step.  A wave first sums its face block (64 sites) and writes it, then the hops
// inside the aggregate (192 sites) and a quarter of the clover term; the four
// waves' parts of G are added in wave order.  Bound by the FP64 matrix products
// (54 of them per four sites, direction and 16 columns at 2n = 40, half of their
// peak rate); the loads are gathers of four sites from 16 vectors.  At 16^3x32, 2n =
// 40, BF16 vectors: 1.88 ms, against 7.9 ms of nine passes over all sites that
// wrote D lambda and restricted it.
template <int N, typename Sp>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_galerkin(
    GeomDev g, const double2* __restrict__ links, const double2* __restrict__ clov, const Sp* __restrict__ P,
    double2* __restrict__ Dc) {
  constexpr int NC = 2 * N, MT = (NC + 15) / 16;
  __shared__ double2 red[3][MT * 16][16];
  const int per_x = g.Vc / 8, k0 = blockIdx.x >> 3;   // Vc is a multiple of 16
  const int X = g.lex_slot[(blockIdx.x & 7) * per_x + k0 / MT], ct = k0 % MT;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  const long long V = g.V, base = (long long)X * kBv;
  const int col = 16 * ct + li, colc = col < NC ? col : NC - 1;
  const bool clow = colc >= N;
  const Sp* Pc = P + (long long)((colc - (clow ? N : 0)) * 12 + (clow ? 6 : 0)) * V;
  bool rlow[MT];
  const Sp* Pr[MT];
#pragma unroll
  for (int rt = 0; rt < MT; ++rt) {
    const int row = 16 * rt + li < NC ? 16 * rt + li : NC - 1;
    rlow[rt] = row >= N;
    Pr[rt] = P + (long long)((row - (rlow[rt] ? N : 0)) * 12 + (rlow[rt] ? 6 : 0)) * V;
  }
  Acc64 acc[MT];

  // groups [g0, g1) of four sites of direction MU, sites ordered with MU slowest; the neighbours of a
  // group lie in the block at nbase
  auto hops = [&](auto mu_c, int g0, int g1, long long nbase) {
    constexpr int MU = decltype(mu_c)::value;
#pragma unroll 1
    for (int gi = g0; gi < g1; ++gi) {
      const int idx = 4 * gi + lk;
      int l[4], e = idx;
#pragma unroll
      for (int d = 0; d < 4; ++d)
        if (d != MU) {
          l[d] = e & 3;
          e >>= 2;
        }
      l[MU] = e;
      const long long x = base + local_of(l);
      l[MU] = (e + 1) & 3;
      const long long y = nbase + local_of(l);
      Sp fr[6], ar[MT][6];
      cx<double> u[9];
#pragma unroll
      for (int k = 0; k < 6; ++k) fr[k] = Pc[k * V + y];
      load_link<double, double2>(links, V, MU, x, u);
#pragma unroll
      for (int rt = 0; rt < MT; ++rt)
#pragma unroll
        for (int k = 0; k < 6; ++k) ar[rt][k] = Pr[rt][k * V + x];
      __builtin_amdgcn_sched_barrier(0);   // every load is issued before the first product
      cx<double> f[6], wv[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) f[k] = ld<double, Sp>(&fr[k]);
      half_part<MU>(clow, f);
      su3_mul_half<double>(u, f, wv);
#pragma unroll
      for (int rt = 0; rt < MT; ++rt) {
#pragma unroll
        for (int k = 0; k < 6; ++k) f[k] = ld<double, Sp>(&ar[rt][k]);
        half_part<MU>(rlow[rt], f);
#pragma unroll
        for (int k = 0; k < 6; ++k) acc[rt].add(f[k], wv[k]);
      }
    }
  };
  auto direction = [&](auto mu_c) {
    constexpr int MU = decltype(mu_c)::value;
#pragma unroll
    for (int rt = 0; rt < MT; ++rt) acc[rt].zero();
    const int e = g.blk_nbr[MU * g.Vc + X];
    hops(mu_c, 48, 64, (long long)(e & DD_SLOT_MASK) * kBv);   // the face sites (coordinate MU = 3)
    const double coef = (e & DD_WRAP_BIT) ? -0.5 * g.bc_t : -0.5;
    double2* out = Dc + ((long long)X * 9 + 1 + MU) * NC * NC;
#pragma unroll
    for (int rt = 0; rt < MT; ++rt) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * rt + lk + 4 * v;
        const cx<double> o = coef * acc[rt].get(v);
        if (row < NC && col < NC) out[col * NC + row] = make_double2(o.re, o.im);
      }
      acc[rt].zero();
    }
    hops(mu_c, 0, 48, base);
  };
  switch (w) {
    case 0: direction(std::integral_constant<int, 0>()); break;
    case 1: direction(std::integral_constant<int, 1>()); break;
    case 2: direction(std::integral_constant<int, 2>()); break;
    default: direction(std::integral_constant<int, 3>()); break;
  }
  // minus the clover term of sites 64 w .. 64 w + 63 (the sum is scaled by -1/2 below, which leaves half of it),
  // one chirality at a time, where both the columns and the rows of the tile have it
#pragma unroll 1
  for (int c = 0; c < 2; ++c) {
    if (c == 0 ? 16 * ct >= N : 16 * ct + 15 < N) continue;   // uniform per workgroup
    const double2* C = clov + (long long)(18 * c) * V;
#pragma unroll 1
    for (int gi = 16 * w; gi < 16 * w + 16; ++gi) {
      const long long x = base + 4 * gi + lk;
      cx<double> f[6], o[6];
      const bool con = clow == (c == 1);
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        f[k] = ld<double, Sp>(Pc + k * V + x);
        if (!con) f[k] = {0.0, 0.0};
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const cx<double> d = ld<double, double2>(C + k * V + x);
        o[2 * k] = -d.re * f[2 * k];
        o[2 * k + 1] = -d.im * f[2 * k + 1];
      }
      int k = 3;
#pragma unroll
      for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int q = r + 1; q < 6; ++q) {
          const cx<double> m = -ld<double, double2>(C + (long long)(k++) * V + x);
          cfma4(o[r], m, f[q]);
          cfma4_conj(o[q], m, f[r]);
        }
#pragma unroll
      for (int rt = 0; rt < MT; ++rt) {
        if (c == 0 ? 16 * rt >= N : 16 * rt + 15 < N) continue;
        const bool ron = rlow[rt] == (c == 1);
#pragma unroll
        for (int r = 0; r < 6; ++r) {
          cx<double> a = ld<double, Sp>(Pr[rt] + r * V + x);
          if (!ron) a = {0.0, 0.0};
          acc[rt].add(a, o[r]);
        }
      }
    }
  }
  if (w > 0)
#pragma unroll
    for (int rt = 0; rt < MT; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const cx<double> o = acc[rt].get(v);
        red[w - 1][16 * rt + lk + 4 * v][li] = make_double2(o.re, o.im);
      }
  __syncthreads();
  if (w == 0) {
    double2* out = Dc + (long long)X * 9 * NC * NC;
#pragma unroll
    for (int rt = 0; rt < MT; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * rt + lk + 4 * v;
        cx<double> o = acc[rt].get(v);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const double2 b = red[p][row][li];
          o = o + cx<double>{b.x, b.y};
        }
        if (row < NC && col < NC) out[col * NC + row] = make_double2(-0.5 * o.re, -0.5 * o.im);
      }
  }
}

// The self block from G, and the backward blocks from the forward ones: one
// workgroup per (aggregate, block 0 .. 4), transposed through LDS.
template <int NC>
__global__ void __launch_bounds__(256) k_galerkin_fold(GeomDev g, double2* __restrict__ Dc) {
  __shared__ double2 M[NC][NC + 1];
  const int X = blockIdx.x / 5, b = blockIdx.x % 5;
  const int Y = b == 0 ? X : g.blk_nbr[(b - 1) * g.Vc + X] & DD_SLOT_MASK;
  const double2* src = Dc + ((long long)X * 9 + b) * NC * NC;
  double2* dst = Dc + ((long long)Y * 9 + (b == 0 ? 0 : b + 4)) * NC * NC;
  for (int e = threadIdx.x; e < NC * NC; e += blockDim.x) M[e / NC][e % NC] = src[e];   // M[col][row]
  __syncthreads();
  for (int e = threadIdx.x; e < NC * NC; e += blockDim.x) {
    const int col = e / NC, row = e % NC;
    const double2 t = M[row][col];
    const bool same = (col >= NC / 2) == (row >= NC / 2);
    double2 o = same ? make_double2(t.x, -t.y) : make_double2(-t.x, t.y);
    if (b == 0) {
      const double2 u = M[col][row];
      o = make_double2(u.x + o.x, u.y + o.y);
    }
    dst[e] = o;
  }
}

template <int N, typename Sp>
void run(const GeomDev& g, const OpSet& ops64, const void* P, double2* Dc, hipStream_t st) {
  constexpr int MT = (2 * N + 15) / 16;
  k_galerkin<N, Sp><<<(unsigned)g.Vc * MT, 256, 0, st>>>(g, (const double2*)ops64.links, (const double2*)ops64.clover,
                                                         (const Sp*)P, Dc);
  k_galerkin_fold<2 * N><<<(unsigned)g.Vc * 5, 256, 0, st>>>(g, Dc);
}

template <typename Sp>
void run_n(const GeomDev& g, const OpSet& ops64, int n, const void* P, double2* Dc, hipStream_t st) {
  switch (n) {
    case 6: run<6, Sp>(g, ops64, P, Dc, st); break;
    case 8: run<8, Sp>(g, ops64, P, Dc, st); break;
    case 12: run<12, Sp>(g, ops64, P, Dc, st); break;
    case 16: run<16, Sp>(g, ops64, P, Dc, st); break;
    case 20: run<20, Sp>(g, ops64, P, Dc, st); break;
    default: run<24, Sp>(g, ops64, P, Dc, st); break;
  }
}

}  // namespace

bool galerkin_direct(const GeomDev& g) {
  return g.b[0] == 4 && g.b[1] == 4 && g.b[2] == 4 && g.b[3] == 4 && g.Vc % 8 == 0;
}

void launch_galerkin(const GeomDev& g, const OpSet& ops64, dd_dtype pst, int n, const void* P, double2* Dc64,
                     hipStream_t st) {
  switch (pst) {
    case DD_F64: run_n<double2>(g, ops64, n, P, Dc64, st); break;
    case DD_F32: run_n<float2>(g, ops64, n, P, Dc64, st); break;
    case DD_F16: run_n<__half2>(g, ops64, n, P, Dc64, st); break;
    case DD_BF16: run_n<bf16x2>(g, ops64, n, P, Dc64, st); break;
  }
}
