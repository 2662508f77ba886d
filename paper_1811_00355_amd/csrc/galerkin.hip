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

// N packed neighbours read at once (the address is a multiple of their size)
template <typename Sp, int N>
struct alignas(N * sizeof(Sp)) Sites {
  Sp v[N];
  __device__ __forceinline__ void load(const Sp* p) { *this = *reinterpret_cast<const Sites*>(p); }
};

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

// two-spinor part of one chirality for a forward hop: upper spins as they are, lower
// spins as -A_mu d.  A_mu only permutes and changes signs: in FP32 for narrow types.
enum Chir { kUpper, kLower, kEither };
template <int MU, Chir C, typename Sp, int NS>
__device__ __forceinline__ void half_part(const Sites<Sp, NS>* s, int q, bool lower, cx<double>* f) {
  using R = std::conditional_t<std::is_same<Sp, double2>::value, double, float>;
  cx<R> d[6], o[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) d[k] = ld<R, Sp>(&s[k].v[q]);
  A_mul<MU, R>(d, d + 3, o, o + 3);
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const cx<R> r = C == kUpper ? d[k] : C == kLower ? -o[k] : lower ? -o[k] : d[k];
    f[k] = {(double)r.re, (double)r.im};
  }
}

// One workgroup per (aggregate, 16 columns of its blocks), one wave per direction.
// Lane (li, lk) of a wave holds, for its site of a group of four, the six entries
// of row 16 rt + li (A operand) and of column li (B operand): it loads the latter at
// x + mu, multiplies them by the link itself, and every entry is one k step.  A
// wave first sums its face block (64 sites) and writes it, then the hops inside
// the aggregate (192 sites) and a quarter of the clover term; the four waves'
// parts of G are added in wave order.  Every 16 sites the accumulators are added to
// the wave's sums in LDS: chains of 96 products instead of up to 1500 (error of D_c
// against 80 bits 4.4e-16 -> 1.4e-16, 2.8e-16 in the sums over D lambda before this
// form; 1-2 % of a new mass).  The operand loads are gathers over 16
// vectors, one cache access a lane whatever its width, and keep the L1 busier than
// the FP64 products do the matrix cores (54 of them per four sites, direction and 16
// columns at 2n = 40; 47 % busy): half types take two packed neighbours to a load,
// the others let the four lanes lk of a vector take neighbours of one line.
// 16^3x32, 2n = 40, BF16 vectors: 1.43-1.49 ms, 1.88 with single sites in lexicographic
// order (nine passes over all sites that wrote D lambda and restricted it: 7.9);
// loads a whole step ahead of the products gave 1.41, but spilled in FP64.  New
// mass on 16^4 before / after: FP64 2270 / 1966 us, FP32 1942 / 1680, BF16 1690 / 1516.
template <int N, typename Sp>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_galerkin(
    GeomDev g, const double2* __restrict__ links, const double2* __restrict__ clov, const Sp* __restrict__ P,
    double2* __restrict__ Dc) {
  constexpr int NC = 2 * N, MT = (NC + 15) / 16;
  __shared__ double2 sum[4][MT * 16][16];   // of each wave, what its accumulators have handed over
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

  // the accumulators to the wave's sums in LDS (first: nothing there yet), and cleared
  auto hand_over = [&](bool first) {
#pragma unroll
    for (int rt = 0; rt < MT; ++rt) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double2* p = &sum[w][16 * rt + lk + 4 * v][li];
        const cx<double> o = acc[rt].get(v);
        if (first) {
          *p = make_double2(o.re, o.im);
        } else {   // the lane's own entry, added in the LDS: nothing to wait for
          __hip_atomic_fetch_add(&p->x, o.re, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_fetch_add(&p->y, o.im, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
      acc[rt].zero();
    }
  };

  // Hops in direction MU from the sites x, x + 1, .. of every lane (NS of them, packed neighbours) to y, y + 1, ..
  auto hops = [&](auto mu_c, auto ns_c, long long x, long long y) {
    constexpr int MU = decltype(mu_c)::value, NS = decltype(ns_c)::value;
    Sites<Sp, NS> fr[6], ar[MT][6];
    cx<double> u[9];
    load_link<double, double2>(links, V, MU, x, u);
    // (addresses opaque: the compiler would keep all of a lane's 6 (MT + 1) row addresses in registers)
    const Sp* p = Pc + y;
    asm volatile("" : "+v"(p));
#pragma unroll
    for (int k = 0; k < 6; ++k) fr[k].load(p + k * V);
    constexpr int AT = sizeof(Sp) == 16 && MT > 2 ? 2 : MT;   // row tiles read with the rest (registers)
    auto rows = [&](int rt) {
      p = Pr[rt] + x;
      asm volatile("" : "+v"(p));
#pragma unroll
      for (int k = 0; k < 6; ++k) ar[rt][k].load(p + k * V);
    };
#pragma unroll
    for (int rt = 0; rt < AT; ++rt) rows(rt);
    __builtin_amdgcn_sched_barrier(0);   // every load is issued before the first product
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      cx<double> f[6], wv[6];
      if (q) {
        __builtin_amdgcn_sched_barrier(0);
        load_link<double, double2>(links, V, MU, x + q, u);
      }
      half_part<MU, kEither>(fr, q, clow, f);
      su3_mul_half<double>(u, f, wv);
      if (AT < MT && q == 0) {
        __builtin_amdgcn_sched_barrier(0);
        rows(MT - 1);
      }
#pragma unroll
      for (int rt = 0; rt < MT; ++rt) {
        if (16 * rt + 15 < N) half_part<MU, kUpper>(ar[rt], q, false, f);
        else if (16 * rt >= N) half_part<MU, kLower>(ar[rt], q, true, f);
        else half_part<MU, kEither>(ar[rt], q, rlow[rt], f);
#pragma unroll
        for (int k = 0; k < 6; ++k) acc[rt].add(f[k], wv[k]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // the pair of packed sites with the same (y, z, t) and parity: x = x0, x0 + 2, x0 = (parity + y + z + t) % 2
  auto pair_at = [&](int par, int cy, int cz, int ct4) { return par * kBvh + 2 * (cy + 4 * (cz + 4 * ct4)); };
  auto direction = [&](auto mu_c) {
    constexpr int MU = decltype(mu_c)::value;
    constexpr int NS = sizeof(Sp) <= 4 ? 2 : 1;   // sites of a lane's load
    const int e = g.blk_nbr[MU * g.Vc + X];
    const long long nb = (long long)(e & DD_SLOT_MASK) * kBv;
    const double coef = (e & DD_WRAP_BIT) ? -0.5 * g.bc_t : -0.5;
#pragma unroll
    for (int rt = 0; rt < MT; ++rt) acc[rt].zero();
    // first the hops across the face, summed by themselves, then those inside the aggregate
#pragma unroll 1
    for (int inside = 0; inside < 2; ++inside) {
      if constexpr (MU == 0) {
        // the pairs x = 1, 3: the second site hops across the face, the first one to the other pair's second site
#pragma unroll 1
        for (int i = 0; i < 16; ++i) {
          const int cz = i & 3, t = i >> 2, par = (lk + cz + t + 1) & 1;
          const int q = pair_at(par, lk, cz, t), r = pair_at(par ^ 1, lk, cz, t);
          hops(mu_c, std::integral_constant<int, 1>(), base + q + (inside ? 0 : 1), inside ? base + r + 1 : nb + r);
          if ((i + 1) % 4 == 0) hand_over(i < 4);
        }
        if (inside) {   // the pairs x = 0, 2 to the pairs 1, 3
#pragma unroll 1
          for (int i = 0; i < 32 / NS; ++i) {
            const int h = NS == 1 ? lk & 1 : 0, cy = NS == 1 ? 2 * (i & 1) + (lk >> 1) : lk, j = NS == 1 ? i >> 1 : i;
            const int cz = j & 3, t = j >> 2, par = (cy + cz + t) & 1;
            hops(mu_c, std::integral_constant<int, NS>(), base + pair_at(par, cy, cz, t) + h,
                 base + pair_at(par ^ 1, cy, cz, t) + h);
            if ((i + 1) % (4 / NS) == 0) hand_over(false);
          }
        }
      } else {
        // coordinate MU slowest: 0 .. 2 stay inside
#pragma unroll 1
        for (int i = inside ? 0 : 48 / NS; i < (inside ? 48 / NS : 64 / NS); ++i) {
          const int h = NS == 1 ? lk & 1 : 0, a = NS == 1 ? 2 * (i & 1) + (lk >> 1) : lk, j = NS == 1 ? i >> 1 : i;
          const int c = j >> 3, o = j & 3, par = (j >> 2) & 1, d = (c + 1) & 3;
          const int q = MU == 1 ? pair_at(par, c, a, o) : MU == 2 ? pair_at(par, a, c, o) : pair_at(par, a, o, c);
          const int r = MU == 1 ? pair_at(par ^ 1, d, a, o) : MU == 2 ? pair_at(par ^ 1, a, d, o) : pair_at(par ^ 1, a, o, d);
          hops(mu_c, std::integral_constant<int, NS>(), base + q + h, (inside ? base : nb) + r + h);
          if ((i + 1) % (4 / NS) == 0) hand_over(i < (inside ? 0 : 48 / NS) + 4 / NS);
        }
      }
      if (inside) break;
      double2* out = Dc + ((long long)X * 9 + 1 + MU) * NC * NC;
#pragma unroll
      for (int rt = 0; rt < MT; ++rt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 16 * rt + lk + 4 * v;
          const double2 t = sum[w][row][li];
          const cx<double> o = coef * cx<double>{t.x, t.y};
          if (row < NC && col < NC) out[col * NC + row] = make_double2(o.re, o.im);
        }
      }
    }
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
      if ((gi + 1) % 4 == 0) hand_over(false);
    }
  }
  __syncthreads();
  if (w == 0) {
    double2* out = Dc + (long long)X * 9 * NC * NC;
#pragma unroll
    for (int rt = 0; rt < MT; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * rt + lk + 4 * v;
        cx<double> o = {0.0, 0.0};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const double2 b = sum[p][row][li];
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

void launch_galerkin(const GeomDev& g, const OpSet& ops64, dd_dtype pst, int n, const void* P, double2* Dc64,
                     hipStream_t st) {
  switch (pst) {
    case DD_F64: run_n<double2>(g, ops64, n, P, Dc64, st); break;
    case DD_F32: run_n<float2>(g, ops64, n, P, Dc64, st); break;
    case DD_F16: run_n<__half2>(g, ops64, n, P, Dc64, st); break;
    case DD_BF16: run_n<bf16x2>(g, ops64, n, P, Dc64, st); break;
  }
}
