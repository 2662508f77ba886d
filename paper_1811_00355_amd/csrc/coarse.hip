// Coarse-grid operator apply (Eq. 2 stencil, Sec. 3: "effective links" and
// "clover" blocks of size 2n x 2n).  Blocks are column major, so the lanes of
// a wave read consecutive rows of one column.
//
//   out(X) = a_self * M(X) xs(X) + a_hop * sum_{d=1..8} D_c(X, d) xh(X + d) + beta * z(X)
//
// with M(X) = D_c(X, 0) (self block) or, for odd sites, the stored inverse of
// the self block.  This covers the full stencil (xs = xh = x), the two halves
// of the even-site Schur complement and the odd-site reconstruction.
#include <type_traits>

#include "dd_internal.h"
#include "ktimer.h"

namespace {

// Matrix-core form.  For one coarse site and one direction the stencil term is a
// complex product Y (2n x rhs) += B (2n x 2n) X (2n x rhs) with the right-hand
// side as the column index, computed by real 16x16x4 MFMAs over (16-row tile,
// 4-deep k step).  Lane layout: A[i][k] at lane i + 16k, B[k][j] at lane j + 16k;
// up to 16 right-hand sides per pass, 2n <= 48.
// Matrix-core order of one NC x NC block (the FP32 and half copies the FP32
// apply reads).  Element (row, col) lies in row tile t = row / 16 (RT = min(16,
// NC - 16 t) rows), lane group lk = col / KS and k-step ks = col % KS, with KS =
// NC / 4 k-steps (so a lane's columns are consecutive, and it reads its part of
// an input vector with wide loads); P consecutive k-steps form a group q = ks / P.  Within a tile the order is
// [q][lk][li][e]: lane (li, lk) of the MFMA operand reads its P k-steps of row
// 16 t + li with one load of P elements, and a wave reads one contiguous stretch.
// No padding: a block still holds NC * NC elements.
__host__ __device__ inline long long tiled_off(int row, int col, int NC, int P) {
  const int t = row >> 4, li = row & 15, RT = NC - 16 * t < 16 ? NC - 16 * t : 16;
  const int KS = NC >> 2, ks = col % KS, lk = col / KS, q = ks / P, e = ks % P;
  return (long long)16 * t * NC + ((long long)(q * 4 + lk) * RT + li) * P + e;
}
// P: the largest power of two k-steps per load (at most 16 bytes) that divides NC / 4
__host__ __device__ constexpr int tile_group(int NC, int elem_bytes) {
  return ((NC / 4) % (16 / elem_bytes) == 0) ? 16 / elem_bytes : (((NC / 4) % 2 == 0 && 16 / elem_bytes >= 2) ? 2 : 1);
}

// FP64 column-major blocks -> FP32 blocks in matrix-core order
__global__ void k_tile_f32(const double2* __restrict__ src, float2* __restrict__ dst, long long nblk, int NC) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long per = (long long)NC * NC;
  if (i >= nblk * per) return;
  const long long b = i / per, w = i % per;
  const int row = (int)(w % NC), col = (int)(w / NC);
  const double2 v = src[i];
  dst[b * per + tiled_off(row, col, NC, tile_group(NC, 8))] = make_float2((float)v.x, (float)v.y);
}
// FP32 matrix-core blocks -> half matrix-core blocks (rounded from the FP32 values)
template <typename H>
__global__ void k_tile_half(const float2* __restrict__ src, H* __restrict__ dst, long long nblk, int NC) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long per = (long long)NC * NC;
  if (i >= nblk * per) return;
  const long long b = i / per, w = i % per;
  const int row = (int)(w % NC), col = (int)(w / NC);
  const float2 v = src[b * per + tiled_off(row, col, NC, tile_group(NC, 8))];
  H* d = dst + b * per + tiled_off(row, col, NC, tile_group(NC, 4));
  if constexpr (sizeof(H) == 4 && std::is_same<H, __half2>::value) {
    *d = __floats2half2_rn(v.x, v.y);
  } else {
    d->u = f32_to_bf16_bits(v.x) | (f32_to_bf16_bits(v.y) << 16);
  }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kMfmaMaxNc = 48;

// One accumulator set of a complex product on matrix cores, in FP32 (three real
// products, Gauss: with A = a + ib and x = c + id, k1 += a (c + d), k2 +=
// (a + b)(-d), k3 += (b - a) c, Re = k1 + k2, Im = k1 + k3) or FP64 (four real
// products, chained: the matrix cores are not what bounds it, and three would
// add roundings of sums of entries; kFine below is about the length of the
// chains).  row(lk, v): the row that element v of lane group lk holds.
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <typename R> struct Cacc;
template <> struct Cacc<float> {
  typedef float2 vec;
  f32x4 k1 = {0.f, 0.f, 0.f, 0.f}, k2 = {0.f, 0.f, 0.f, 0.f}, k3 = {0.f, 0.f, 0.f, 0.f};
  __device__ __forceinline__ void add(cx<float> m, float2 x) {
    k1 = __builtin_amdgcn_mfma_f32_16x16x4f32(m.re, x.x + x.y, k1, 0, 0, 0);
    k2 = __builtin_amdgcn_mfma_f32_16x16x4f32(m.re + m.im, -x.y, k2, 0, 0, 0);
    k3 = __builtin_amdgcn_mfma_f32_16x16x4f32(m.im - m.re, x.x, k3, 0, 0, 0);
  }
  __device__ __forceinline__ cx<float> get(int v) const { return {k1[v] + k2[v], k1[v] + k3[v]}; }
  __device__ static int row(int lk, int v) { return 4 * lk + v; }
};
template <> struct Cacc<double> {
  typedef double2 vec;
  f64x4 kr = {0.0, 0.0, 0.0, 0.0}, ki = {0.0, 0.0, 0.0, 0.0};
  __device__ __forceinline__ void add(cx<double> m, double2 x) {
    kr = __builtin_amdgcn_mfma_f64_16x16x4f64(m.re, x.x, kr, 0, 0, 0);
    ki = __builtin_amdgcn_mfma_f64_16x16x4f64(m.re, x.y, ki, 0, 0, 0);
    kr = __builtin_amdgcn_mfma_f64_16x16x4f64(-m.im, x.y, kr, 0, 0, 0);
    ki = __builtin_amdgcn_mfma_f64_16x16x4f64(m.im, x.x, ki, 0, 0, 0);
  }
  __device__ __forceinline__ cx<double> get(int v) const { return {kr[v], ki[v]}; }
  __device__ static int row(int lk, int v) { return lk + 4 * v; }
};

// NC = 2n (a multiple of 4, at most 48).  A workgroup takes one coarse site with
// DS groups of MT / TW waves, MT = ceil(NC / 16) row tiles: the groups share out
// the stencil's directions (group q takes directions d_begin + q, + DS, ...), a
// wave takes TW row tiles.  It loads its rows of a direction's block and the
// neighbour's x for 16 right-hand sides straight into matrix-core operand
// registers (no LDS and no barrier per direction; every load of a direction is
// issued before its first product, which the compiler would otherwise interleave
// at half the loads in flight); the groups' sums are added in group order at the
// end through LDS.  Columns past nrhs and rows past the tile repeat valid ones
// and are not stored.  NT: the blocks are read past the caches.
// INV: the result is multiplied by Minv(X) before it is stored (odd-site inverse,
// loaded before the first direction):
//   out = Minv (a_self M xs + a_hop sum D_c xh + beta z)
// which is the odd half of the Schur complement in one launch.
// Sites go to the XCDs in contiguous eighths, so the neighbours' x of one range
// come from the same L2.  Bound by the blocks' bytes on large lattices (12
// right-hand sides, 2n = 40, 24^3x48: 78 -> 71 us, 4.5 TB/s; 32^3x48 4.6 TB/s; one
// right-hand side 5.1-5.7 TB/s against 4.9 TB/s of a large copy) and by the latency
// of a launch on small ones (16^3x32, even sites only: 13.7 us before); the form
// before took one direction at a time through LDS with a barrier for each.
template <int NC, typename Sd, typename R, bool INV, int DS, int TW, bool NT>
__global__ void __launch_bounds__(64 * DS * ((NC + 15) / 16) / TW) k_coarse_mfma(
    GeomDev g, const Sd* __restrict__ Dc, const Sd* __restrict__ Minv, int use_inv, int nrhs, int site_begin,
    int count, R a_self, const typename Cacc<R>::vec* __restrict__ xs, R a_hop,
    const typename Cacc<R>::vec* __restrict__ xh, R beta, const typename Cacc<R>::vec* __restrict__ z,
    typename Cacc<R>::vec* __restrict__ out, Gate gt) {
  if (gate_closed(gt)) return;
  typedef Cacc<R> Acc;
  typedef typename Acc::vec Tv;
  constexpr int MT = (NC + 15) / 16, KS = NC / 4, WG = MT / TW;   // WG: waves per group
  constexpr bool kTiled = sizeof(R) == 4;   // FP64 blocks are column major
  // FP64: two chains for a block's columns, added before they meet the other directions, and the self term last.  Against
  // 80 bits, 2n = 16 / 40: 1.60 / 2.27e-16, a plain sum by columns 1.53 / 2.18, one chain with the self term first 2.12 /
  // 3.06 (thirds: 1.58 / 1.99, but 3-10 % of the time; halves 0-4 %)
  constexpr bool kFine = sizeof(R) == 8;
  constexpr int P = kTiled ? tile_group(NC, (int)sizeof(Sd)) : 1;
  struct alignas(P * sizeof(Sd)) Pack {
    Sd v[P];
  };
  struct Rows {
    Pack a[KS / P];
  };
  __shared__ Tv red[DS > 1 ? DS - 1 : 1][MT * 16][16];
  __shared__ Tv rsh[INV ? NC : 1][INV ? 17 : 1];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int q = wv / WG, t0 = (wv % WG) * TW;
  const int per_x = (count + 7) / 8;
  const int local = (blockIdx.x & 7) * per_x + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_x || local >= count) return;   // uniform per workgroup
  const int X = site_begin + local;
  const long long vstride = (long long)g.Vc * NC;
  const int d_begin = a_self != (R)0 ? 0 : 1, d_end = a_hop != (R)0 ? 9 : 1;
  const int nd = d_end - d_begin;
  const int li = lane & 15, lk = lane >> 4;
  // rows 16 t + li, columns lk KS + ks of a block
  auto load_rows = [&](const Sd* B, int t, Rows& r) {
    const int RT = NC - 16 * t < 16 ? NC - 16 * t : 16, row_c = li < RT ? li : RT - 1;
#pragma unroll
    for (int i = 0; i < KS / P; ++i) {
      if constexpr (kTiled && NT && sizeof(Pack) == 16) {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        r.a[i] = __builtin_bit_cast(
            Pack, __builtin_nontemporal_load(reinterpret_cast<const u4*>(B + 16 * t * NC + ((i * 4 + lk) * RT + row_c) * P)));
      } else if constexpr (kTiled) {
        r.a[i] = *reinterpret_cast<const Pack*>(B + 16 * t * NC + ((i * 4 + lk) * RT + row_c) * P);
      } else {
        r.a[i].v[0] = B[(lk * KS + i) * NC + 16 * t + row_c];
      }
    }
  };
  const Sd* Mx = INV || use_inv ? Minv + (long long)(X - g.Vch) * NC * NC : nullptr;
  // the inverse's row tiles are dealt to the waves in turn
  constexpr int kWaves = DS * WG, kInvT = INV ? (MT + kWaves - 1) / kWaves : 1;
  Rows minv[kInvT];
  if constexpr (INV) {
#pragma unroll
    for (int i = 0; i < kInvT; ++i)
      if (wv + i * kWaves < MT) load_rows(Mx, wv + i * kWaves, minv[i]);
  }
  for (int r0 = 0; r0 < nrhs; r0 += 16) {
    const int nr = nrhs - r0 < 16 ? nrhs - r0 : 16;
    const long long roff = (long long)(r0 + (li < nr ? li : nr - 1)) * vstride + lk * KS;
    cx<R> tot[TW][4];
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) tot[i][v] = {(R)0, (R)0};
#pragma unroll 1
    for (int p = q; p < nd; p += DS) {
      const int d = !kFine ? d_begin + p : p + 1 == nd && d_begin == 0 ? 0 : p + 1;
      const int Y = d == 0 ? X : __builtin_amdgcn_readfirstlane(g.blk_nbr[(d - 1) * g.Vc + X] & DD_SLOT_MASK);
      const Tv* xp = (d == 0 ? xs : xh) + roff + (long long)Y * NC;
      const Sd* B = d == 0 && use_inv ? Mx : Dc + ((long long)X * 9 + d) * NC * NC;
      const R sc = d == 0 ? a_self : a_hop;
      Tv x[KS];
      Rows rows[TW];
#pragma unroll
      for (int k = 0; k < KS; ++k) x[k] = xp[k];
#pragma unroll
      for (int i = 0; i < TW; ++i) load_rows(B, t0 + i, rows[i]);
      __builtin_amdgcn_sched_barrier(0);   // every load is issued before the first product
#pragma unroll
      for (int i = 0; i < TW; ++i) {
        Acc acc;
        cx<R> part[4];
#pragma unroll
        for (int k = 0; k < KS; ++k) {
          acc.add(ld<R, Sd>(&rows[i].a[k / P].v[k % P]), x[k]);
          if (kFine && k == KS / 2 - 1) {
#pragma unroll
            for (int v = 0; v < 4; ++v) part[v] = acc.get(v);
            acc = Acc();
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) tot[i][v] = tot[i][v] + sc * (kFine ? part[v] + acc.get(v) : acc.get(v));
      }
    }
    if constexpr (DS > 1) {
      if (q > 0)
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            red[q - 1][16 * (t0 + i) + Acc::row(lk, v)][li] = Tv{tot[i][v].re, tot[i][v].im};
      __syncthreads();
    }
    if (q == 0) {
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 16 * (t0 + i) + Acc::row(lk, v);
          cx<R> o = tot[i][v];
          if constexpr (kFine && DS > 1) {   // the group of the self term last
            const Tv first = red[0][row][li];
            cx<R> h = {first.x, first.y};
#pragma unroll
            for (int p = 1; p < DS - 1; ++p) {
              const Tv b = red[p][row][li];
              h = h + cx<R>{b.x, b.y};
            }
            o = o + h;
          } else if constexpr (DS > 1) {
#pragma unroll
            for (int p = 0; p < DS - 1; ++p) {
              const Tv b = red[p][row][li];
              o = o + cx<R>{b.x, b.y};
            }
          }
          if (row < NC) {
            const long long oi = (long long)(r0 + li) * vstride + (long long)X * NC + row;
            if (li < nr && beta != (R)0) {
              const Tv zz = z[oi];
              o = o + beta * cx<R>{zz.x, zz.y};
            }
            if constexpr (INV) rsh[row][li] = Tv{o.re, o.im};
            else if (li < nr) out[oi] = Tv{o.re, o.im};
          }
        }
    }
    if constexpr (INV) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kInvT; ++i) {
        const int t = wv + i * kWaves;
        if (t >= MT) break;
        Acc acc;
#pragma unroll
        for (int k = 0; k < KS; ++k) acc.add(ld<R, Sd>(&minv[i].a[k / P].v[k % P]), rsh[lk * KS + k][li]);
        if (li < nr)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = 16 * t + Acc::row(lk, v);
            const cx<R> o = acc.get(v);
            if (row < NC) out[(long long)(r0 + li) * vstride + (long long)X * NC + row] = Tv{o.re, o.im};
          }
      }
    }
    if constexpr (DS > 1 || INV) __syncthreads();   // red and rsh are refilled by the next 16 right-hand sides
  }
}

// Half-precision matrix-core form (opt-in, half-precision blocks only): the
// blocks feed 16x16x16 FP16 / BF16 MFMAs directly and sc * x(Y) is rounded to
// the same type when staged; products accumulate in FP32 (four real MFMAs per
// complex product: k1 = a c, k2 = b d, k3 = a d, k4 = b c).  MFMA K-slot
// (lk, v) of K-step s takes column lk KS + 4 s + v, so every lane's four A
// values sit at one (row, lk) of the tiled block layout (see tiled_off);
// columns past NC are zero on both sides.
typedef _Float16 h16x4 __attribute__((ext_vector_type(4)));
typedef short b16x4 __attribute__((ext_vector_type(4)));

template <typename Sd> struct HalfOp;
template <> struct HalfOp<__half2> {
  typedef h16x4 vec;
  typedef _Float16 elem;
  __device__ static elem from_f32(float f) { return (_Float16)f; }
  __device__ static void split(const __half2& v, elem& re, elem& im) {
    const __half2_raw r = v;
    re = __builtin_bit_cast(_Float16, r.x);
    im = __builtin_bit_cast(_Float16, r.y);
  }
  __device__ static f32x4 mfma(vec a, vec b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0); }
};
template <> struct HalfOp<bf16x2> {
  typedef b16x4 vec;
  typedef short elem;
  __device__ static elem from_f32(float f) { return (short)f32_to_bf16_bits(f); }
  __device__ static void split(const bf16x2& v, elem& re, elem& im) {
    re = (short)(v.u & 0xffffu);
    im = (short)(v.u >> 16);
  }
  __device__ static f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
  }
};

// Two directions per barrier phase: the loads of both directions' blocks and
// inputs are in flight together (five phases for the nine-block stencil
// instead of nine), which matters because one apply is a single round of
// workgroups whose time is the chain of load latencies.  The directions are
// still accumulated in order, so the result is that of one direction per phase.
// With both directions' operands live the compiler would take about 164
// registers (two waves per SIMD); the register budget is capped at four waves
// per SIMD instead (the BF16 form then spills 12 bytes per lane).
template <int NC, int S, typename Sd>
__global__ void __launch_bounds__(64 * S * ((NC + 15) / 16)) __attribute__((amdgpu_waves_per_eu(4))) k_coarse_mfma_h(
    GeomDev g, const Sd* __restrict__ Dc, const Sd* __restrict__ Minv, int use_inv, int nrhs, int site_begin,
    int count, float a_self, const float2* __restrict__ xs, float a_hop, const float2* __restrict__ xh, float beta,
    const float2* __restrict__ z, float2* __restrict__ out, Gate gt) {
  if (gate_closed(gt)) return;
  typedef HalfOp<Sd> H;
  typedef typename H::vec vec;
  typedef typename H::elem elem;
  constexpr int MT = (NC + 15) / 16, KS = NC / 4, NS = (KS + 3) / 4, DP = 2;
  constexpr int P = tile_group(NC, (int)sizeof(Sd));
  constexpr int XI = (16 * NC + 64 * MT - 1) / (64 * MT);
  // staged x: [site][buffer][direction of the phase][s][lk][rhs][v], real and imaginary parts
  __shared__ alignas(16) elem xc[S][2][DP][NS][4][16][4];
  __shared__ alignas(16) elem xd[S][2][DP][NS][4][16][4];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int s_in = wv / MT, t = wv % MT, tid_site = threadIdx.x - 64 * MT * s_in;
  const int ngroups = (count + S - 1) / S, per_x = (ngroups + 7) / 8;
  const int group = (blockIdx.x & 7) * per_x + (blockIdx.x >> 3);
  if (group >= ngroups) return;   // uniform per workgroup
  const int local = group * S + s_in;
  const bool site_ok = local < count;
  // the site is the same on every lane of a wave: keep it (and the block and
  // neighbour addresses derived from it) in scalar registers
  const int X = __builtin_amdgcn_readfirstlane(site_begin + (site_ok ? local : 0));
  const int RT = NC - 16 * t < 16 ? NC - 16 * t : 16;
  const long long vstride = (long long)g.Vc * NC;
  const bool has_self = a_self != 0.f, has_hop = a_hop != 0.f;
  const int d_begin = has_self ? 0 : 1, d_end = has_hop ? 9 : 1;
  const int li = lane & 15, lk = lane >> 4;
  const bool row_ok = li < RT;
  // K-slots past NC stay zero in every buffer
  {
    elem* pc = &xc[s_in][0][0][0][0][0][0];
    elem* pd = &xd[s_in][0][0][0][0][0][0];
    for (int e = tid_site; e < 2 * DP * NS * 4 * 16 * 4; e += 64 * MT) {
      pc[e] = H::from_f32(0.f);
      pd[e] = H::from_f32(0.f);
    }
  }
  __syncthreads();
  int buf = 0;
  for (int r0 = 0; r0 < nrhs; r0 += 16) {
    const int nr = nrhs - r0 < 16 ? nrhs - r0 : 16;
    const bool rhs_ok = li < nr;
    const int nx = nr * NC;
    f32x4 k1 = {0.f, 0.f, 0.f, 0.f}, k2 = k1, k3 = k1, k4 = k1;
    for (int d0 = d_begin; d0 < d_end; d0 += DP) {
      const int nd = d_end - d0 < DP ? d_end - d0 : DP;   // uniform
      float2 xv[DP][XI];
      Sd av[DP][NS][4];
#pragma unroll
      for (int q = 0; q < DP; ++q) {
        if (q >= nd) break;
        const int d = d0 + q;
        const int Y = d == 0 ? X : __builtin_amdgcn_readfirstlane(g.blk_nbr[(d - 1) * g.Vc + X] & DD_SLOT_MASK);
        const float2* xsrc = (d == 0 ? xs : xh) + (long long)r0 * vstride + (long long)Y * NC;
        const Sd* B = d == 0 ? (use_inv ? Minv + (long long)(X - g.Vch) * NC * NC : Dc + (long long)X * 9 * NC * NC)
                             : Dc + ((long long)X * 9 + d) * NC * NC;
        const Sd* Bt = B + 16 * t * NC;
#pragma unroll
        for (int i = 0; i < XI; ++i) {
          const int e = tid_site + 64 * MT * i, ec = e < nx ? e : nx - 1;
          const int r = ec / NC, col = ec - r * NC;
          xv[q][i] = xsrc[(unsigned)(r * (int)vstride + col)];   // < 16 * Vc * NC elements
        }
        // this wave's rows: K-step s, slot v -> tiled column group ks = 4 s + v at this lane's lk
#pragma unroll
        for (int st = 0; st < NS; ++st)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int ks = 4 * st + v;
            if (ks < KS) av[q][st][v] = Bt[(unsigned)((((ks / P) * 4 + lk) * RT + (row_ok ? li : 0)) * P + ks % P)];
          }
      }
#pragma unroll
      for (int q = 0; q < DP; ++q) {
        if (q >= nd) break;
        const float sc = d0 + q == 0 ? a_self : a_hop;
#pragma unroll
        for (int i = 0; i < XI; ++i) {
          const int e = tid_site + 64 * MT * i;
          if (e < nx) {
            const int r = e / NC, col = e - r * NC;
            const int ks = col % KS, cl = col / KS;
            xc[s_in][buf][q][ks >> 2][cl][r][ks & 3] = H::from_f32(sc * xv[q][i].x);
            xd[s_in][buf][q][ks >> 2][cl][r][ks & 3] = H::from_f32(sc * xv[q][i].y);
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < DP; ++q) {
        if (q >= nd) break;
#pragma unroll
        for (int st = 0; st < NS; ++st) {
          vec a, b;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            elem re = H::from_f32(0.f), im = H::from_f32(0.f);
            if (4 * st + v < KS && row_ok) H::split(av[q][st][v], re, im);
            a[v] = re;
            b[v] = im;
          }
          vec c = *reinterpret_cast<const vec*>(&xc[s_in][buf][q][st][lk][li][0]);
          vec dd = *reinterpret_cast<const vec*>(&xd[s_in][buf][q][st][lk][li][0]);
          if (!rhs_ok) {
            c = vec{};
            dd = vec{};
          }
          k1 = H::mfma(a, c, k1);
          k2 = H::mfma(b, dd, k2);
          k3 = H::mfma(a, dd, k3);
          k4 = H::mfma(b, c, k4);
        }
      }
      buf ^= 1;
    }
    if (site_ok && rhs_ok) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * t + 4 * lk + v;
        if (row < NC) {
          long long oi = (long long)(r0 + li) * vstride + (long long)X * NC + row;
          float2 o = make_float2(k1[v] - k2[v], k3[v] + k4[v]);
          if (beta != 0.f) {
            float2 zz = z[oi];
            o.x += beta * zz.x;
            o.y += beta * zz.y;
          }
          out[oi] = o;
        }
      }
    }
  }
}

template <typename R>
using MfmaFn = void (*)(GeomDev, const void*, const void*, int, int, int, int, R, const typename Cacc<R>::vec*, R,
                        const typename Cacc<R>::vec*, R, const typename Cacc<R>::vec*, typename Cacc<R>::vec*, Gate);

template <typename R>
struct MfmaLaunch {
  MfmaFn<R> fn;
  dim3 grid, blk;
};

// half blocks on half matrix cores; spw: target waves per workgroup, sites per workgroup S = max(1, spw / MT), at most 4
template <int NC, typename Sd>
MfmaLaunch<float> half_launch(int spw, int count) {
  constexpr int MT = (NC + 15) / 16;
  int S = spw / MT;
  S = S >= 4 ? 4 : S >= 2 ? 2 : 1;
  MfmaFn<float> fn = S == 4 ? (MfmaFn<float>)k_coarse_mfma_h<NC, 4, Sd> : S == 2 ? (MfmaFn<float>)k_coarse_mfma_h<NC, 2, Sd>
                                                                                 : (MfmaFn<float>)k_coarse_mfma_h<NC, 1, Sd>;
  const unsigned per_x = ((count + S - 1) / S + 7) / 8;
  return {fn, dim3(8 * per_x), dim3(64 * S * MT)};
}

// Two splits of the full-precision form, by whether the lattice's stencil blocks
// fit the 256 MB last-level cache:
//  - they fit: the apply is short and its time a chain of latencies, so a site's
//    work is spread over four direction groups with one row tile per wave
//    (at 2n = 40 12 waves per site), and the blocks are kept cached for the next apply;
//  - they do not: HBM bounds it, so two direction groups whose waves take all
//    row tiles of a site (its x is loaded once per direction instead of once per
//    tile) and stream the blocks past the caches, unless another 16 right-hand
//    sides read them again (us, twenty right-hand sides, streamed / cached: 2n = 40,
//    24^3x48 137 / 119, 32^3x64 398 / 339; 2n = 48, 24^3x48 180 / 166; twelve, 32^3x64 206 either way).
// Measured full applies, us, first / second split, 12 right-hand sides, FP32
// blocks: 2n = 40 on 88 MB (16x16x24x32) 20 / 25, 199 MB (24^3x32) 40 / 49,
// 299 MB (24^3x48) 76 / 71, 708 MB (32^3x48) 179 / 156; 2n = 48 on 430 MB 111 / 94.
constexpr double kCachedStencilBytes = 256e6;

template <int NC, typename Sd, typename R>
MfmaLaunch<R> full_launch(int Vc, int count, bool inv, int nrhs) {
  constexpr int MT = (NC + 15) / 16;
  const bool cached = 9.0 * Vc * NC * NC * sizeof(Sd) <= kCachedStencilBytes;
  MfmaFn<R> fn;
  if (cached)
    fn = inv ? (MfmaFn<R>)k_coarse_mfma<NC, Sd, R, true, 4, 1, false> : (MfmaFn<R>)k_coarse_mfma<NC, Sd, R, false, 4, 1, false>;
  else if (nrhs > 16)
    fn = inv ? (MfmaFn<R>)k_coarse_mfma<NC, Sd, R, true, 2, MT, false> : (MfmaFn<R>)k_coarse_mfma<NC, Sd, R, false, 2, MT, false>;
  else
    fn = inv ? (MfmaFn<R>)k_coarse_mfma<NC, Sd, R, true, 2, MT, true> : (MfmaFn<R>)k_coarse_mfma<NC, Sd, R, false, 2, MT, true>;
  const unsigned per_x = (count + 7) / 8;
  return {fn, dim3(8 * per_x), dim3(cached ? 64 * 4 * MT : 64 * 2)};
}

#define DD_NC_SWITCH(nc, CALL)  \
  switch (nc) {                 \
    case 12: return CALL(12);   \
    case 16: return CALL(16);   \
    case 24: return CALL(24);   \
    case 32: return CALL(32);   \
    case 40: return CALL(40);   \
    default: return CALL(48);   \
  }
template <typename Sd, typename R>
MfmaLaunch<R> full_pick(int nc, int Vc, int count, bool inv, int nrhs) {
#define DD_FULL(N) (full_launch<N, Sd, R>(Vc, count, inv, nrhs))
  DD_NC_SWITCH(nc, DD_FULL)
#undef DD_FULL
}
template <typename Sd>
MfmaLaunch<float> half_pick(int nc, int count, int spw) {
#define DD_HALF(N) (half_launch<N, Sd>(spw, count))
  DD_NC_SWITCH(nc, DD_HALF)
#undef DD_HALF
}
#undef DD_NC_SWITCH

}  // namespace

void launch_coarse_tile(int nc, const double2* src64, long long nblk, float2* dst32, dd_dtype half, void* dsth,
                        hipStream_t st) {
  const long long n = nblk * nc * nc;
  const unsigned nb = (unsigned)((n + 255) / 256);
  k_tile_f32<<<nb, 256, 0, st>>>(src64, dst32, nblk, nc);
  if (half == DD_F16) k_tile_half<__half2><<<nb, 256, 0, st>>>(dst32, (__half2*)dsth, nblk, nc);
  if (half == DD_BF16) k_tile_half<bf16x2><<<nb, 256, 0, st>>>(dst32, (bf16x2*)dsth, nblk, nc);
}

void launch_coarse_mv(const GeomDev& g, dd_dtype vt, int nc, const void* Dc, const void* Minv, int use_inv, int nrhs,
                      int site_begin, int count, double a_self, const void* xs, double a_hop, const void* xh,
                      double beta, const void* z, void* out, hipStream_t st, int spw, dd_dtype bt, bool hm,
                      bool post_inv) {
  if (count <= 0) return;
  const int nblk = (a_self != 0.0 ? 1 : 0) + (a_hop != 0.0 ? 8 : 0) + (post_inv ? 1 : 0);
  const double bytes = (double)count * nblk * nc * nc * storage_pair_bytes(bt) +
                       (double)count * nc * nrhs * vector_pair_bytes(vt) * (2 + (beta != 0.0 ? 1 : 0));
  const double flops = 8.0 * count * nblk * nc * nc * nrhs;
  if (vt == DD_F64) {
    const MfmaLaunch<double> k = full_pick<double2, double>(nc, g.Vc, count, post_inv, nrhs);
    DD_TIMED("k_coarse_mv", st, bytes, flops,
             (k.fn<<<k.grid, k.blk, 0, st>>>(g, Dc, Minv, use_inv, nrhs, site_begin, count, a_self, (const double2*)xs,
                                             a_hop, (const double2*)xh, beta, (const double2*)z, (double2*)out,
                                             current_gate())));
    return;
  }
  hm = hm && (bt == DD_F16 || bt == DD_BF16);
  const MfmaLaunch<float> k = bt == DD_F16    ? (hm ? half_pick<__half2>(nc, count, spw) : full_pick<__half2, float>(nc, g.Vc, count, post_inv, nrhs))
                              : bt == DD_BF16 ? (hm ? half_pick<bf16x2>(nc, count, spw) : full_pick<bf16x2, float>(nc, g.Vc, count, post_inv, nrhs))
                                              : full_pick<float2, float>(nc, g.Vc, count, post_inv, nrhs);
  DD_TIMED("k_coarse_mfma", st, bytes, flops,
           (k.fn<<<k.grid, k.blk, 0, st>>>(g, Dc, Minv, use_inv, nrhs, site_begin, count, (float)a_self,
                                           (const float2*)xs, (float)a_hop, (const float2*)xh, (float)beta,
                                           (const float2*)z, (float2*)out, current_gate())));
}

// canonical coarse vectors [rhs][lex][nc] complex128 <-> packed [rhs][slot][nc]
namespace {
template <typename Tv>
__global__ void k_coarse_perm(GeomDev g, int nc, int nrhs, int to_packed, const void* __restrict__ src,
                              void* __restrict__ dst) {
  long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long per = (long long)g.Vc * nc;
  if (e >= per * nrhs) return;
  long long r = e / per, q = e % per;
  int slot = (int)(q / nc), k = (int)(q % nc);
  int bc = g.blk_coord[slot];
  int NB0 = g.L[0] / g.b[0], NB1 = g.L[1] / g.b[1], NB2 = g.L[2] / g.b[2];
  long long lex = (bc & 255) + NB0 * (((bc >> 8) & 255) + NB1 * (((bc >> 16) & 255) + (long long)NB2 * ((bc >> 24) & 255)));
  long long ip = r * per + (long long)slot * nc + k, ic = r * per + lex * nc + k;
  if (to_packed) {
    double2 v = ((const double2*)src)[ic];
    st<Tv, double>((Tv*)dst + ip, cx<double>{v.x, v.y});
  } else {
    cx<double> v = ld<double, Tv>((const Tv*)src + ip);
    ((double2*)dst)[ic] = make_double2(v.re, v.im);
  }
}
}  // namespace

void launch_coarse_perm(const GeomDev& g, dd_dtype vt, int nc, int nrhs, int to_packed, const void* src, void* dst,
                        hipStream_t st) {
  long long n = (long long)g.Vc * nc * nrhs;
  unsigned nb = (unsigned)((n + 255) / 256);
  if (vt == DD_F64)
    k_coarse_perm<double2><<<nb, 256, 0, st>>>(g, nc, nrhs, to_packed, src, dst);
  else
    k_coarse_perm<float2><<<nb, 256, 0, st>>>(g, nc, nrhs, to_packed, src, dst);
}
