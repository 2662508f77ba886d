// Wilson-clover operator apply: out = A psi + hopping term (Sec. 3), one
// thread per (site, right-hand side).  Tiles are visited in slab order: the
// workgroups of one tile (all right-hand sides) run on the same XCD back to back,
// so its links and clover come from that XCD's L2 after the first fetch, and
// neighbouring blocks run together on that XCD, so halo spinors and backward
// links are shared through the same L2.  Lattices with 4^4 blocks take the
// block form (k_dirac_blk), whose in-block hops read spinors staged in LDS.
#include "dslash.h"
#include "ktimer.h"

namespace {

template <typename R, typename S, typename Tv, typename To = Tv>
__global__ void __launch_bounds__(256) k_dirac(GeomDev g, const S* __restrict__ links, const S* __restrict__ clov,
                                               int nrhs, const Tv* __restrict__ in, To* __restrict__ out) {
  int tile, r;
  if (g.Bv >= (int)blockDim.x) {   // whole blocks per tile range: slab order (see xcd_slab_tile)
    if (!xcd_slab_tile(g, g.Bv / blockDim.x, nrhs, tile, r)) return;
  } else {
    xcd_tile_rhs(nrhs, tile, r);
  }
  long long I = (long long)tile * blockDim.x + threadIdx.x;
  if (I >= g.V) return;
  const Tv* x = in + (long long)r * 12 * g.V;
  SiteLoc s = decode_site(g, I);
  cx<R> psi[12], acc[12];
  load_spinor<R, Tv>(x, g.V, I, psi);
  clover_mul<R, S, false>(clov, g.V, I, psi, acc);
  auto fetch = [&](long long J, bool, cx<R>* p) { load_spinor<R, Tv>(x, g.V, J, p); };
  hop_all<R, S>(g, links, s, I, false, fetch, acc);
  store_spinor<R, To>(out + (long long)r * 12 * g.V, g.V, I, acc);
}

// Streams that no other workgroup reads soon take non-temporal accesses, so that L2
// keeps what is read again: the links (a site's forward link is its backward
// neighbour's backward link), the spinors of x and y neighbours and, for the other
// right-hand sides' workgroups, the operator.  The streams are the output, with one
// right-hand side the clover operand, and with more than four z and t neighbours'
// spinors where x and y ones are read ahead (FP64).  32^3x64, FP64, twelve right-hand
// sides: 6112 us without, 5950 with the output, 5862 with the neighbours as well; y
// neighbours too 5820, but 4 % slower on 24^3x48; the own spinors too 7236.  (Two and
// three right-hand sides, 16^3x24, neighbours streamed / not: 50.5 / 47.2, 73.8 / 68.8.)
template <typename R, typename S>
__device__ __forceinline__ cx<R> ld_stream(const S* p) {
  return ld<R, S>(p);
}
template <>
__device__ __forceinline__ cx<double> ld_stream<double, double2>(const double2* p) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
  return {v.x, v.y};
}
template <>
__device__ __forceinline__ cx<float> ld_stream<float, float2>(const float2* p) {
  typedef float v2 __attribute__((ext_vector_type(2)));
  const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
  return {v.x, v.y};
}
template <typename To, typename R>
__device__ __forceinline__ void st_stream(To* p, cx<R> v) {
  st<To, R>(p, v);
}
template <>
__device__ __forceinline__ void st_stream<double2, double>(double2* p, cx<double> v) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  __builtin_nontemporal_store(v2{v.re, v.im}, reinterpret_cast<v2*>(p));
}
template <>
__device__ __forceinline__ void st_stream<float2, float>(float2* p, cx<float> v) {
  typedef float v2 __attribute__((ext_vector_type(2)));
  __builtin_nontemporal_store(v2{v.re, v.im}, reinterpret_cast<v2*>(p));
}

template <typename R, typename Tv>
__device__ __forceinline__ void load_spinor_stream(const Tv* p, long long V, long long I, cx<R>* psi) {
#pragma unroll
  for (int c = 0; c < 12; ++c) psi[c] = ld_stream<R, Tv>(p + (long long)c * V + I);
}

// C psi for the packed clover (two Hermitian 6x6 blocks), operand read as a stream
template <typename R, typename S>
__device__ __forceinline__ void clover_mul_stream(const S* C, long long V, long long I, const cx<R>* in,
                                                  cx<R>* out) {
#pragma unroll 1
  for (int c = 0; c < 2; ++c) {
    const S* B = C + (long long)(18 * c) * V + I;
    cx<R> v[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) v[r] = c ? in[6 + r] : in[r];
    cx<R> o[6];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const cx<R> d = ld_stream<R, S>(B + k * V);
      o[2 * k] = d.re * v[2 * k];
      o[2 * k + 1] = d.im * v[2 * k + 1];
    }
    int k = 3;
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
      for (int q = r + 1; q < 6; ++q) {
        const cx<R> u = ld_stream<R, S>(B + (long long)(k++) * V);
        cfma4(o[r], u, v[q]);
        cfma4_conj(o[q], u, v[r]);
      }
#pragma unroll
    for (int r = 0; r < 6; ++r) {   // constant indices (c is not unrolled): acc stays in registers
      if (c) out[6 + r] = o[r];
      else out[r] = o[r];
    }
  }
}

// Face halo of a 4^4 block in LDS.  Face f (mu = f >> 1; f even: the hop +mu, f odd:
// -mu) has 64 sites, one wave: lane p takes the neighbour of the face site whose
// other three coordinates are the base-4 digits of p, reads its spinor and keeps
// the projected half spinor (6 entries) of that hop in halo[f][.][p].
//
// The halos are read with the block's own spinors, before the operator streams
// through.  Read where each hop needs them, the lines of the x and y neighbours
// (which hold few face sites each) had left the L2 by then, although those
// blocks run on the same XCD at nearly the same time.
__device__ __forceinline__ int face_pos(int mu, const int l[4]) {
  // the base-4 digits l[0..3] without digit mu
  const int all = l[0] | (l[1] << 2) | (l[2] << 4) | (l[3] << 6), low = (1 << (2 * mu)) - 1;
  return (all & low) | ((all >> 2) & ~low & 63);
}
template <int F, typename R, typename Tv>
__device__ __forceinline__ void face_load(const GeomDev& g, int slot, const Tv* __restrict__ x, int p,
                                          cx<R> (*halo)[64]) {
  constexpr int MU = F >> 1;
  constexpr bool fwd = (F & 1) == 0;
  SiteLoc s;
  s.slot = slot;
  int e = p;
#pragma unroll
  for (int d = 0; d < 4; ++d)
    if (d != MU) {
      s.l[d] = e & 3;
      e >>= 2;
    }
  s.l[MU] = fwd ? 0 : 3;   // the neighbour's coordinate
  const int nb = g.blk_nbr[(fwd ? MU : 4 + MU) * g.Vc + slot] & DD_SLOT_MASK;
  const long long J = (long long)nb * 256 + encode_local(g, s.l);
  cx<R> psi[12], h[6];
  load_spinor<R, Tv>(x, g.V, J, psi);
  project<MU, fwd ? -1 : +1, R>(psi, h);
#pragma unroll
  for (int c = 0; c < 6; ++c) halo[c][p] = h[c];
}
// faces 0 .. NF - 1 of the block, dealt to the four waves of the workgroup
template <int NF, typename R, typename Tv>
__device__ __forceinline__ void load_faces(const GeomDev& g, int slot, const Tv* __restrict__ x,
                                           cx<R> (*halo)[6][64]) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 3, p = threadIdx.x & 63;
#pragma unroll
  for (int f0 = 0; f0 < NF; f0 += 4) {
    switch (f0 + w) {
#define DD_FACE(F) \
  case F:          \
    if constexpr (F < NF) face_load<F, R, Tv>(g, slot, x, p, halo[F]); \
    break;
      DD_FACE(0) DD_FACE(1) DD_FACE(2) DD_FACE(3) DD_FACE(4) DD_FACE(5) DD_FACE(6) DD_FACE(7)
#undef DD_FACE
      default: break;
    }
  }
}

// The eight hops in the order of hop_all (forward then backward per direction),
// with both links of a direction loaded together: the backward neighbour's
// forward link U_mu(x - mu) lies, for most sites, in the lines the workgroup's
// own forward loads have just fetched, which the L2 does not keep until a
// later backward hop once many blocks stream through it.  fetch(k, J, inside,
// psi) gives the neighbour's spinor, or its half spinor with zero lower spins.
template <typename R, typename S, typename Fetch>
__device__ __forceinline__ void hop_pairs(const GeomDev& g, const S* links, const SiteLoc& s, long long I,
                                          Fetch fetch, cx<R>* acc) {
#pragma unroll 1
  for (int mu = 0; mu < 4; ++mu) {
    bool wf, inf, wb, inb;
    const long long Jf = neighbor(g, s, mu, +1, wf, inf);
    const long long Jb = neighbor(g, s, mu, -1, wb, inb);
    cx<R> uf[9], ub[9], psi[12];
    load_link<R, S>(links, g.V, mu, I, uf);
    load_link<R, S>(links, g.V, mu, Jb, ub);
    fetch(2 * mu, Jf, inf, psi);
    const R cf = (R)1 * (R)(wf ? -0.5 * g.bc_t : -0.5);
    switch (mu) {
      case 0: hop_t<0, -1, false, R>(uf, psi, cf, acc); break;
      case 1: hop_t<1, -1, false, R>(uf, psi, cf, acc); break;
      case 2: hop_t<2, -1, false, R>(uf, psi, cf, acc); break;
      default: hop_t<3, -1, false, R>(uf, psi, cf, acc); break;
    }
    fetch(2 * mu + 1, Jb, inb, psi);
    const R cb = (R)1 * (R)(wb ? -0.5 * g.bc_t : -0.5);
    switch (mu) {
      case 0: hop_t<0, +1, true, R>(ub, psi, cb, acc); break;
      case 1: hop_t<1, +1, true, R>(ub, psi, cb, acc); break;
      case 2: hop_t<2, +1, true, R>(ub, psi, cb, acc); break;
      default: hop_t<3, +1, true, R>(ub, psi, cb, acc); break;
    }
  }
}

// Block form (blocks of 256 sites: one workgroup of Bv = 256 threads per block and
// right-hand side).  The block's spinors and its first NF faces' half spinors
// (4^4 blocks only, see face_load) are staged in LDS once; hops read them there, so
// memory sees one read of every spinor plus the faces.  NF (see blk_launch) is what
// leaves the CU its workgroups:
// all eight faces in FP32 (48 KB), x and y in FP64 (72 KB; the z and t faces are whole
// lines, and their blocks run far apart in the slab order).  Bound by traffic:
// at 32^3x64, FP64, twelve right-hand sides, 31.2 GB a launch (2.6 times the
// algorithmic bytes) at 5.3 TB/s; two right-hand sides of a block in one workgroup
// measured slower (7.2 against 6.1 ms).
template <typename R, typename S, typename Tv, typename To, bool NT, int NF, bool FAR>
__global__ void __launch_bounds__(256) k_dirac_blk(GeomDev g, const S* __restrict__ links,
                                                   const S* __restrict__ clov, int nrhs, const Tv* __restrict__ in,
                                                   To* __restrict__ out) {
  __shared__ cx<R> sp[12][256];
  __shared__ cx<R> halo[NF ? NF : 1][6][64];
  int tile, r;
  if (!xcd_slab_tile(g, 1, nrhs, tile, r)) return;   // uniform per workgroup
  const long long base = (long long)tile * 256;
  const long long I = base + threadIdx.x;
  const Tv* x = in + (long long)r * 12 * g.V;
  SiteLoc s = decode_site(g, I);
  cx<R> psi[12], acc[12];
  load_spinor<R, Tv>(x, g.V, I, psi);
#pragma unroll
  for (int c = 0; c < 12; ++c) sp[c][threadIdx.x] = psi[c];
  load_faces<NF, R, Tv>(g, tile, x, halo);
  __syncthreads();
  if constexpr (NT) clover_mul_stream<R, S>(clov, g.V, I, psi, acc);
  else clover_mul<R, S, false>(clov, g.V, I, psi, acc);
  auto fetch = [&](int k, long long J, bool inside, cx<R>* p) {
    if (inside) {
      const int j = (int)(J - base);
#pragma unroll
      for (int c = 0; c < 12; ++c) p[c] = sp[c][j];
    } else if (k < NF) {
      const int q = face_pos(k >> 1, s.l);
#pragma unroll
      for (int c = 0; c < 6; ++c) p[c] = halo[k][c][q];
#pragma unroll
      for (int c = 6; c < 12; ++c) p[c] = {(R)0, (R)0};
    } else {
      if constexpr (FAR) load_spinor_stream<R, Tv>(x, g.V, J, p);   // z and t neighbours
      else load_spinor<R, Tv>(x, g.V, J, p);
    }
  };
  hop_pairs<R, S>(g, links, s, I, fetch, acc);
  To* o = out + (long long)r * 12 * g.V;
#pragma unroll
  for (int c = 0; c < 12; ++c) st_stream<To, R>(o + (long long)c * g.V + I, acc[c]);
}

// Half-precision operands, several right-hand sides (4^4 blocks): one workgroup
// per block takes every right-hand side in turn.  A site's 8 links (4 forward,
// the 4 backward U_mu(x - mu)) stay in registers in their storage type (72
// 32-bit registers) and the block's packed clover in LDS, both loaded once, so
// links and clover are read once per launch instead of once per right-hand
// side.  Each right-hand side's block spinors are staged in LDS; hops across the
// block faces read memory.  Same arithmetic, in the same order, as k_dirac_blk.
template <typename S, int STRIDE>
__device__ __forceinline__ void clover_rows(const S* C, const cx<float>* in, cx<float>* out) {
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const S* B = C + 18 * c * STRIDE;
    cx<float> v[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) v[r] = in[6 * c + r];
    cx<float> o[6];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const cx<float> d = ld<float, S>(B + k * STRIDE);
      o[2 * k] = d.re * v[2 * k];
      o[2 * k + 1] = d.im * v[2 * k + 1];
    }
    int k = 3;
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
      for (int q = r + 1; q < 6; ++q) {
        const cx<float> u = ld<float, S>(B + (k++) * STRIDE);
        cfma4(o[r], u, v[q]);
        cfma4_conj(o[q], u, v[r]);
      }
#pragma unroll
    for (int r = 0; r < 6; ++r) out[6 * c + r] = o[r];
  }
}

template <typename S>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_dirac_hl(
    GeomDev g, const S* __restrict__ links, const S* __restrict__ clov, int nrhs, int full, int parts,
    const float2* __restrict__ in, float2* __restrict__ out) {
  __shared__ cx<float> sp[12][256];
  __shared__ S sc[36][256];
  // slab order (xcd_slab_tile): the first `full` blocks of an XCD's eighth with every right-hand side, the rest in
  // `parts` workgroups each (see hl_split)
  const int k = blockIdx.x >> 3, t = k - full;
  const int kk = t < 0 ? k : full + t / parts, part = t < 0 ? 0 : t % parts, np = t < 0 ? 1 : parts;
  const int tile = g.lex_slot[(blockIdx.x & 7) * (g.Vc / 8) + kk];
  const int r0 = part * nrhs / np, r1 = (part + 1) * nrhs / np;
  const long long V = g.V, base = (long long)tile * 256, I = base + threadIdx.x;
  const SiteLoc s = decode_site(g, I);
  unsigned J[8];   // packed neighbour indices (V < 2^32)
  unsigned inside = 0, wrap = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    bool w, in_;
    J[k] = (unsigned)neighbor(g, s, k >> 1, (k & 1) ? -1 : +1, w, in_);
    inside |= (unsigned)in_ << k;
    wrap |= (unsigned)w << k;
  }
  S u[8][9];
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int e = 0; e < 9; ++e)
      u[k][e] = links[(long long)((k >> 1) * 9 + e) * V + ((k & 1) ? (long long)J[k] : I)];
#pragma unroll
  for (int e = 0; e < 36; ++e) sc[e][threadIdx.x] = clov[(long long)e * V + I];
#pragma unroll 1
  for (int r = r0; r < r1; ++r) {
    const float2* x = in + (long long)r * 12 * V;
    cx<float> psi[12], acc[12];
    load_spinor<float, float2>(x, V, I, psi);
    __syncthreads();   // the previous right-hand side's reads of sp are done
#pragma unroll
    for (int c = 0; c < 12; ++c) sp[c][threadIdx.x] = psi[c];
    __syncthreads();
    clover_rows<S, 256>(&sc[0][threadIdx.x], psi, acc);
#pragma unroll 1
    for (int k = 0; k < 8; ++k) {
      cx<float> nb[12], uk[9];
      if ((inside >> k) & 1) {
        const int jl = (int)(J[k] - (unsigned)base);
#pragma unroll
        for (int c = 0; c < 12; ++c) nb[c] = sp[c][jl];
      } else {
        load_spinor<float, float2>(x, V, (long long)J[k], nb);
      }
      const float coef = -0.5f * (((wrap >> k) & 1) ? (float)g.bc_t : 1.f);
      switch (k) {
#define DD_HOP(K, MU, SG, DG)                                                      \
  case K:                                                                         \
    _Pragma("unroll") for (int e = 0; e < 9; ++e) uk[e] = ld<float, S>(&u[K][e]); \
    hop_t<MU, SG, DG, float>(uk, nb, coef, acc);                                  \
    break;
        DD_HOP(0, 0, -1, false)
        DD_HOP(1, 0, +1, true)
        DD_HOP(2, 1, -1, false)
        DD_HOP(3, 1, +1, true)
        DD_HOP(4, 2, -1, false)
        DD_HOP(5, 2, +1, true)
        DD_HOP(6, 3, -1, false)
        default: DD_HOP(7, 3, +1, true)
#undef DD_HOP
      }
    }
    store_spinor<float, float2>(out + (long long)r * 12 * V, V, I, acc);
  }
}

// useful flops of one site's D apply: eight hops (project, SU(3) times a half
// spinor, reconstruct and accumulate: 1320), the two packed 6x6 clover blocks
// (504) and the final sum (24)
constexpr double kDiracFlopsPerSite = 1320.0 + 504.0 + 24.0;

}  // namespace

// Block form.  With one right-hand side the clover is streamed.
// Faces in LDS (the same bits as without): x and y in FP64, all in FP32, none for half
// operands (their launch moves half the bytes, and the halos gave nothing), none on
// lattices of at most 256 blocks, which run together anyway, so that the faces
// would be one more latency, and none on FP64 spinors for more than four right-hand
// sides on up to 1024 blocks.  (FP32 spinors under the FP64 operator, as the outer solver
// applies it, gain there too.)  None either for blocks
// of 256 sites with other edges than four, whose faces do not have face_load's 64
// sites.  us, without / with faces: FP64 384 blocks (16^3x24) one right-hand side 33.7 / 31.9,
// two 46.9 / 47.2, five 105 / 110, twelve 245 / 268; 768 (16^2x24x32) four 177 / 173, twelve 486 /
// 517; 2592 (24^3x48) two 367 / 354, twelve 1797 / 1723; 32^3x64 one 733 / 697, twelve 6522 / 5862;
// FP32 16^3x24 one 22.5 / 21.2, twelve 134 / 130, 24^3x48 117 / 107, 1128 / 1012; 8^4 FP32 13.1 / 14.1,
// FP64 14.1 / 15.8.  FP64 operator on FP32 spinors within a solve: 16^3x32 five 139 / 132, twelve 295 / 279,
// 16^2x32^2 twelve 620 / 574.
template <typename R, typename S, typename Tv, typename To>
void blk_launch(const GeomDev& g, const OpSet& ops, int nrhs, const void* in, void* out, hipStream_t st) {
  const unsigned nb = xcd_grid(g.Vc, nrhs);
  const S* L = (const S*)ops.links;
  const S* C = (const S*)ops.clover;
  constexpr bool F64 = sizeof(R) == 8;
  constexpr int NF = F64 ? 4 : sizeof(S) == 8 ? 8 : 0;
  const bool faces = g.Vc > 256 && g.b[0] == 4 && g.b[1] == 4 && g.b[2] == 4 && g.b[3] == 4 &&
                     (sizeof(Tv) == 8 || nrhs <= 4 || g.Vc > 1024);
  auto* fn = nrhs == 1 ? (faces ? k_dirac_blk<R, S, Tv, To, true, NF, false> : k_dirac_blk<R, S, Tv, To, true, 0, false>)
             : !faces  ? k_dirac_blk<R, S, Tv, To, false, 0, false>
             : F64 && nrhs > 4 ? k_dirac_blk<R, S, Tv, To, false, NF, F64>
                               : k_dirac_blk<R, S, Tv, To, false, NF, false>;
  fn<<<nb, 256, 0, st>>>(g, L, C, nrhs, (const Tv*)in, (To*)out);
}

static void blk_dispatch(const GeomDev& g, dd_dtype dt, const OpSet& ops, int nrhs, const void* in, void* out,
                         hipStream_t st) {
  switch (dt) {
    case DD_F64: blk_launch<double, double2, double2, double2>(g, ops, nrhs, in, out, st); break;
    case DD_F32: blk_launch<float, float2, float2, float2>(g, ops, nrhs, in, out, st); break;
    case DD_F16: blk_launch<float, __half2, float2, float2>(g, ops, nrhs, in, out, st); break;
    case DD_BF16: blk_launch<float, bf16x2, float2, float2>(g, ops, nrhs, in, out, st); break;
  }
}

// Blocks of an XCD (32 CUs, two workgroups each) beyond whole rounds of 64 would take a
// round of all right-hand sides, most of the chip idle: they are split over the
// right-hand sides, into the number of workgroups with the least rounds times work
// (a block's links and clover cost about as much as one right-hand side).  us before /
// after, BF16: 24^3x48 (4 left of 324) five right-hand sides 388 / 361, twelve 868 / 789;
// 24^4 (34 of 162, in three) twelve 439 / 414; 8^4 (2) two 18.2 / 12, twelve 78.5 / 12.8;
// none left over, 16^3x32: 60 / 60.
static void hl_split(int blocks, int nrhs, int& full, int& parts) {
  constexpr int kSlots = 64;
  const int rest = blocks % kSlots;
  full = blocks - rest;
  parts = 1;
  int best = 1 << 30;
  for (int p = 1; p <= std::min(nrhs, kSlots); ++p) {
    const int cost = ((rest * p + kSlots - 1) / kSlots) * (1 + (nrhs + p - 1) / p);
    if (cost < best) best = cost, parts = p;
  }
}

// blocks of 256 sites have a workgroup each, in slab order
bool dirac_threads_read(const GeomDev& g) { return g.Bv != 256 || g.Vc % 16 != 0; }

static void dirac_dispatch(const GeomDev& g, dd_dtype dt, const OpSet& ops, int nrhs, const void* in, void* out,
                           int threads, hipStream_t st) {
  if (!dirac_threads_read(g) && nrhs >= 2 && (dt == DD_F16 || dt == DD_BF16)) {
    // operator in registers across the right-hand sides
    int full, parts;
    hl_split(g.Vc / 8, nrhs, full, parts);
    const unsigned nb = 8 * (full + (g.Vc / 8 - full) * parts);
    if (dt == DD_F16)
      k_dirac_hl<__half2><<<nb, 256, 0, st>>>(g, (const __half2*)ops.links, (const __half2*)ops.clover, nrhs, full,
                                               parts, (const float2*)in, (float2*)out);
    else
      k_dirac_hl<bf16x2><<<nb, 256, 0, st>>>(g, (const bf16x2*)ops.links, (const bf16x2*)ops.clover, nrhs, full,
                                              parts, (const float2*)in, (float2*)out);
    return;
  }
  if (!dirac_threads_read(g)) {   // block form, slab order over the blocks
    blk_dispatch(g, dt, ops, nrhs, in, out, st);
    return;
  }
  if (threads != 64 && threads != 128) threads = 256;
  unsigned nb = xcd_grid((unsigned)((g.V + threads - 1) / threads), nrhs);
  switch (dt) {
    case DD_F64:
      k_dirac<double, double2, double2><<<nb, threads, 0, st>>>(g, (const double2*)ops.links, (const double2*)ops.clover,
                                                            nrhs, (const double2*)in, (double2*)out);
      break;
    case DD_F32:
      k_dirac<float, float2, float2><<<nb, threads, 0, st>>>(g, (const float2*)ops.links, (const float2*)ops.clover, nrhs,
                                                         (const float2*)in, (float2*)out);
      break;
    case DD_F16:
      k_dirac<float, __half2, float2><<<nb, threads, 0, st>>>(g, (const __half2*)ops.links, (const __half2*)ops.clover,
                                                          nrhs, (const float2*)in, (float2*)out);
      break;
    case DD_BF16:
      k_dirac<float, bf16x2, float2><<<nb, threads, 0, st>>>(g, (const bf16x2*)ops.links, (const bf16x2*)ops.clover, nrhs,
                                                         (const float2*)in, (float2*)out);
      break;
  }
}

void launch_dirac(const GeomDev& g, dd_dtype dt, const OpSet& ops, int nrhs, const void* in, void* out,
                  hipStream_t st, int threads) {
  // algorithmic traffic: spinor in + out per RHS, 4 links + packed clover once per site
  double bytes = (double)g.V * (24.0 * vector_pair_bytes(dt) * nrhs + 72.0 * storage_pair_bytes(dt));
  double flops = (double)g.V * nrhs * kDiracFlopsPerSite;
  DD_TIMED("k_dirac", st, bytes, flops, dirac_dispatch(g, dt, ops, nrhs, in, out, threads, st));
}

void launch_dirac_f32_in(const GeomDev& g, const OpSet& ops64, int nrhs, const float2* in, double2* out,
                         hipStream_t st, int threads) {
  // FP64 operator on an FP32 input (widened exactly on load), FP64 output
  const double bytes = (double)g.V * (12.0 * (sizeof(float2) + sizeof(double2)) * nrhs + 72.0 * sizeof(double2));
  const double flops = (double)g.V * nrhs * kDiracFlopsPerSite;
  const double2* L = (const double2*)ops64.links;
  const double2* C = (const double2*)ops64.clover;
  if (!dirac_threads_read(g)) {
    DD_TIMED("k_dirac", st, bytes, flops,
             (blk_launch<double, double2, float2, double2>(g, ops64, nrhs, in, out, st)));
    return;
  }
  if (threads != 64 && threads != 128) threads = 256;
  const unsigned nb = xcd_grid((unsigned)((g.V + threads - 1) / threads), nrhs);
  DD_TIMED("k_dirac", st, bytes, flops,
           (k_dirac<double, double2, float2, double2><<<nb, threads, 0, st>>>(g, L, C, nrhs, in, out)));
}
