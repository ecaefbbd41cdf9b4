// The multi-level gravity iteration on a uniform octree (the paper's
// three-step iteration, Sec. VII-C: bottom-up traversal, cell-to-cell
// interactions on every level, top-down traversal; Sec. IV-C: the octree's
// cells carry multipole moments).
//
// Domain: n^3 finest cells of spacing h; level l has n / 2^l cells per axis of
// spacing 2^l h, down to 4 per axis. Level arrays are [C][n_l][n_l][n_l]
// (x fastest), finest level first, back to back.
//
//   P2M  finest level: M_k(j) = sum_i m_i (y_i - c_j)^k / k!
//   M2M  M_k(J) = sum_{children j} sum_{q <= k} M_q(j) s^(k-q) / (k-q)!,  s = c_j - c_J
//   M2L  every level: L_n(t) = sum_{d in IL(t)} sum_k M_k(t + d) T_d[k][n] at the
//        level's spacing, IL(t) = {d : |d|^2 > 4, |floor((t mod 2 + d) / 2)|^2 <= 4}
//        (sources not near the target whose parents are near the target's
//        parent); on the 4-per-axis level every parent is near every other, so
//        the same lists give all non-near sources there. Sources outside the
//        domain are absent.
//   L2L  L_n(j) += sum_{m >= n} L_m(J) s^(m-n) / (m-n)!, coarsest level first.
//
// IL(t) depends only on the parity sigma of t: 231 offsets per parity, all
// inside the shell 5 <= |d|^2 <= 36 with |d_i| <= 5. The level M2L kernel
// gives each of its waves one parity class of an 8^3 target block (or of one of
// its planes), so a wave's 16-cell tiles, one per plane of that z parity, share
// one offset list and one table stream: [16 cells x 4 offsets] x [4 offsets x
// columns] on v_mfma_f64_16x16x4 and 4x4x4_4b as in the single-level kernels,
// with the source window of two moment components per round in LDS. The harmonic
// form (as FMM_FP64_HARMONIC: T_d is harmonic in both
// indices, so the moments fold onto the (p+1)^2 components with kz <= 1 and
// only those columns of L are computed, then expanded) uses the single-level
// form's fold plan per round and expansion of L.
#include <vector>

#include "kernels.h"
#include "m2l_mfma.h"
#include "p2m_common.h"

namespace fmm {

namespace {

constexpr int kTreeW = 18;                         // window (y, z): block cells -5 .. 12
constexpr int kTreeList = 231;                     // interaction-list length per parity
constexpr int kTreeQuads = (kTreeList + 3) / 4;    // 58 (the last quad has one empty slot)
constexpr int kTreeMaxLevels = 8;
constexpr int kTreeWideMin = 64;                   // levels of at least this many cells per axis: wide workgroups

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4d mfma16(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// b^i / i! per axis for i <= P
template <int P>
__device__ __forceinline__ void powers(double bx, double by, double bz, double (&px)[P + 1],
                                       double (&py)[P + 1], double (&pz)[P + 1]) {
  px[0] = py[0] = pz[0] = 1.0;
#pragma unroll
  for (int i = 1; i <= P; ++i) {
    px[i] = px[i - 1] * bx * (1.0 / i);
    py[i] = py[i - 1] * by * (1.0 / i);
    pz[i] = pz[i - 1] * bz * (1.0 / i);
  }
}

// The (k, q) pairs with q <= k componentwise and their difference r = k - q,
// built at compile time so the shift loops unroll into straight-line code.
template <int P>
struct ShiftTerms {
  int n;
  signed char k[ncomp(P) * ncomp(P)], q[ncomp(P) * ncomp(P)];
  signed char rx[ncomp(P) * ncomp(P)], ry[ncomp(P) * ncomp(P)], rz[ncomp(P) * ncomp(P)];
};
template <int P>
constexpr ShiftTerms<P> make_shift_terms() {
  ShiftTerms<P> t{};
  for (int ck = 0; ck < ncomp(P); ++ck) {
    const MI k = mi_of(ck);
    for (int cq = 0; cq < ncomp(P); ++cq) {
      const MI q = mi_of(cq);
      if (q.x <= k.x && q.y <= k.y && q.z <= k.z) {
        t.k[t.n] = (signed char)ck;
        t.q[t.n] = (signed char)cq;
        t.rx[t.n] = (signed char)(k.x - q.x);
        t.ry[t.n] = (signed char)(k.y - q.y);
        t.rz[t.n] = (signed char)(k.z - q.z);
        ++t.n;
      }
    }
  }
  return t;
}

template <int P>
__global__ void __launch_bounds__(256) p2m_grid_kernel(const double* __restrict__ pos,
                                                       const double* __restrict__ mass, int ppc,
                                                       int n, double h, double* __restrict__ M) {
  constexpr int C = ncomp(P);
  const int64_t n3 = (int64_t)n * n * n;
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= n3) return;
  const int x = (int)(j % n), y = (int)((j / n) % n), z = (int)(j / ((int64_t)n * n));
  const double cx = (x + 0.5) * h, cy = (y + 0.5) * h, cz = (z + 0.5) * h;
  double acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = 0.0;
  for (int i = 0; i < ppc; ++i) {
    const int64_t pi = j * ppc + i;
    p2m_accumulate<P>(mass[pi], pos[3 * pi] - cx, pos[3 * pi + 1] - cy, pos[3 * pi + 2] - cz, acc);
  }
#pragma unroll
  for (int c = 0; c < C; ++c) M[c * n3 + j] = acc[c];
}

// A thread per child, the eight of a parent in neighbouring lanes: each shifts its
// child's moments to the parent's centre, then they are summed over the lanes. (A
// thread per parent, its children one after another, is a chain of eight loads and
// shifts: 19 us on the smallest levels. All upward passes of a tree, p = 3: 16^3
// 38.3 -> 15.0 us, 32^3 57.8 -> 22.9, 128^3 541 -> 478.)
template <int P>
__global__ void __launch_bounds__(256) m2m_kernel(const double* __restrict__ Mc,
                                                        double* __restrict__ Mp, int nc, double hc) {
  constexpr int C = ncomp(P);
  const int np = nc / 2;
  const int64_t np3 = (int64_t)np * np * np, nc3 = (int64_t)nc * nc * nc;
  const int64_t i = (int64_t)blockIdx.x * 32 + threadIdx.x / 8;
  if (i >= np3) return;   // (np^3 is a multiple of 64: whole waves)
  const int o = threadIdx.x & 7, ox = o & 1, oy = (o >> 1) & 1, oz = o >> 2;
  const int X = (int)(i % np), Y = (int)((i / np) % np), Z = (int)(i / ((int64_t)np * np));
  const int64_t g = (2 * X + ox) + (int64_t)nc * (2 * Y + oy) + (int64_t)nc * nc * (2 * Z + oz);
  double mc[C], acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) mc[c] = Mc[c * nc3 + g];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = 0.0;
  double px[P + 1], py[P + 1], pz[P + 1];
  powers<P>((ox - 0.5) * hc, (oy - 0.5) * hc, (oz - 0.5) * hc, px, py, pz);
  constexpr ShiftTerms<P> T = make_shift_terms<P>();
#pragma unroll
  for (int e = 0; e < T.n; ++e)
    acc[T.k[e]] = __builtin_fma(mc[T.q[e]], px[T.rx[e]] * py[T.ry[e]] * pz[T.rz[e]], acc[T.k[e]]);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    double s = acc[c];
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    if (o == c % 8) Mp[c * np3 + i] = s;
  }
}

// One child cell per thread: adds its parent's local polynomial re-expanded
// about the child centre.
template <int P>
__global__ void __launch_bounds__(256) l2l_kernel(const double* __restrict__ Lp,
                                                  double* __restrict__ Lc, int nc, double hc) {
  constexpr int C = ncomp(P);
  const int np = nc / 2;
  const int64_t np3 = (int64_t)np * np * np, nc3 = (int64_t)nc * nc * nc;
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= nc3) return;
  const int x = (int)(j % nc), y = (int)((j / nc) % nc), z = (int)(j / ((int64_t)nc * nc));
  const int64_t G = (x >> 1) + (int64_t)np * (y >> 1) + (int64_t)np * np * (z >> 1);
  double lp[C];
#pragma unroll
  for (int c = 0; c < C; ++c) lp[c] = Lp[c * np3 + G];
  double px[P + 1], py[P + 1], pz[P + 1];
  powers<P>(((x & 1) - 0.5) * hc, ((y & 1) - 0.5) * hc, ((z & 1) - 0.5) * hc, px, py, pz);
  // child n from parent m >= n: the terms (k, q) = (m, n) of the shift table
  constexpr ShiftTerms<P> T = make_shift_terms<P>();
  double s[C];
#pragma unroll
  for (int c = 0; c < C; ++c) s[c] = 0.0;
#pragma unroll
  for (int e = 0; e < T.n; ++e)
    s[T.q[e]] = __builtin_fma(lp[T.k[e]], px[T.rx[e]] * py[T.ry[e]] * pz[T.rz[e]], s[T.q[e]]);
#pragma unroll
  for (int c = 0; c < C; ++c) Lc[c * nc3 + j] += s[c];
}

// Tables of the level kernel, per order p:
//   B[sigma][round][quad][group][kk * 4 + j][c2] = T_d[2 round + c2][4 group + j]
// at unit spacing, d = the kk-th offset of the quad in sigma's list (zero for
// the empty slot, k >= C or n >= C). Built from the canonical [892][C][C]
// tables with the map sidx[sigma][quad][kk] (stencil index or -1).
__global__ void pack_tree_kernel(const double* __restrict__ T, int C, const int* __restrict__ sidx,
                                 double* __restrict__ B) {
  const int NG = (C + 3) / 4, R = (C + 1) / 2;
  const int64_t total = (int64_t)8 * R * kTreeQuads * 2 * NG * 16;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    int64_t r_ = e;
    const int c2 = (int)(r_ % 2); r_ /= 2;
    const int v = (int)(r_ % 16); r_ /= 16;
    const int g = (int)(r_ % NG); r_ /= NG;
    const int q = (int)(r_ % kTreeQuads); r_ /= kTreeQuads;
    const int r = (int)(r_ % R);
    const int sigma = (int)(r_ / R);
    const int kk = v >> 2, j = v & 3;
    const int k = 2 * r + c2, nn = 4 * g + j;
    const int s = sidx[(sigma * kTreeQuads + q) * 4 + kk];
    B[e] = (s >= 0 && k < C && nn < C) ? T[((int64_t)s * C + k) * C + nn] : 0.0;
  }
}

// Harmonic tables: Bh[sigma][round][quad][group][kk * 4 + j][c2] =
// T_d[rowk[2 round + c2]][colk[4 group + j]] (zero where a map is -1).
struct TreeHMaps {
  int rowk[32];
  int colk[32];
};
__global__ void pack_tree_h_kernel(const double* __restrict__ T, int C, int R, int NG,
                                   const int* __restrict__ sidx, TreeHMaps mp, double* __restrict__ B) {
  const int64_t total = (int64_t)8 * R * kTreeQuads * 2 * NG * 16;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    int64_t r_ = e;
    const int c2 = (int)(r_ % 2); r_ /= 2;
    const int v = (int)(r_ % 16); r_ /= 16;
    const int g = (int)(r_ % NG); r_ /= NG;
    const int q = (int)(r_ % kTreeQuads); r_ /= kTreeQuads;
    const int r = (int)(r_ % R);
    const int sigma = (int)(r_ / R);
    const int kk = v >> 2, j = v & 3;
    const int k = mp.rowk[2 * r + c2], nn = 4 * g + j < 32 ? mp.colk[4 * g + j] : -1;
    const int s = sidx[(sigma * kTreeQuads + q) * 4 + kk];
    B[e] = (s >= 0 && k >= 0 && nn >= 0) ? T[((int64_t)s * C + k) * C + nn] : 0.0;
  }
}

// Every level in one launch: the levels' blocks back to back, coarsest level
// first, so the few long-running blocks of the small levels start at once and
// overlap with the finest level's many blocks.
struct TreeLevels {
  int nlev;
  int first[kTreeMaxLevels + 1];   // first block of each level in launch order, then the total
  int n[kTreeMaxLevels];           // cells per axis
  int lg[kTreeMaxLevels];          // log2 of the spacing
  int64_t off[kTreeMaxLevels];     // element offset of the level in M and L
};

// Columns of a tile: N16 sixteens on 16x16x4 products, then N4 groups of four on
// 4x4x4 products.
template <int P, bool HARM>
struct TreeCols {
  static constexpr int CR = HARM ? (P + 1) * (P + 1) : ncomp(P);   // contracted components (rows and columns)
  static constexpr int NG = (CR + 3) / 4;
  static constexpr int N16 = CR / 16, N4 = NG - 4 * N16;
};
// A workgroup's targets. Wide: two 8^3 blocks side by side in x, each wave one
// parity class of both (8 tiles; one workgroup per CU). Plane: one plane of one
// block, each wave one of the plane's four parity classes (one tile; two
// workgroups per CU).
template <bool WIDE>
struct TreeShape {
  static constexpr int NBLK = WIDE ? 2 : 1;
  static constexpr int NT = WIDE ? 512 : 256;
  static constexpr int TPW = WIDE ? 8 : 1;
  static constexpr int WX = 8 * NBLK + 10, WZ = WIDE ? kTreeW : 11;   // window cells in x and z
  static constexpr int CELLS = WX * kTreeW * WZ;
  static constexpr int OUT = WIDE ? kNTarget : 64;                    // targets of a write-out pass
  static constexpr int AD = WIDE ? 1 : 3, AR = AD + 1;                // window operands: quads ahead, sets
};
constexpr int kTreeOffPad = 12;   // quads past a list whose offsets are read ahead
constexpr int kTreePad = 8 * 9 * 32;   // and doubles past the tables

// What bounds it: the matrix units, at sizes that fill them (wide: one b128 table
// load per four columns or sixteen serves 8 tiles), and on the coarse levels the
// chain of one tile's products, 2 per quad and round, so the work of a block is
// spread over eight workgroups (planes) and table operands are loaded up to eight
// quads ahead. The window stays in LDS; both shapes take each sum in the order of
// the quads. All levels, harmonic p = 3, against one shape of 4x4x4 products with
// two 8-byte table loads per four columns: n = 8 327 -> 53 us, 32 354 -> 151,
// 64 929 -> 707, 128 5119 -> 4592 (p = 4: 16.5 -> 13.2 ms, dense 26.6 -> 20.5).
template <int P, bool HARM, bool WIDE>
__global__ void __launch_bounds__(TreeShape<WIDE>::NT, WIDE ? 1 : 2) m2l_level_kernel(
    const double* __restrict__ Mall, double* __restrict__ Lall, TreeLevels lv,
    const double* __restrict__ B, const int* __restrict__ doff, const HRound* __restrict__ hround,
    const HExp* __restrict__ hexp) {
  using S = TreeShape<WIDE>;
  using F = TreeCols<P, HARM>;
  constexpr int C = ncomp(P), CR = F::CR, NG = F::NG;
  constexpr int ROUNDS = (CR + 1) / 2;
  constexpr int NBLK = S::NBLK, NT = S::NT, TPW = S::TPW, WX = S::WX, AD = S::AD, AR = S::AR;
  constexpr int WCELLS = S::CELLS;
  constexpr int STAGE = (WCELLS + NT - 1) / NT;
  constexpr int K16 = F::N16 > 0 ? F::N16 : 1, K4 = F::N4 > 0 ? F::N4 : 1;
  constexpr int U = WIDE ? 2 : F::N16 + F::N4 == 1 ? 8 : 4;   // quads of table operands in flight
  static_assert(U % AR == 0 && U + AD <= kTreeOffPad && U * NG * 32 <= kTreePad, "read ahead");
  constexpr int CS = CR | 1;                          // column stride of a cell in the write-out
  // the window, and afterwards the columns of a block (or plane)
  constexpr int SMEM = S::OUT * CS / 2 + 1 > WCELLS ? S::OUT * CS / 2 + 1 : WCELLS;
  __shared__ double2 smem[SMEM];
  __shared__ short s_doff[(8 * kTreeQuads + kTreeOffPad) * 4];
  int li = 0;
  while (li + 1 < lv.nlev && (int)blockIdx.x >= lv.first[li + 1]) ++li;
  const int n = lv.n[li], lg = lv.lg[li];
  const double* __restrict__ M = Mall + lv.off[li];
  double* __restrict__ L = Lall + lv.off[li];
  const int nb = n >= 8 ? n / 8 : 1;
  const int nbx = n >= 8 * NBLK ? n / (8 * NBLK) : 1;
  const int planes = WIDE ? 1 : n < 8 ? n : 8;
  const int blk = ((int)blockIdx.x - lv.first[li]) / planes;
  const int plane = ((int)blockIdx.x - lv.first[li]) % planes;   // of the block (Plane)
  const int B0x = 8 * NBLK * (blk % nbx), B0y = 8 * ((blk / nbx) % nb), B0z = 8 * (blk / (nbx * nb));
  const int W0z = B0z + (WIDE ? 0 : plane) - 5;                  // the window's first plane
  const int64_t n3 = (int64_t)n * n * n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sigma = WIDE ? wave : wave + 4 * (plane & 1);        // parity class of this wave
  const int sx = sigma & 1, sy = (sigma >> 1) & 1, sz = sigma >> 2;
  const int kk = lane >> 4, ci = lane & 15;
  // offsets of the lists, packed (dx + 8) | (dy + 8) << 5 | (dz + 8) << 10, as window deltas
  for (int i = tid; i < (8 * kTreeQuads + kTreeOffPad) * 4; i += NT) {
    const int v = i < 8 * kTreeQuads * 4 ? doff[i] : 8 | (8 << 5) | (8 << 10);
    s_doff[i] = (short)(((v & 31) - 8) + WX * (((v >> 5) & 31) - 8) + WX * kTreeW * (((v >> 10) & 31) - 8));
  }

  // tile t: block t / 4, plane z = 2 (t % 4) + sz, cells (8 (t / 4) + 2 (ci & 3) + sx, 2 (ci >> 2) + sy)
  auto tile_z = [&](int t) { return WIDE ? 2 * (t & 3) + sz : plane; };
  int abase[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
    abase[t] = (8 * (t >> 2) + 2 * (ci & 3) + sx + 5) + WX * (2 * (ci >> 2) + sy + 5) +
               WX * kTreeW * ((WIDE ? tile_z(t) : 0) + 5);
  v4d acc16[TPW][K16];
  double acc4[TPW][K4];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
#pragma unroll
    for (int g = 0; g < F::N16; ++g) acc16[t][g] = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int g = 0; g < F::N4; ++g) acc4[t][g] = 0.0;
  }

  // this thread's window cells: global index, or -1 outside the domain
  // (n^3 <= 2^21 cells per level, so a cell index fits 32 bits)
  int wg[STAGE];
#pragma unroll
  for (int i = 0; i < STAGE; ++i) {
    const int c = tid + i * NT;
    const int gx = B0x - 5 + c % WX, gy = B0y - 5 + (c / WX) % kTreeW, gz = W0z + c / (WX * kTreeW);
    wg[i] = (c < WCELLS && gx >= 0 && gx < n && gy >= 0 && gy < n && gz >= 0 && gz < n)
                ? gx + n * gy + n * n * gz
                : -1;
  }
  // tables through a buffer resource: a per-quad scalar offset and fixed lane
  // offsets (quads read ahead in the last round fall in the tables' padding)
  const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<double*>(B), (short)0, 8 * ROUNDS * kTreeQuads * NG * 256 + kTreePad * 8, 0x00020000);
  const int vb16 = ((ci >> 2) * 16 + kk * 4 + (lane & 3)) * 16;      // column ci of a sixteen
  const int vb4 = (4 * F::N16 * 16 + kk * 4 + (lane & 3)) * 16;
  for (int r = 0; r < ROUNDS; ++r) {
    double s0, s1;
    double2 v[STAGE];
#pragma unroll
    for (int i = 0; i < STAGE; ++i) v[i] = make_double2(0.0, 0.0);
    if (HARM) {
      // the round's two folded components, each an integer combination of moment
      // components of one order
      const HRound& rd = hround[r];
      s0 = ldexp(1.0, -lg * rd.ord0);
      s1 = rd.ord1 >= 0 ? ldexp(1.0, -lg * rd.ord1) : 0.0;
      // two components at a time, so both sets of loads are in flight together
      // (an odd count's last pass reads its component twice, the second time
      // with zero coefficients)
      for (int u = 0; u < rd.nsup; u += 2) {
        const int u1 = u + 1 < rd.nsup ? u + 1 : u;
        const double* srcA = M + (int64_t)rd.comp[u] * n3;
        const double* srcB = M + (int64_t)rd.comp[u1] * n3;
        const double a0 = rd.c0[u], a1 = rd.c1[u];
        const double b0 = u1 != u ? rd.c0[u1] : 0.0, b1 = u1 != u ? rd.c1[u1] : 0.0;
        double ma[STAGE], mb[STAGE];
#pragma unroll
        for (int i = 0; i < STAGE; ++i) {
          ma[i] = wg[i] >= 0 ? srcA[wg[i]] : 0.0;
          mb[i] = wg[i] >= 0 ? srcB[wg[i]] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < STAGE; ++i) {
          v[i].x = __builtin_fma(b0, mb[i], __builtin_fma(a0, ma[i], v[i].x));
          v[i].y = __builtin_fma(b1, mb[i], __builtin_fma(a1, ma[i], v[i].y));
        }
      }
    } else {
      const int k0 = 2 * r, k1 = 2 * r + 1;
      s0 = ldexp(1.0, -lg * order_of(k0));
      s1 = k1 < C ? ldexp(1.0, -lg * order_of(k1)) : 0.0;
      const double* src0 = M + (int64_t)k0 * n3;
      const double* src1 = M + (int64_t)(k1 < C ? k1 : k0) * n3;
#pragma unroll
      for (int i = 0; i < STAGE; ++i) {
        if (wg[i] >= 0) {
          v[i].x = src0[wg[i]];
          v[i].y = src1[wg[i]];
        }
      }
    }
    __syncthreads();   // the previous round's window reads are done
#pragma unroll
    for (int i = 0; i < STAGE; ++i) {
      const int c = tid + i * NT;
      if (c < WCELLS) smem[c] = make_double2(v[i].x * s0, v[i].y * s1);
    }
    __syncthreads();
    int sq = (sigma * ROUNDS + r) * kTreeQuads * NG * 256;    // table offset of the quad group
    const short* sp = s_doff + sigma * kTreeQuads * 4 + kk;   // and its window deltas
    double2 b16[U][K16], b4[U][K4], a[AR][TPW];
    int o[U];
#define TR_LOADB(SET, Q)                                                                           \
  {                                                                                                \
    _Pragma("unroll") for (int g = 0; g < F::N16; ++g) b16[SET][g] = __builtin_bit_cast(double2,   \
        __builtin_amdgcn_raw_buffer_load_b128(brs, vb16 + 4 * g * 256, sq + (Q) * NG * 256, 0));   \
    _Pragma("unroll") for (int g = 0; g < F::N4; ++g) b4[SET][g] = __builtin_bit_cast(double2,     \
        __builtin_amdgcn_raw_buffer_load_b128(brs, vb4 + g * 256, sq + (Q) * NG * 256, 0));        \
  }
#define TR_LOADA(SET, OSET) \
  _Pragma("unroll") for (int t = 0; t < TPW; ++t) a[SET][t] = smem[abase[t] + o[OSET]];
#define TR_MMA(u, X)                                                                               \
  _Pragma("unroll") for (int t = 0; t < TPW; ++t) {                                                \
    _Pragma("unroll") for (int g = 0; g < F::N16; ++g) acc16[t][g] = mfma16(a[(u) % AR][t].X, b16[u][g].X, acc16[t][g]); \
    _Pragma("unroll") for (int g = 0; g < F::N4; ++g) acc4[t][g] = mfma4(a[(u) % AR][t].X, b4[u][g].X, acc4[t][g]); \
  }
// one quad: window operands AD quads ahead, then the delta that operand set needs
// next; the products; the table operands of quad u + U. The fences keep the reads
// in issue order, so that every wait covers the oldest reads only.
#define TR_STEP(u)                                                                                 \
  {                                                                                                \
    __builtin_amdgcn_sched_barrier(0);                                                             \
    TR_LOADA(((u) + AD) % AR, ((u) + AD) % U);                                                     \
    o[((u) + AD) % U] = sp[((u) + AD + U) * 4];                                                    \
    TR_MMA(u, x);                                                                                  \
    TR_MMA(u, y);                                                                                  \
    TR_LOADB(u, (u) + U);                                                                          \
    __builtin_amdgcn_sched_barrier(0);                                                             \
  }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      TR_LOADB(u, u);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) o[u] = sp[u * 4];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < AD; ++u) {
      TR_LOADA(u, u % U);
      o[u % U] = sp[(u + U) * 4];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll 1
    for (int q = 0; q < kTreeQuads / U * U; q += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) TR_STEP(u);
      sq += U * NG * 256;
      sp += U * 4;
    }
#pragma unroll
    for (int u = 0; u < kTreeQuads % U; ++u) TR_STEP(u);
#undef TR_LOADB
#undef TR_LOADA
#undef TR_MMA
#undef TR_STEP
  }

  // This lane's sums: cells (2 xi + sx, 2 y + sy) of each tile, column 16 g + ci with
  // y = v, or 4 g + j with y = yi. Through LDS, a block (or the plane) at a time,
  // then each thread writes components of single cells (harmonic form: expanded
  // from the columns; column c has order floor(sqrt(c))).
  const int xi = lane >> 4, yi = (lane & 15) >> 2, j = lane & 3;
  double* sh = reinterpret_cast<double*>(smem);     // [cells][CS], x fastest
#pragma unroll
  for (int b = 0; b < NBLK; ++b) {
    __syncthreads();                                // the window, or the previous block, is no longer read
#pragma unroll
    for (int t = b * (TPW / NBLK); t < (b + 1) * (TPW / NBLK); ++t) {
      auto put = [&](int c, int y, double sum) __attribute__((always_inline)) {
        int ord = order_of(c < C ? c : 0);
        if constexpr (HARM)
          for (ord = 0; (ord + 1) * (ord + 1) <= c;) ++ord;
        const int cell = (2 * xi + sx) + 8 * (2 * y + sy) + (WIDE ? 64 * tile_z(t) : 0);
        if (c < CR) sh[cell * CS + c] = ldexp(sum, -lg * (1 + ord));
      };
#pragma unroll
      for (int g = 0; g < F::N16; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v) put(16 * g + ci, v, acc16[t][g][v]);
#pragma unroll
      for (int g = 0; g < F::N4; ++g) put(16 * F::N16 + 4 * g + j, yi, acc4[t][g]);
    }
    __syncthreads();
    for (int e = tid; e < S::OUT * C; e += NT) {
      const int cell = e % S::OUT, nn = e / S::OUT;
      const int gx = B0x + 8 * b + cell % 8, gy = B0y + (cell / 8) % 8,
                gz = B0z + (WIDE ? cell / 64 : plane);
      if (gx >= n || gy >= n || gz >= n) continue;
      const double* lh = sh + cell * CS;
      double val;
      if constexpr (HARM) {
        const HExp& ex = hexp[nn];
        val = 0.0;
        for (int u = 0; u < ex.nterm; ++u) val = __builtin_fma(ex.coef[u], lh[ex.col[u]], val);
      } else {
        val = lh[nn];
      }
      L[nn * n3 + gx + (int64_t)n * gy + (int64_t)n * n * gz] = val;
    }
  }
}

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

// Interaction lists on the host: for each parity sigma (x + 2 y + 4 z bits),
// the offsets d (dz slowest, then dy, dx, ascending) with |d|^2 > 4 whose
// parents' offset floor((sigma + d) / 2) has squared length <= 4.
static std::vector<int> tree_lists() {
  std::vector<int> out;
  auto fl2 = [](int a) { return a >= 0 ? a / 2 : -((1 - a) / 2); };   // floor(a / 2)
  for (int sigma = 0; sigma < 8; ++sigma) {
    const int sg[3] = {sigma & 1, (sigma >> 1) & 1, sigma >> 2};
    int count = 0;
    for (int dz = -6; dz <= 6; ++dz)
      for (int dy = -6; dy <= 6; ++dy)
        for (int dx = -6; dx <= 6; ++dx) {
          if (dx * dx + dy * dy + dz * dz <= 4) continue;
          const int Dx = fl2(sg[0] + dx), Dy = fl2(sg[1] + dy), Dz = fl2(sg[2] + dz);
          if (Dx * Dx + Dy * Dy + Dz * Dz > 4) continue;
          out.push_back(dx);
          out.push_back(dy);
          out.push_back(dz);
          ++count;
        }
    if (count != kTreeList) return {};
  }
  return out;
}

hipError_t tree_tables_create(TreeTables* tt, const double* const* d_T, const int* stencil_xyz,
                              int nstencil, hipStream_t s) {
  const std::vector<int> lists = tree_lists();
  if (lists.empty()) return hipErrorInvalidValue;
  std::vector<int> sidx(8 * kTreeQuads * 4, -1), doff(8 * kTreeQuads * 4, 8 | (8 << 5) | (8 << 10));
  for (int sigma = 0; sigma < 8; ++sigma)
    for (int e = 0; e < kTreeList; ++e) {
      const int* d = &lists[3 * (sigma * kTreeList + e)];
      int found = -1;
      for (int i = 0; i < nstencil; ++i)
        if (stencil_xyz[3 * i] == d[0] && stencil_xyz[3 * i + 1] == d[1] && stencil_xyz[3 * i + 2] == d[2]) {
          found = i;
          break;
        }
      if (found < 0) return hipErrorInvalidValue;
      sidx[sigma * kTreeQuads * 4 + e] = found;
      doff[sigma * kTreeQuads * 4 + e] = (d[0] + 8) | ((d[1] + 8) << 5) | ((d[2] + 8) << 10);
    }
  hipError_t e;
  int* d_sidx = nullptr;
  if ((e = hipMalloc(&tt->doff, sizeof(int) * doff.size())) != hipSuccess) return e;
  if ((e = hipMemcpy(tt->doff, doff.data(), sizeof(int) * doff.size(), hipMemcpyHostToDevice)) != hipSuccess) return e;
  if ((e = hipMalloc(&d_sidx, sizeof(int) * sidx.size())) != hipSuccess) return e;
  if ((e = hipMemcpy(d_sidx, sidx.data(), sizeof(int) * sidx.size(), hipMemcpyHostToDevice)) != hipSuccess) {
    (void)hipFree(d_sidx);
    return e;
  }
  for (int p = 2; p <= kMaxP; ++p) {
    const int C = ncomp(p), NG = (C + 3) / 4, R = (C + 1) / 2;
    const size_t count = (size_t)8 * R * kTreeQuads * 2 * NG * 16;
    if ((e = hipMalloc(&tt->B[p], sizeof(double) * (count + kTreePad))) != hipSuccess) break;
    hipLaunchKernelGGL(pack_tree_kernel, dim3(1024), dim3(256), 0, s, d_T[p], C, d_sidx, tt->B[p]);
    if ((e = hipGetLastError()) != hipSuccess) break;
    TreeHMaps mp;
    int rh = 0;
    if (!harmonic_plan_maps(p, mp.rowk, mp.colk, &rh) || rh != ((p + 1) * (p + 1) + 1) / 2) {
      e = hipErrorInvalidValue;
      break;
    }
    const int CRh = (p + 1) * (p + 1), NGh = (CRh + 3) / 4;
    const size_t counth = (size_t)8 * rh * kTreeQuads * 2 * NGh * 16;
    if ((e = hipMalloc(&tt->Bh[p], sizeof(double) * (counth + kTreePad))) != hipSuccess) break;
    hipLaunchKernelGGL(pack_tree_h_kernel, dim3(1024), dim3(256), 0, s, d_T[p], C, rh, NGh, d_sidx, mp,
                       tt->Bh[p]);
    if ((e = hipGetLastError()) != hipSuccess) break;
  }
  hipError_t e2 = hipStreamSynchronize(s);
  (void)hipFree(d_sidx);
  return e != hipSuccess ? e : e2;
}

void tree_tables_destroy(TreeTables* tt) {
  for (int p = 0; p <= kMaxP; ++p) {
    if (tt->B[p]) (void)hipFree(tt->B[p]);
    if (tt->Bh[p]) (void)hipFree(tt->Bh[p]);
  }
  if (tt->doff) (void)hipFree(tt->doff);
  *tt = TreeTables{};
}

hipError_t launch_tree_p2m(int p, const double* pos, const double* mass, int ppc, int n, double h,
                           double* M, hipStream_t s) {
  const int64_t n3 = (int64_t)n * n * n;
  const dim3 grid(blocks_for(n3, 256)), block(256);
  switch (p) {
    case 2: hipLaunchKernelGGL(p2m_grid_kernel<2>, grid, block, 0, s, pos, mass, ppc, n, h, M); break;
    case 3: hipLaunchKernelGGL(p2m_grid_kernel<3>, grid, block, 0, s, pos, mass, ppc, n, h, M); break;
    case 4: hipLaunchKernelGGL(p2m_grid_kernel<4>, grid, block, 0, s, pos, mass, ppc, n, h, M); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_tree_m2m(int p, const double* Mc, double* Mp, int nc, double hc, hipStream_t s) {
  const int64_t np3 = (int64_t)(nc / 2) * (nc / 2) * (nc / 2);
  const dim3 grid(blocks_for(np3, 32)), block(256);
  switch (p) {
    case 2: hipLaunchKernelGGL(m2m_kernel<2>, grid, block, 0, s, Mc, Mp, nc, hc); break;
    case 3: hipLaunchKernelGGL(m2m_kernel<3>, grid, block, 0, s, Mc, Mp, nc, hc); break;
    case 4: hipLaunchKernelGGL(m2m_kernel<4>, grid, block, 0, s, Mc, Mp, nc, hc); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_tree_l2l(int p, const double* Lp, double* Lc, int nc, double hc, hipStream_t s) {
  const int64_t nc3 = (int64_t)nc * nc * nc;
  const dim3 grid(blocks_for(nc3, 256)), block(256);
  switch (p) {
    case 2: hipLaunchKernelGGL(l2l_kernel<2>, grid, block, 0, s, Lp, Lc, nc, hc); break;
    case 3: hipLaunchKernelGGL(l2l_kernel<3>, grid, block, 0, s, Lp, Lc, nc, hc); break;
    case 4: hipLaunchKernelGGL(l2l_kernel<4>, grid, block, 0, s, Lp, Lc, nc, hc); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_tree_m2l(int p, const TreeTables& tt, const MfmaTables& mt, bool harmonic,
                           const double* M, double* L, int nlev, const int* n, const int* lg,
                           const int64_t* off, hipStream_t s) {
  if (nlev < 1 || nlev > kTreeMaxLevels) return hipErrorInvalidValue;
  // Wide workgroups where a level has at least one for every CU (64^3: 256), planes
  // on the coarser levels. Planes everywhere, harmonic p = 3: 64^3 936 us against
  // 707, 128^3 6542 against 4592 (11 planes staged for one); wide everywhere would
  // leave most of the CUs without work below 64^3.
  for (int pass = 0; pass < 2; ++pass) {
    const bool wide = pass == 0;
    TreeLevels lv{};
    int total = 0, cnt = 0;
    for (int i = 0; i < nlev; ++i) {            // coarsest level first
      const int l = nlev - 1 - i;
      if ((n[l] >= kTreeWideMin) != wide) continue;
      const int nb = n[l] >= 8 ? n[l] / 8 : 1;
      lv.first[cnt] = total;
      lv.n[cnt] = n[l];
      lv.lg[cnt] = lg[l];
      lv.off[cnt] = off[l];
      total += wide ? nb / 2 * nb * nb : nb * nb * nb * (n[l] < 8 ? n[l] : 8);
      ++cnt;
    }
    if (cnt == 0) continue;
    lv.nlev = cnt;
    lv.first[cnt] = total;
#define TREE_LAUNCH(P, H, W)                                                                         \
  hipLaunchKernelGGL((m2l_level_kernel<P, H, W>), dim3((unsigned)total), dim3(TreeShape<W>::NT), 0, s, \
                     M, L, lv, H ? tt.Bh[P] : tt.B[P], tt.doff, mt.hround[P], mt.hexp[P])
    switch ((p * 2 + (harmonic ? 1 : 0)) * 2 + pass) {
      case 8: TREE_LAUNCH(2, false, true); break;
      case 9: TREE_LAUNCH(2, false, false); break;
      case 10: TREE_LAUNCH(2, true, true); break;
      case 11: TREE_LAUNCH(2, true, false); break;
      case 12: TREE_LAUNCH(3, false, true); break;
      case 13: TREE_LAUNCH(3, false, false); break;
      case 14: TREE_LAUNCH(3, true, true); break;
      case 15: TREE_LAUNCH(3, true, false); break;
      case 16: TREE_LAUNCH(4, false, true); break;
      case 17: TREE_LAUNCH(4, false, false); break;
      case 18: TREE_LAUNCH(4, true, true); break;
      case 19: TREE_LAUNCH(4, true, false); break;
      default: return hipErrorInvalidValue;
    }
#undef TREE_LAUNCH
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace fmm
