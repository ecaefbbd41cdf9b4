// Matrix-core M2L on gfx950: v_mfma_f64_16x16x4 and v_mfma_f64_4x4x4_4b (four
// independent 4x4x4 products per instruction), workgroups over a longest-first list
// of sub-grids or of parts of them.
//
// Forward (every target's whole sum belongs to one work item):
//   L[t][n] = h^(-1-|n|) sum_d sum_k [h^-|k| M_k(t + d)] T_d[k][n]
// is a sum over (d, k) of rank-1 updates of the [512 x C] output. The
// reduction is taken four stencil offsets at a time for one moment
// component: one instruction multiplies a [16 cells x 4 offsets] slice of the
// shifted source window (A) by [4 offsets x 16 (or 4) columns] of the tables (B).
// The columns past the last sixteen go in groups of four, so no column padding is
// computed at p = 3.
//
// Data movement: the window of two moment components at a time ("round") that the
// item's targets reach is staged in LDS as double2 (128,000 bytes for a whole
// sub-grid), zero on absent blocks and pre-scaled by h^-|k| (exact powers of two);
// every cell of it is then reused by all 892 offsets. Table operands stream from L2
// (the packed tables are laid out in consumption order). The only HBM traffic is the
// window and L.
//
// Operand lane layouts of v_mfma_f64_4x4x4_4b (checked on gfx950; 16x16x4 takes the
// same A, its D layout is with the streamed forward below):
//   A: lane l -> block (l%16)/4, row l%4, k l/16   (so: cell l%16 of a 16-cell tile)
//   B: lane l -> block (l%16)/4, col l%4, k l/16
//   D: lane l -> block (l%16)/4, col l%4, row l/16 (so: cell 4*((l%16)/4) + l/16)
#include <algorithm>
#include <functional>
#include <type_traits>

#include "kernels.h"
#include "m2l_mfma.h"
#include "p2m_common.h"
#include "stencil_pairs.h"

namespace fmm {

namespace {

constexpr int kWinCells = kWin * kWin * kWin;   // 8000

// Rows of the forward's compact window (see the streamed forward below): plane w
// of the window of nz target planes holds the rows within window_reach of the block.
__host__ __device__ constexpr int shell_reach(int dz) {
  int r = 0;
  while ((r + 1) * (r + 1) + dz * dz <= 36) ++r;
  return r;
}
__host__ __device__ constexpr int window_reach(int nz, int w) {
  int r = 0;
  for (int t = 0; t < nz; ++t) {
    const int dz = w - 6 - t;
    if (dz >= -6 && dz <= 6 && shell_reach(dz) > r) r = shell_reach(dz);
  }
  return r;
}
// rows of a window whose targets span `span` rows per plane (8, or 4 for one tile)
__host__ __device__ constexpr int window_rows(int nz, int span) {
  int n = 0;
  for (int w = 0; w < nz + 12; ++w) n += span + 2 * window_reach(nz, w);
  return n;
}
constexpr int kWinRows8 = window_rows(8, 8), kWinRows2 = window_rows(2, 8), kWinRows1 = window_rows(1, 8),
              kWinRowsTile = window_rows(1, 4);
static_assert(kWinRows8 == 344 && kWinRows2 == 224 && kWinRows1 == 204 && kWinRowsTile == 152, "window rows");
// LDS cell of window coordinate (0, 0) of plane w: the plane's first stored row is 6 - reach
__host__ __device__ constexpr int window_base(int nz, int w) {
  int n = 0;
  for (int v = 0; v < w; ++v) n += 8 + 2 * window_reach(nz, v);
  return kWin * (n - 6 + window_reach(nz, w));
}

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

typedef double v4d __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4d mfma16(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__global__ void reset_counter_kernel(unsigned* counter) { *counter = 0u; }

// ---------------------------------------------------------------------------
// forward, table operands loaded per wave (FMM_FP64 configurations 2 to 5)
// ---------------------------------------------------------------------------

template <int P, int WAVES, bool PF>
__device__ __forceinline__ void fwd_subgrid(const DevDesc& d, const double* __restrict__ M,
                                            double* __restrict__ L, const double* __restrict__ Bp,
                                            const int* __restrict__ lds_off,
                                            const uint32_t* __restrict__ touch, double2* smem) {
  constexpr int C = ncomp(P);
  constexpr int NG = (C + 3) / 4;        // output column groups of 4
  constexpr int ROUNDS = (C + 1) / 2;    // moment components staged two at a time
  constexpr int TPW = 32 / WAVES;        // 16-cell tiles per wave
  constexpr int NT = WAVES * 64;
  const int tid = threadIdx.x, lane = tid & 63;
  // wave index as a scalar: keeps the per-quad table lookups on the scalar unit
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kk = lane >> 4;              // offset of the quad this lane feeds
  const int ci = lane & 15;              // cell of the tile this lane feeds

  // tile gt = wave*TPW + t: target plane gt/4, 4x4 patch ((gt&1)*4, ((gt>>1)&1)*4)
  int abase[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int gt = wave * TPW + t;
    const int z = gt >> 2, x = (gt & 1) * 4 + (ci & 3), y = ((gt >> 1) & 1) * 4 + (ci >> 2);
    // window coordinates of the target cell: frame (x+8, y+8, z+8) minus 2
    abase[t] = (x + 6) + kWin * (y + 6) + kWin * kWin * (z + 6);
  }
  const int zlo = (wave * TPW) >> 2, zhi = (wave * TPW + TPW - 1) >> 2;

  double acc[TPW][NG];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int g = 0; g < NG; ++g) acc[t][g] = 0.0;

  const int l2 = d.log2_inv_h;
  const double* src = M + d.m_off;
  for (int r = 0; r < ROUNDS; ++r) {
    const int k0 = 2 * r, k1 = 2 * r + 1;
    const double s0 = ldexp(1.0, l2 * order_of(k0));
    const double s1 = k1 < C ? ldexp(1.0, l2 * order_of(k1)) : 0.0;
    const double* src0 = src + (size_t)k0 * kNCell;
    const double* src1 = src + (size_t)(k1 < C ? k1 : k0) * kNCell;
    // issue every load of this thread's share of the window before any LDS store,
    // so the HBM latency is paid once per round rather than once per cell
    constexpr int kStage = (kWinCells + NT - 1) / NT;
    double2 v[kStage];
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
      const int c = tid + i * NT;
      v[i] = make_double2(0.0, 0.0);
      if (c < kWinCells) {
        const int wx = c % kWin, wy = (c / kWin) % kWin, wz = c / (kWin * kWin);
        const int jx = wx + kWin0, jy = wy + kWin0, jz = wz + kWin0;
        const int cell = jx + kFrame * jy + kFrame * kFrame * jz;
        if (block_present(d.mask, jx, jy, jz)) {
          v[i].x = src0[cell];
          v[i].y = src1[cell];
        }
      }
    }
    __syncthreads();   // previous round's reads of smem are done
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
      const int c = tid + i * NT;
      if (c < kWinCells) smem[c] = make_double2(v[i].x * s0, v[i].y * s1);
    }
    __syncthreads();
    const double* Br = Bp + (size_t)r * kQuads * 2 * NG * 16 + kk * 4 + (lane & 3);
    // table operands of the next quad are loaded while this quad's products run
    double nb0[NG], nb1[NG];
    if (PF) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        nb0[g] = Br[g * 16];
        nb1[g] = Br[(NG + g) * 16];
      }
    }
    // per-quad scalars (blocks touched, LDS offsets) are fetched one quad ahead
    const int4* off4 = reinterpret_cast<const int4*>(lds_off);
    uint32_t tm_next = 0;
    for (int z = zlo; z <= zhi; ++z) tm_next |= touch[z * kQuads];
    int4 o_next = off4[0];
    for (int q = 0; q < kQuads; ++q) {
      const uint32_t tm = tm_next;
      const int4 o = o_next;
      if (q + 1 < kQuads) {
        tm_next = 0;
        for (int z = zlo; z <= zhi; ++z) tm_next |= touch[z * kQuads + q + 1];
        o_next = off4[q + 1];
      }
      double b0[NG], b1[NG];
      if (PF) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          b0[g] = nb0[g];
          b1[g] = nb1[g];
        }
        if (q + 1 < kQuads) {
          const double* Bn = Br + (size_t)(q + 1) * 2 * NG * 16;
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            nb0[g] = Bn[g * 16];
            nb1[g] = Bn[(NG + g) * 16];
          }
        }
      }
      if ((tm & d.mask) == 0) continue;   // every source of this quad is absent for this wave
      // each lane takes the offset of its k-slot (branch-free select of scalars)
      int doff = o.x;
      doff = kk == 1 ? o.y : doff;
      doff = kk == 2 ? o.z : doff;
      doff = kk == 3 ? o.w : doff;
      if (!PF) {
        const double* Bq = Br + (size_t)q * 2 * NG * 16;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          b0[g] = Bq[g * 16];
          b1[g] = Bq[(NG + g) * 16];
        }
      }
      double2 a[TPW];
#pragma unroll
      for (int t = 0; t < TPW; ++t) a[t] = smem[abase[t] + doff];
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[t][g] = mfma4(a[t].x, b0[g], acc[t][g]);
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[t][g] = mfma4(a[t].y, b1[g], acc[t][g]);
      }
    }
  }

  // D layout: this lane holds cell (x = lane/16, y = (lane%16)/4) of each tile, column lane%4
  double* out = L + d.l_off;
  const int xi = lane >> 4, yi = (lane & 15) >> 2, j = lane & 3;
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int gt = wave * TPW + t;
    const int z = gt >> 2, x = (gt & 1) * 4 + xi, y = ((gt >> 1) & 1) * 4 + yi;
    const int tcell = x + kBlock * y + kBlock * kBlock * z;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int n = 4 * g + j;
      if (n < C) out[(size_t)n * kNTarget + tcell] = ldexp(acc[t][g], l2 * (1 + order_of(n)));
    }
  }
}

template <int WAVES, bool PF>
__global__ void __launch_bounds__(WAVES * 64) m2l_fwd_kernel(
    const WorkItem* __restrict__ items, int count, unsigned* __restrict__ counter,
    const DevDesc* __restrict__ desc, const double* __restrict__ M, double* __restrict__ L,
    const double* __restrict__ B2, const double* __restrict__ B3, const double* __restrict__ B4,
    const int* __restrict__ lds_off, const uint32_t* __restrict__ touch) {
  __shared__ double2 smem[kWinCells];
  __shared__ int s_item;
  for (;;) {
    if (threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
    __syncthreads();
    const int item = s_item;
    if (item >= count) break;
    const DevDesc d = desc[items[item].sub];
    switch (d.p) {
      case 2: fwd_subgrid<2, WAVES, PF && (2 < 4 || WAVES == 4)>(d, M, L, B2, lds_off, touch, smem); break;
      case 3: fwd_subgrid<3, WAVES, PF && (3 < 4 || WAVES == 4)>(d, M, L, B3, lds_off, touch, smem); break;
      case 4: fwd_subgrid<4, WAVES, PF && (4 < 4 || WAVES == 4)>(d, M, L, B4, lds_off, touch, smem); break;
      default: break;
    }
    __syncthreads();   // s_item and smem are free for the next item
  }
}

// ---------------------------------------------------------------------------
// forward, table operands streamed from L2
// ---------------------------------------------------------------------------
//
// A workgroup takes a whole sub-grid's targets or a part of them, with the window
// of two components (a round) that they reach in LDS. Each target's sums run over
// the rounds, quads and components in one order whatever the part, so the results
// are the same bits.
//
//   level   targets   of one sub-grid   threads   a wave's share
//   kWhole  8 planes         1            512     4 tiles, all columns
//     0     2 planes         4            256     2 tiles, all columns
//     1     1 plane          8            256     1 tile, all columns
//     2     1 tile          32            256     1 tile, every fourth group of 4 columns
//
// Parts spread a few sub-grids over the GPU (one sub-grid's M2L 920 -> 80 us, 43
// mixed ones 2590 -> 575) and even out the end of a middling batch (300 sub-grids
// 2000 -> 1230 us, where whole ones take two waves); two workgroups share a
// compute unit, but their staging still costs (a window of 14 planes for 2 target
// planes, and one workgroup's loads in flight hold up the other's table
// operands), so large batches go in whole sub-grids (2000 at p = 3, harmonic: 7.29
// ms, in parts 7.53, and 7.69 with the four-block instruction and tables staged
// through LDS; 4096: 14.6 ms, 65.6 TFLOP/s executed). plan_stream and split_items
// choose.
//
// Columns. Sixteen output columns at a time go through v_mfma_f64_16x16x4
// ([16 cells x 4 offsets] x [4 offsets x 16 columns]), which sums the offsets in
// the order the four-block instruction does (both are chains of fused
// multiply-adds over k, so their results are the same bits), takes the same A
// operand, needs a quarter of the B operand reads (no value is replicated over
// blocks) and runs at full rate without independent accumulators: 69 and 77
// TFLOP/s with one accumulator and one or two waves per SIMD, where the
// four-block one reaches 28 and 56. Columns past the last sixteen go four at a
// time through the four-block instruction, so nothing more is padded than there.
//   D of 16x16x4: lane l, element v -> cell 4 v + l/16 of the tile, column l%16
// At level 2, which has waves to spare, the shorter latency of the four-block
// instruction (18 ns against 30) counts.
//
// Operands. A wave reads its tiles' window cells AD quads ahead of their
// products. Table operands come from L2 straight into registers, U quads ahead,
// so the quad loop has no barrier and no wave waits for another one.
//
// Window. At distance dz of a target plane only the cells within
// reach(dz) = floor(sqrt(36 - dz^2)) of the block in x and y are used, so the
// window of a part holds, per plane, the rows within that reach in y (all 20
// cells of each): 224 rows for two target planes (71,680 bytes, two of which fit
// a compute unit) and 204 for one, instead of 280 and 260. A whole sub-grid's
// keeps full planes, with 344 of their 400 rows staged.
//
// Tried: the next round's window loaded into registers during the products, or
// its cache lines touched: both slower, as vector loads return in order and the
// table operands behind them wait for the window's latency. Operand sets 2 and 3
// quads ahead at level 0, and table operands 4 or 16 quads ahead: within 2%.
constexpr int kPartThreads = 256;
constexpr int kWholeThreads = 512;

template <int P, bool HARM>
struct FwdCols {
  static constexpr int CR = HARM ? (P + 1) * (P + 1) : ncomp(P);   // reduced components
  static constexpr int NG = (CR + 3) / 4;                          // columns in groups of four
  static constexpr int N16 = CR / 16, N4 = NG - 4 * N16;
};
constexpr int kWhole = -1;   // the level of a whole sub-grid
template <int LEVEL>
struct PartShape {
  static constexpr int NT = LEVEL == kWhole ? kWholeThreads : kPartThreads, WAVES = NT / 64;
  static constexpr int NZ = LEVEL == kWhole ? 8 : LEVEL == 0 ? 2 : 1;   // target planes of the window
  static constexpr int TPW = LEVEL == kWhole ? 4 : LEVEL == 0 ? 2 : 1;  // tiles per wave
  static constexpr int CS = LEVEL == 2 ? WAVES : 1;         // waves sharing a tile's columns
  static constexpr int TILES = LEVEL == 2 ? 1 : 4 * NZ;
  // LDS rows of the window, and the rows staged
  static constexpr int ROWS = NZ == 8 ? kWin * kWin : NZ == 2 ? kWinRows2 : kWinRows1;
  static constexpr int STAGED = LEVEL == kWhole ? kWinRows8 : LEVEL == 2 ? kWinRowsTile : ROWS;
  static constexpr int FIRST = LEVEL == kWhole ? kWinRows2 + kWinRows1 + 2 * kWinRowsTile   // in the row table
                               : LEVEL == 0 ? 0 : LEVEL == 1 ? kWinRows2 : kWinRows2 + kWinRows1;
  static constexpr int AD = LEVEL <= 0 ? 1 : 3;
};
// A wave's columns: N16 sixteens, then N4 groups of four, every S4-th.
template <int N16_, int N4_, int S4_>
struct Cols {
  static constexpr int N16 = N16_, N4 = N4_, S4 = S4_;
};
constexpr int kOffPad = 20;   // s_off entries past the last quad: offsets are read ahead
// room past the tables for the quads read ahead in the last round (at most 16 of
// 9 column groups; never multiplied)
constexpr size_t kTablePad = 16 * 9 * 32;

// The cells of a part's window that one thread stages, fixed over the rounds:
// frame cell | LDS cell << 16. An absent cell loads the (always present) centre
// cell and stores zero. rowtab: the window's rows, y | plane << 8 | LDS row << 16.
template <int COUNT, int NT>
struct WindowCells {
  int at[COUNT];
  uint32_t on;
  __device__ __forceinline__ void set(const DevDesc& d, const int* __restrict__ rowtab, int rows, int z0) {
    constexpr int kCentre = kBlock * (1 + kFrame + kFrame * kFrame);
    on = 0;
#pragma unroll
    for (int i = 0; i < COUNT; ++i) {
      const int c = (int)threadIdx.x + i * NT;
      const int x = c % kWin, v = rowtab[min(c / kWin, rows - 1)];
      const int jx = x + kWin0, jy = (v & 255) + kWin0, jz = ((v >> 8) & 255) + kWin0 + z0;
      const bool in = block_present(d.mask, jx, jy, jz);
      at[i] = (in ? jx + kFrame * jy + kFrame * kFrame * jz : kCentre) | ((v >> 16) * kWin + x) << 16;
      on |= (uint32_t)in << i;
    }
  }
  __device__ __forceinline__ int cell(int i) const { return at[i] & 0xffff; }
  __device__ __forceinline__ int lds(int i) const { return at[i] >> 16; }
};
static_assert(kWin * kWin * kWin < 1 << 15 && kNCell < 1 << 16, "packed cells");

// a window cell: the two components, or their float32 parts hi, lo, hi, lo
__device__ __forceinline__ void put_cell(double2& w, double a0, double a1) { w = make_double2(a0, a1); }
__device__ __forceinline__ void put_cell(float4& w, double a0, double a1) {
  const float h0 = (float)a0, h1 = (float)a1;
  w = make_float4(h0, (float)(a0 - (double)h0), h1, (float)(a1 - (double)h1));
}

// Round r's two components of the part's window cells, scaled, into LDS; in the
// harmonic form each of the two is a combination of the round's moment
// components. All loads of a pass are in flight together. Barriers: one before
// the first store; the caller's follows.
template <int P, bool HARM, int ROWS, int COUNT, int NT, class Cell>
__device__ __forceinline__ void stage_window(const WindowCells<COUNT, NT>& wc, int l2, const double* __restrict__ src,
                                             const HRound* __restrict__ hround, int r, Cell* win) {
  constexpr int C = ncomp(P);
  constexpr int SUP = HARM ? harmonic_sup(P) : 2;        // components read per round, at most
  constexpr int kPasses = SUP * COUNT > 60 ? 2 : 1;      // (registers)
  constexpr int kPer = (COUNT + kPasses - 1) / kPasses;
#pragma unroll
  for (int pass = 0; pass < kPasses; ++pass) {
    double x[SUP][kPer];
    double2 v[kPer];
    double s0, s1;
#pragma unroll
    for (int u = 0; u < SUP; ++u) {
      int comp;
      if constexpr (HARM) comp = hround[r].comp[min(u, hround[r].nsup - 1)];
      else comp = min(2 * r + u, C - 1);
      const double* su = src + (size_t)comp * kNCell;
#pragma unroll
      for (int i = 0; i < kPer; ++i)
        if (pass * kPer + i < COUNT) x[u][i] = su[wc.cell(pass * kPer + i)];
    }
    if constexpr (HARM) {
      const HRound& rd = hround[r];
      s0 = ldexp(1.0, l2 * rd.ord0);
      s1 = rd.ord1 >= 0 ? ldexp(1.0, l2 * rd.ord1) : 0.0;
#pragma unroll
      for (int i = 0; i < kPer; ++i) v[i] = make_double2(0.0, 0.0);
#pragma unroll
      for (int u = 0; u < SUP; ++u) {
        if (u < rd.nsup) {
          const double f0 = rd.c0[u], f1 = rd.c1[u];
#pragma unroll
          for (int i = 0; i < kPer; ++i) {
            if (pass * kPer + i >= COUNT) continue;
            v[i].x = __builtin_fma(f0, x[u][i], v[i].x);
            v[i].y = __builtin_fma(f1, x[u][i], v[i].y);
          }
        }
      }
    } else {
      s0 = ldexp(1.0, l2 * order_of(2 * r));
      s1 = 2 * r + 1 < C ? ldexp(1.0, l2 * order_of(2 * r + 1)) : 0.0;
#pragma unroll
      for (int i = 0; i < kPer; ++i)
        if (pass * kPer + i < COUNT) v[i] = make_double2(x[0][i], x[1][i]);
    }
    if (pass == 0) __syncthreads();   // the previous round's window reads are done
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int k = pass * kPer + i;
      const bool in = (wc.on >> k) & 1u;
      if (k < COUNT && (int)threadIdx.x + k * NT < ROWS * kWin)
        put_cell(win[wc.lds(k)], in ? v[i].x * s0 : 0.0, in ? v[i].y * s1 : 0.0);
    }
  }
}

// Hook (whole sub-grids): at the top of round r, hook.run() is called if
// hook.wants(r, ROUNDS) (uniform over the workgroup); it starts with a barrier,
// may use the window buffer and must leave no LDS access in flight. Around it
// the sums so far are parked in the sub-grid's own L slots (written only at the
// end), so run() has the registers.
struct NoMoments {
  __device__ bool wants(int, int) const { return false; }
  __device__ void run() const {}
};
// the moments of the next item, at the top of round (workgroup index mod rounds)
template <class F>
struct MomentHook {
  int next, count;
  F moments;
  __device__ bool wants(int r, int rounds) const {
    return next < count && r == (int)(blockIdx.x % (unsigned)rounds);
  }
  __device__ void run() const { moments(next); }
};

// FULL: every neighbour block is present, so no quad is skipped.
// s_off: the quads' LDS offsets; of a part, for either plane of level 0, then for
// the one plane of the other levels.
template <int P, bool HARM, bool FULL, int LEVEL, class Hook = NoMoments>
__device__ __forceinline__ void fwd_part(const DevDesc& d, const double* __restrict__ M, double* __restrict__ L,
                                         const double* __restrict__ Bl, const uint32_t* __restrict__ ttouch,
                                         const int* __restrict__ rowtab, double2* win, const short4 (*s_off)[kQuads + kOffPad],
                                         const HRound* __restrict__ hround, const HExp* __restrict__ hexp, int part,
                                         Hook hook = Hook()) {
  using S = PartShape<LEVEL>;
  using F = FwdCols<P, HARM>;
  constexpr int C = ncomp(P), CR = F::CR, NG = F::NG;
  constexpr int ROUNDS = (CR + 1) / 2;
  constexpr int TPW = S::TPW, CS = S::CS, AD = S::AD;
  constexpr int AR = AD == 1 ? 2 : 4;                  // window operand sets
  // quads of table operands in flight: 64 registers of them in a part, up to 48
  // beside the tiles of a whole sub-grid, whose quads take longer
  constexpr int kUnits = CS == 1 ? F::N16 + F::N4 : (NG + CS - 1) / CS;
  constexpr int U = LEVEL == kWhole ? (kUnits > 3 ? 2 : 4) : kUnits == 1 ? 16 : kUnits == 2 ? 8 : 4;
  static_assert(U % AR == 0 && U + AD <= kOffPad && U * NG * 32 <= (int)kTablePad, "read ahead");
  // this wave's columns: all, or groups of four wave, wave + 4, ... (Most of them, or one fewer)
  using Most = std::conditional_t<CS == 1, Cols<F::N16, F::N4, 1>, Cols<0, (NG + CS - 1) / CS, CS>>;
  using Less = Cols<0, Most::N4 - (CS > 1), CS>;
  constexpr int M16 = Most::N16, M4 = Most::N4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kk = lane >> 4, ci = lane & 15;
  const int f4 = CS == 1 ? 4 * F::N16 : wave;          // this wave's first group of four
  // first tile of the wave (4 plane + 2 y + x in the 2 x 2 tiles of a plane)
  const int tile0 = part * S::TILES + (CS == 1 ? wave * TPW : 0);
  const int plane = tile0 >> 2, z0 = (part * S::TILES) >> 2;
  auto tile_x = [&](int t) { return (TPW == 1 ? tile0 & 1 : t & 1) * 4; };
  const int ty = ((tile0 >> 1) & 1) * 4;
  auto tile_y = [&](int t) { return TPW == 4 ? (t >> 1) * 4 : ty; };
  int abase[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
    abase[t] = (tile_x(t) + (ci & 3) + 6) + kWin * (tile_y(t) + (ci >> 2) + 6) +
               (LEVEL == kWhole ? kWin * kWin * (plane + 6) : 0);
  v4d acc16[TPW][M16 > 0 ? M16 : 1];
  double acc4[TPW][M4 > 0 ? M4 : 1];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
#pragma unroll
    for (int g = 0; g < M16; ++g) acc16[t][g] = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int g = 0; g < M4; ++g) acc4[t][g] = 0.0;
  }
  auto columns = [&](auto f) __attribute__((always_inline)) {
    if (CS == 1 || wave < NG - (M4 - 1) * CS) f(Most{});
    else if constexpr (CS > 1 && Less::N4 > 0) f(Less{});
  };
  // sum = f(column, target of the sub-grid, sum) over this wave's sums
  auto each_sum = [&](auto f) __attribute__((always_inline)) {
    const int xi = lane >> 4, yi = (lane & 15) >> 2, j = lane & 3;
    columns([&](auto cols) __attribute__((always_inline)) {
      using K = decltype(cols);
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const int t0 = tile_x(t) + xi + kBlock * tile_y(t) + kBlock * kBlock * plane;
#pragma unroll
        for (int g = 0; g < K::N16; ++g)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc16[t][g][v] = f(16 * g + ci, t0 + kBlock * v, acc16[t][g][v]);
#pragma unroll
        for (int g = 0; g < K::N4; ++g) acc4[t][g] = f(4 * (f4 + g * K::S4) + j, t0 + kBlock * yi, acc4[t][g]);
      }
    });
  };
  const int l2 = d.log2_inv_h;
  const double* src = M + d.m_off;
  const short* so = reinterpret_cast<const short*>(s_off[LEVEL == kWhole ? 0 : LEVEL == 0 ? plane - z0 : 2]) + kk;
  // per tile: the quads with a present source, one bit each; lane 4 t + i holds word i of tile t
  uint64_t live = 0;
  if constexpr (!FULL) {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = 64 * i + lane;
        const uint64_t w = __ballot(q < kQuads && (ttouch[(tile0 + t) * kQuads + min(q, kQuads - 1)] & d.mask) != 0);
        live = lane == 4 * t + i ? w : live;
      }
  }
  WindowCells<(S::STAGED * kWin + S::NT - 1) / S::NT, S::NT> wc;
  wc.set(d, rowtab + S::FIRST + (LEVEL == 2 && ty ? kWinRowsTile : 0), S::STAGED, z0);
  // tables through a buffer resource: a per-quad scalar offset and fixed lane
  // offsets (quads read ahead in the last round fall in the tables' padding)
  const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<double*>(Bl), (short)0, ROUNDS * kQuads * NG * 256 + (int)kTablePad * 8, 0x00020000);
  const int vb16 = ((ci >> 2) * 16 + kk * 4 + (lane & 3)) * 16;      // column ci of a sixteen
  const int vb4 = (f4 * 16 + kk * 4 + (lane & 3)) * 16;
  for (int r = 0; r < ROUNDS; ++r) {
    if (hook.wants(r, ROUNDS)) {
      double* park = L + d.l_off;
      each_sum([&](int n, int target, double a) __attribute__((always_inline)) {
        if (n < CR) park[(size_t)n * kNTarget + target] = a;
        return a;
      });
      asm volatile("" ::: "memory");   // the sums are reloaded, not kept in registers
      hook.run();
      asm volatile("" ::: "memory");
      each_sum([&](int n, int target, double) __attribute__((always_inline)) {
        return n < CR ? park[(size_t)n * kNTarget + target] : 0.0;
      });
    }
    stage_window<P, HARM, S::STAGED>(wc, l2, src, hround, r, win);
    __syncthreads();
    columns([&](auto cols) __attribute__((always_inline)) {
      using K = decltype(cols);
      constexpr int KN16 = K::N16 > 0 ? K::N16 : 1, KN4 = K::N4 > 0 ? K::N4 : 1;
      int sq = r * kQuads * NG * 256;                  // table offset of the quad group
      const short* sp = so;                            // and its LDS offsets
      double2 b16[U][KN16], b4[U][KN4], a[AR][TPW];
      int o[U];
#define PT_LOADB(SET, Q)                                                                           \
  {                                                                                                \
    _Pragma("unroll") for (int g = 0; g < K::N16; ++g) b16[SET][g] = __builtin_bit_cast(double2,   \
        __builtin_amdgcn_raw_buffer_load_b128(brs, vb16 + 4 * g * 256, sq + (Q) * NG * 256, 0));   \
    _Pragma("unroll") for (int g = 0; g < K::N4; ++g) b4[SET][g] = __builtin_bit_cast(double2,     \
        __builtin_amdgcn_raw_buffer_load_b128(brs, vb4 + g * K::S4 * 256, sq + (Q) * NG * 256, 0)); \
  }
#define PT_LOADA(SET, OSET) \
  _Pragma("unroll") for (int t = 0; t < TPW; ++t) a[SET][t] = win[abase[t] + o[OSET]];
#define PT_MMA1(u, t, X)                                                                           \
  {                                                                                                \
    _Pragma("unroll") for (int g = 0; g < K::N16; ++g) acc16[t][g] = mfma16(a[(u) % AR][t].X, b16[u][g].X, acc16[t][g]); \
    _Pragma("unroll") for (int g = 0; g < K::N4; ++g) acc4[t][g] = mfma4(a[(u) % AR][t].X, b4[u][g].X, acc4[t][g]); \
  }
// one quad: window operands AD quads ahead, then the offset that operand set
// needs next; the products (each tile on its own where blocks are absent); the
// table operands of quad u + U. The fences keep the reads in issue order and out
// of the conditional blocks: then every wait covers the oldest reads only.
#define PT_STEP(u, MORE)                                                                           \
  {                                                                                                \
    __builtin_amdgcn_sched_barrier(0);                                                             \
    PT_LOADA(((u) + AD) % AR, ((u) + AD) % U);                                                     \
    o[((u) + AD) % U] = sp[((u) + AD + U) * 4];                                                    \
    if constexpr (FULL) {                                                                          \
      _Pragma("unroll") for (int t = 0; t < TPW; ++t) PT_MMA1(u, t, x);                            \
      _Pragma("unroll") for (int t = 0; t < TPW; ++t) PT_MMA1(u, t, y);                            \
    } else {                                                                                       \
      asm volatile("" ::: "memory");                                                               \
      _Pragma("unroll") for (int t = 0; t < TPW; ++t) if ((uint32_t)lw[t][0] >> (u) & 1u) {        \
        PT_MMA1(u, t, x);                                                                          \
        PT_MMA1(u, t, y);                                                                          \
      }                                                                                            \
      asm volatile("" ::: "memory");                                                               \
    }                                                                                              \
    if (MORE) PT_LOADB(u, u + U);                                                                  \
    __builtin_amdgcn_sched_barrier(0);                                                             \
  }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        PT_LOADB(u, u);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) o[u] = sp[u * 4];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < AD; ++u) {
        PT_LOADA(u, u);
        o[u] = sp[(u + U) * 4];
        __builtin_amdgcn_sched_barrier(0);
      }
      uint64_t lw[TPW][4];                             // live quads from the loop's first quad on
      if constexpr (!FULL) {
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            lw[t][i] = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)live, 4 * t + i) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(live >> 32), 4 * t + i) << 32;
      }
#pragma unroll 1
      for (int q = 0; q < kQuads / U * U; q += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) PT_STEP(u, true);
        if constexpr (!FULL) {
#pragma unroll
          for (int t = 0; t < TPW; ++t) {
#pragma unroll
            for (int i = 0; i < 3; ++i) lw[t][i] = lw[t][i] >> U | lw[t][i + 1] << (64 - U);
            lw[t][3] >>= U;
          }
        }
        sq += U * NG * 256;
        sp += U * 4;
      }
#pragma unroll
      for (int u = 0; u < kQuads % U; ++u) PT_STEP(u, false);
#undef PT_LOADB
#undef PT_LOADA
#undef PT_MMA1
#undef PT_STEP
    });
  }
  double* out = L + d.l_off;
  if constexpr (!HARM) {
    each_sum([&](int n, int target, double a) __attribute__((always_inline)) {
      if (n < C) out[(size_t)n * kNTarget + target] = ldexp(a, l2 * (1 + order_of(n)));
      return a;
    });
  } else {
    // harmonic columns to LDS ([column][target of the part], over the window, which
    // every wave has finished reading), then every target is expanded to all C
    constexpr int NTG = 16 * S::TILES;
    double* lh = reinterpret_cast<double*>(win);
    static_assert(CR * NTG <= 2 * kWin * S::ROWS, "harmonic columns fit the window buffer");
    // position of a target in the part: level 2 holds one tile, the others whole planes
    auto local = [&](int target) { return LEVEL == 2 ? (target & 3) + 4 * ((target >> 3) & 3) : target - 64 * z0; };
    __syncthreads();
    each_sum([&](int n, int target, double a) __attribute__((always_inline)) {
      if (n < CR) lh[n * NTG + local(target)] = a;
      return a;
    });
    __syncthreads();
    const int tg = tid % NTG;
    const int target = 64 * z0 + (LEVEL == 2 ? tile_x(0) + (tg & 3) + kBlock * (ty + (tg >> 2)) : tg);
    for (int n = tid / NTG; n < C; n += S::NT / NTG) {
      const HExp& e = hexp[n];
      double v = 0.0;
      for (int u = 0; u < e.nterm; ++u) v = __builtin_fma(e.coef[u], lh[e.col[u] * NTG + tg], v);
      out[(size_t)n * kNTarget + target] = ldexp(v, l2 * (1 + order_of(n)));
    }
  }
}

// The quads' LDS offsets to LDS: tables [first, first + N) of woff.
template <int N, int NT>
__device__ __forceinline__ void load_offsets(short4 (*s_off)[kQuads + kOffPad], const short4* __restrict__ woff, int first) {
  for (int i = threadIdx.x; i < N * (kQuads + kOffPad); i += NT) {
    const int t = i / (kQuads + kOffPad), q = i % (kQuads + kOffPad);
    s_off[t][q] = q < kQuads ? woff[(first + t) * kQuads + q] : make_short4(0, 0, 0, 0);
  }
}

// Parts of sub-grids, two workgroups per compute unit. With a counter the
// workgroups take items from it; without, workgroup i runs item i.
template <bool HARM>
__global__ void __launch_bounds__(kPartThreads, 2) m2l_fwd_part_kernel(
    const WorkItem* __restrict__ items, int count, unsigned* __restrict__ counter,
    const DevDesc* __restrict__ desc, const double* __restrict__ M, double* __restrict__ L,
    const double* __restrict__ B2, const double* __restrict__ B3, const double* __restrict__ B4,
    const short4* __restrict__ woff, const uint32_t* __restrict__ ttouch, const int* __restrict__ rowtab,
    const HRound* __restrict__ hr2, const HRound* __restrict__ hr3, const HRound* __restrict__ hr4,
    const HExp* __restrict__ he2, const HExp* __restrict__ he3, const HExp* __restrict__ he4) {
  __shared__ double2 win[kWin * kWinRows2];
  __shared__ short4 s_off[3][kQuads + kOffPad];
  __shared__ int s_item;
  load_offsets<3, kPartThreads>(s_off, woff, 0);
  for (;;) {
    if (counter && threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
    __syncthreads();
    const int item = counter ? s_item : (int)blockIdx.x;
    if (item >= count) {
      // every workgroup draws one number past the items: the last one drawn clears
      // the counter for the next launch
      if (counter && threadIdx.x == 0 && item == count + (int)gridDim.x - 1) *counter = 0u;
      break;
    }
    const WorkItem w = items[item];
    const DevDesc d = desc[w.sub];
    auto run = [&](auto order, const double* B, const HRound* hr, const HExp* he) __attribute__((always_inline)) {
      constexpr int P = decltype(order)::value;
      const int level = w.part & 15, idx = w.part >> 4;
      auto part = [&](auto lv) __attribute__((always_inline)) {
        constexpr int LV = decltype(lv)::value;
        if (d.mask == kFullMask) fwd_part<P, HARM, true, LV>(d, M, L, B, ttouch, rowtab, win, s_off, hr, he, idx);
        else fwd_part<P, HARM, false, LV>(d, M, L, B, ttouch, rowtab, win, s_off, hr, he, idx);
      };
      if (level == 0) part(std::integral_constant<int, 0>{});
      else if (level == 1) part(std::integral_constant<int, 1>{});
      else part(std::integral_constant<int, 2>{});
    };
    switch (d.p) {
      case 2: run(std::integral_constant<int, 2>{}, B2, hr2, he2); break;
      case 3: run(std::integral_constant<int, 3>{}, B3, hr3, he3); break;
      case 4: run(std::integral_constant<int, 4>{}, B4, hr4, he4); break;
      default: break;
    }
    if (!counter) break;
    __syncthreads();   // every thread has read s_item; the item's LDS use is done
  }
}

// Whole sub-grids, one workgroup per compute unit, items from the counter.
//
// FUSE: the kernel computes each sub-grid's moments itself (the frame rows
// holding the reachable window, 8 particles per cell, written to M as the P2M
// kernel writes them) before that sub-grid's M2L reads them. A workgroup takes
// its next item when it starts an item and computes the next item's moments at
// the top of round (workgroup index mod rounds) of the current one, so at any
// time only about 1/rounds of the workgroups are in their HBM-bound moment
// phase while the others keep the matrix cores busy. Only the first item's
// moments are computed before any M2L. The moments are written and read by the
// same workgroup, with barriers between.
template <bool HARM, bool FUSE>
__global__ void __launch_bounds__(kWholeThreads) m2l_fwd_whole_kernel(
    const WorkItem* __restrict__ items, int count, unsigned* __restrict__ counter,
    const DevDesc* __restrict__ desc, const double* M, double* __restrict__ L,
    const double* __restrict__ B2, const double* __restrict__ B3, const double* __restrict__ B4,
    const short4* __restrict__ woff, const uint32_t* __restrict__ ttouch, const int* __restrict__ rowtab,
    const HRound* __restrict__ hr2, const HRound* __restrict__ hr3, const HRound* __restrict__ hr4,
    const HExp* __restrict__ he2, const HExp* __restrict__ he3, const HExp* __restrict__ he4,
    const double* __restrict__ pos, const double* __restrict__ mass, double* Mw) {
  // (FUSE: Mw is M, writable; the moment phase writes through it)
  __shared__ double2 win[kWinCells];
  __shared__ short4 s_off[1][kQuads + kOffPad];
  __shared__ int s_item;
  static_assert(kP2MRowsLds <= 2 * kWinCells && kWholeThreads == kP2MRowsThreads,
                "the moment phase fits the window buffer and the workgroup");
  load_offsets<1, kWholeThreads>(s_off, woff, 3);
  // moments of item `it` into M (the window buffer is free whenever this runs)
  auto moments = [&](int it) __attribute__((always_inline)) {
    const DevDesc dn = desc[items[it].sub];
    double* lds = reinterpret_cast<double*>(win);
    switch (dn.p) {
      case 2: p2m_window_rows<2>(dn, pos, mass, Mw, lds); break;
      case 3: p2m_window_rows<3>(dn, pos, mass, Mw, lds); break;
      case 4: p2m_window_rows<4>(dn, pos, mass, Mw, lds); break;
      default: break;
    }
  };
  int cur = 0;
  if constexpr (FUSE) {
    if (threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
    __syncthreads();
    cur = s_item;
    __syncthreads();   // every thread holds cur before s_item is written again
    if (cur < count) moments(cur);
  }
  for (;;) {
    if (threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
    __syncthreads();
    // FUSE: s_item is the next item, whose moments are computed during this one
    const int next = s_item;
    const int item = FUSE ? cur : next;
    if (item >= count) {
      // the last number any workgroup draws (one past the items each, two in the
      // fused form) clears the counter for the next launch
      if (threadIdx.x == 0 && next == count + (FUSE ? 2 : 1) * (int)gridDim.x - 1) *counter = 0u;
      break;
    }
    const DevDesc d = desc[items[item].sub];
    auto run = [&](auto order, const double* B, const HRound* hr, const HExp* he) __attribute__((always_inline)) {
      constexpr int P = decltype(order)::value;
      const auto hook = [&]() {
        if constexpr (FUSE) return MomentHook<decltype(moments)>{next, count, moments};
        else return NoMoments{};
      }();
      if (d.mask == kFullMask) fwd_part<P, HARM, true, kWhole>(d, M, L, B, ttouch, rowtab, win, s_off, hr, he, 0, hook);
      else fwd_part<P, HARM, false, kWhole>(d, M, L, B, ttouch, rowtab, win, s_off, hr, he, 0, hook);
    };
    switch (d.p) {
      case 2: run(std::integral_constant<int, 2>{}, B2, hr2, he2); break;
      case 3: run(std::integral_constant<int, 3>{}, B3, hr3, he3); break;
      case 4: run(std::integral_constant<int, 4>{}, B4, hr4, he4); break;
      default: break;
    }
    __syncthreads();   // every thread has read s_item; the item's LDS use is done
    cur = next;
  }
}

// ---------------------------------------------------------------------------
// split precision forward
// ---------------------------------------------------------------------------
//
// M = M_hi + M_lo and T = T_hi + T_lo (float32 parts of the float64 values;
// T_hi/T_lo are split from the float64 tables, M after its h-scaling). Per
// offset block the three products M_hi T_hi + M_hi T_lo + M_lo T_hi are
// summed in float32 on the matrix cores; each block sum is added to float64
// accumulators, and the h^(-1-|n|) scaling is applied in float64. One block
// is 16 offset quads (64 offsets) of one staged component pair.
//
// Columns n < 16 * N16 use v_mfma_f32_16x16x4 (A: lane -> cell l%16, offset
// slot l/16; B: lane -> offset slot l/16, column l%16; D: lane, v -> cell
// 4*(l/16)+v, column l%16). The remaining C - 16 * N16 columns use
// v_mfma_f32_4x4x1_16b on the same A register: block b = l/4 takes offset
// slot b/4 and cells 4*(b%4)..+3, so its D (lane, v -> cell 4*((l/4)%4)+v,
// column l%4) holds one partial sum per offset slot, added across slots
// at the end.

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f mfma16(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma4x1(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// One launch takes every sub-grid in quarters (two target planes, each wave two
// tiles) or eighths (one plane, one tile a wave), two 256-thread workgroups per
// compute unit, with the streamed forward's windows; a lane's hi and lo parts of
// both components are one 16-byte LDS read and one 16-byte table load, from L2,
// four quads ahead. Every block sum is taken in the order of the quads.
// What bounds it: the matrix units (float32: 6 products a quad, component pair and
// 16 columns), 0.8 of their time in use. Against one 512-thread workgroup per
// sub-grid with 4-byte table loads (p = 3): 1 sub-grid 2600 -> 350 us, 513 8.0 ->
// 4.57 ms, 1024 10.4 -> 8.46, 3000 31.1 -> 23.5; 1024 of p = 4 38.6 -> 24.9 (which
// took two passes over its columns).
constexpr int kSplitBlockQuads = 16;   // 64 offsets per float32 block sum

template <int P>
struct SplitCols {
  static constexpr int C = ncomp(P);
  static constexpr int N16 = C >= 16 ? C / 16 : 1;   // 16-wide column tiles
  static constexpr int REM = C > 16 * N16 ? 1 : 0;   // and a group of four on 4x4x1
  static constexpr int NG = 4 * N16 + REM;           // groups of 4 columns in the packed tables
};

template <int P, bool FULL, int LEVEL>
__device__ __forceinline__ void fwd_split_part(const DevDesc& d, const double* __restrict__ M, double* __restrict__ L,
                                               const float4* __restrict__ Bs, const uint32_t* __restrict__ ttouch,
                                               const int* __restrict__ rowtab, float4* win,
                                               const short4 (*s_off)[kQuads + kOffPad], int part) {
  using S = PartShape<LEVEL>;
  using F = SplitCols<P>;
  static_assert(LEVEL == 0 || LEVEL == 1, "quarters and eighths");
  constexpr int C = F::C, N16 = F::N16, REM = F::REM, NG = F::NG;
  constexpr int ROUNDS = (C + 1) / 2;
  constexpr int TPW = S::TPW;
  constexpr int U = 4;                                 // sets of table operands
  constexpr int AD = TPW * (N16 + REM) > 4 ? 1 : 3, AR = AD + 1;   // window operands: quads ahead (registers), sets
  static_assert(kSplitBlockQuads % U == 0 && U + AD <= kOffPad && U * NG * 32 <= (int)kTablePad, "read ahead");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kk = lane >> 4, ci = lane & 15;
  const int tile0 = part * S::TILES + wave * TPW;      // 4 plane + 2 y + x in the 2 x 2 tiles of a plane
  const int plane = tile0 >> 2, z0 = (part * S::TILES) >> 2;
  auto tile_x = [&](int t) { return (TPW == 1 ? tile0 & 1 : t & 1) * 4; };
  const int ty = ((tile0 >> 1) & 1) * 4;
  int abase[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) abase[t] = (tile_x(t) + (ci & 3) + 6) + kWin * (ty + (ci >> 2) + 6);
  const short* so = reinterpret_cast<const short*>(s_off[LEVEL == 0 ? plane - z0 : 2]) + kk;
  double acc[TPW][N16 + REM][4];                       // (the group of four last)
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int c = 0; c < N16 + REM; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[t][c][v] = 0.0;
  // per tile: the quads with a present source, one bit each; lane 4 t + i holds word i of tile t
  uint64_t live = 0;
  if constexpr (!FULL) {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = 64 * i + lane;
        const uint64_t w = __ballot(q < kQuads && (ttouch[(tile0 + t) * kQuads + min(q, kQuads - 1)] & d.mask) != 0);
        live = lane == 4 * t + i ? w : live;
      }
  }
  const int l2 = d.log2_inv_h;
  WindowCells<(S::STAGED * kWin + S::NT - 1) / S::NT, S::NT> wc;
  wc.set(d, rowtab + S::FIRST, S::STAGED, z0);
  const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float4*>(Bs), (short)0, ROUNDS * kQuads * NG * 256 + (int)kTablePad * 8, 0x00020000);
  const int vb16 = ((ci >> 2) * 16 + kk * 4 + (lane & 3)) * 16;      // column ci of a sixteen
  const int vb4 = (4 * N16 * 16 + kk * 4 + (lane & 3)) * 16;
  for (int r = 0; r < ROUNDS; ++r) {
    stage_window<P, false, S::STAGED>(wc, l2, M + d.m_off, nullptr, r, win);
    __syncthreads();
    int sq = r * kQuads * NG * 256;
    const short* sp = so;
    v4f f[TPW][N16 + REM];
    float4 b[U][N16 + REM], a[AR][TPW];
    int o[U];
    uint64_t lw[TPW][4];                               // live quads from the loop's first quad on
    auto load_b = [&](int set, int q) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < N16; ++c)
        b[set][c] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(brs, vb16 + 4 * c * 256, sq + q * NG * 256, 0));
      if (REM) b[set][N16 + REM - 1] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(brs, vb4, sq + q * NG * 256, 0));
    };
    auto load_a = [&](int u) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < TPW; ++t) a[u % AR][t] = win[abase[t] + o[u % U]];
    };
    // the products of tile t (of all tiles, interleaved, for t < 0)
    auto mma = [&](int u, int t0, int t1) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 6; ++i)                      // per component: hi hi, hi lo, lo hi
#pragma unroll
        for (int t = t0; t < t1; ++t) {
          const float av = i == 0 || i == 1 ? a[u % AR][t].x : i == 2 ? a[u % AR][t].y : i == 5 ? a[u % AR][t].w : a[u % AR][t].z;
#pragma unroll
          for (int c = 0; c < N16 + REM; ++c) {
            const float4 bb = b[u][c];
            const float bv = i == 0 || i == 2 ? bb.x : i == 1 ? bb.y : i == 4 ? bb.w : bb.z;
            f[t][c] = c < N16 ? mfma16(av, bv, f[t][c]) : mfma4x1(av, bv, f[t][c]);
          }
        }
    };
    auto fold_block = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int c = 0; c < N16 + REM; ++c)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[t][c][v] += (double)f[t][c][v];
    };
    // one quad, as in the streamed forward: window operands AD quads ahead, the
    // offset that operand set needs next, the products, the table operands of quad u + U
    auto step = [&](int u) __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
      load_a(u + AD);
      o[(u + AD) % U] = sp[(u + AD + U) * 4];
      if constexpr (FULL) {
        mma(u, 0, TPW);
      } else {
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < TPW; ++t)
          if ((uint32_t)lw[t][0] >> u & 1u) mma(u, t, t + 1);
        asm volatile("" ::: "memory");
      }
      load_b(u, u + U);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int u = 0; u < U; ++u) {
      load_b(u, u);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) o[u] = sp[u * 4];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < AD; ++u) {
      load_a(u);
      o[u] = sp[(u + U) * 4];
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!FULL) {
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          lw[t][i] = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)live, 4 * t + i) |
                     (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(live >> 32), 4 * t + i) << 32;
    }
#pragma unroll 1
    for (int q = 0; q < kQuads / U * U; q += U) {
      if (q % kSplitBlockQuads == 0) {
        if (q > 0) fold_block();
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
          for (int c = 0; c < N16 + REM; ++c) f[t][c] = (v4f){0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int u = 0; u < U; ++u) step(u);
      if constexpr (!FULL) {
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
#pragma unroll
          for (int i = 0; i < 3; ++i) lw[t][i] = lw[t][i] >> U | lw[t][i + 1] << (64 - U);
          lw[t][3] >>= U;
        }
      }
      sq += U * NG * 256;
      sp += U * 4;
    }
    static_assert(kQuads / U * U % kSplitBlockQuads != 0, "the last quads belong to the last block");
#pragma unroll
    for (int u = 0; u < kQuads % U; ++u) step(u);
    fold_block();
  }

  double* out = L + d.l_off;
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int t0 = tile_x(t) + kBlock * ty + kBlock * kBlock * plane;
    // 16x16 tiles: lane, v -> cell 4*(lane/16) + v (x = v, y = lane/16), column lane%16
#pragma unroll
    for (int c = 0; c < N16; ++c) {
      const int n = 16 * c + ci;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (n < C) out[(size_t)n * kNTarget + t0 + v + kBlock * kk] = ldexp(acc[t][c][v], l2 * (1 + order_of(n)));
    }
    if constexpr (REM > 0) {
      // sum the four offset-slot partials (lanes l, l^16, l^32, l^48)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double s = acc[t][N16][v];
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        const int n = 16 * N16 + (lane & 3);           // x = v, y = (lane/4)%4
        if (lane < 16 && n < C)
          out[(size_t)n * kNTarget + t0 + v + kBlock * ((lane >> 2) & 3)] = ldexp(s, l2 * (1 + order_of(n)));
      }
    }
  }
}

// Work: 4 (LEVEL 0) or 8 parts of every sub-grid of `items`, count in total. With
// a counter the workgroups take parts from it; without, workgroup i runs part i.
template <int LEVEL>
__global__ void __launch_bounds__(kPartThreads, 2) m2l_fwd_split_kernel(
    const WorkItem* __restrict__ items, int count, unsigned* __restrict__ counter,
    const DevDesc* __restrict__ desc, const double* __restrict__ M, double* __restrict__ L,
    const float4* __restrict__ B2, const float4* __restrict__ B3, const float4* __restrict__ B4,
    const short4* __restrict__ woff, const uint32_t* __restrict__ ttouch, const int* __restrict__ rowtab) {
  constexpr int kCut = kLevelParts[LEVEL];
  __shared__ float4 win[kWin * kWinRows2];
  __shared__ short4 s_off[3][kQuads + kOffPad];
  __shared__ int s_item;
  load_offsets<3, kPartThreads>(s_off, woff, 0);
  for (;;) {
    if (counter && threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
    __syncthreads();
    const int item = counter ? s_item : (int)blockIdx.x;
    if (item >= count) {
      // the last of the numbers past the items clears the counter for the next launch
      if (counter && threadIdx.x == 0 && item == count + (int)gridDim.x - 1) *counter = 0u;
      break;
    }
    const DevDesc d = desc[items[item / kCut].sub];
    auto run = [&](auto order, const float4* B) __attribute__((always_inline)) {
      constexpr int P = decltype(order)::value;
      if (d.mask == kFullMask) fwd_split_part<P, true, LEVEL>(d, M, L, B, ttouch, rowtab, win, s_off, item % kCut);
      else fwd_split_part<P, false, LEVEL>(d, M, L, B, ttouch, rowtab, win, s_off, item % kCut);
    };
    switch (d.p) {
      case 2: run(std::integral_constant<int, 2>{}, B2); break;
      case 3: run(std::integral_constant<int, 3>{}, B3); break;
      case 4: run(std::integral_constant<int, 4>{}, B4); break;
      default: break;
    }
    if (!counter) break;
    __syncthreads();   // every thread has read s_item; the item's LDS use is done
  }
}

// ---------------------------------------------------------------------------
// adjoint: dM_k(s) = h^-|k| sum_{(t, d) : t + d = s} sum_n [h^(-1-|n|) dL_n(t)] T_d[k][n]
// ---------------------------------------------------------------------------
//
// Scatter form: every (target t, offset d) pair contributes to exactly one
// output cell s = t + d of the 20^3 window, so no product is wasted (a
// gather over output tiles would compute mostly zeros, since dL lives on
// the 8^3 block only). One workgroup owns one sub-grid; for each pair of
// output components ("round") the window's accumulators live in LDS. Wave w
// holds target plane w (its dL values stay in registers for the whole
// sub-grid) and applies the offsets of one group at a time (one dz, or two dz
// at least 8 apart), so within a group every output cell has one writing wave.
// One instruction multiplies [16 targets x 4 dL components] by [4 components
// x (2 output components x 2 offsets)]; the two offsets of a pair never map
// two cells of one 4x4 tile to the same output cell (|dx2 - dx1| >= 4 or
// |dy2 - dy1| >= 4, or different dz). Results
// are added with LDS atomic adds that return nothing; one wave's LDS
// operations execute in issue order, so each cell's sum is taken in pair
// order and the result is reproducible bit for bit.

constexpr int kBwdWaves = 8;
constexpr int kBwdThreads = kBwdWaves * 64;
// component stride of the LDS accumulators: odd, so that the two components a
// lane pair adds (lanes 2i and 2i + 1) fall in different banks; an even stride
// doubles the LDS cycles of every add (measured: 16.2 against 8.3 cycles for a
// 64-lane ds_add_f64 in this kernel's address pattern)
constexpr int kAccStride = kWinCells + 17;
constexpr int kMaxPairs = 512;
constexpr int kBwdGroups = 8;       // offset groups, between barriers (see build_pairs)

// Hook: at the top of round r, after the round's first barrier and with the
// accumulators all zero, hook.run(lds) is called if hook.wants(r, ROUNDS)
// (uniform over the workgroup); it may use the accumulators as scratch, and they
// are cleared again after it. The A operands are rebuilt from dL after it.
struct NoHook {
  __device__ bool wants(int, int) const { return false; }
  __device__ void run(double*) const {}
};

// FULL: every neighbour block is present, so no pair is skipped and the pair
// loop carries no branches.
// HARM: the harmonic form; dL is folded to the (p+1)^2 harmonic columns, the
// rounds accumulate folded output components and the write-out expands them.
template <int P, bool FULL, bool HARM = false, class Hook = NoHook>
__device__ __forceinline__ void bwd_subgrid(const DevDesc& d, const double* __restrict__ dL,
                                            double* dM, const double* __restrict__ Bp,
                                            int npairs, const int* s_gs,
                                            const uint32_t* __restrict__ ptouch, double* smem,
                                            const int4* __restrict__ pairs, const HFold* __restrict__ hfold,
                                            const HOut* __restrict__ hout, Hook hook, uint32_t rounds) {
  constexpr int C = ncomp(P);
  constexpr int CR = HARM ? (P + 1) * (P + 1) : C;   // reduced components
  constexpr int KC = (CR + 3) / 4;    // dL component chunks of 4 (the reduction)
  constexpr int KC2 = (KC + 1) / 2;   // and pairs of chunks, one table load each
  constexpr int ROUNDS = (CR + 1) / 2;
  constexpr int TPW = 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // target plane
  const int kk = lane >> 4, ci = lane & 15, j = lane & 3;
  const int slot = j & 1, half = j >> 1;    // output component of the round, offset of the pair
  const int l2 = d.log2_inv_h;

  // A operands: dL of this wave's four 4x4 tiles, scaled by h^(-1-|n|)
  double a[TPW][KC];
  int obase[TPW];
  const double* src = dL + d.l_off;
  auto load_a = [&]() {
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int x0 = (t & 1) * 4, y0 = (t >> 1) * 4;
    const int tcell = x0 + (ci & 3) + kBlock * (y0 + (ci >> 2)) + kBlock * kBlock * wave;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      const int n = 4 * kc + kk;
      if constexpr (HARM) {
        // folded dL: the components that fold onto column n' (all of one order)
        double v = 0.0;
        if (n < CR) {
          const HFold& f = hfold[n];
          for (int u = 0; u < f.nterm; ++u)
            v = __builtin_fma(f.coef[u], src[(size_t)f.comp[u] * kNTarget + tcell], v);
          v = ldexp(v, l2 * (1 + order_of(f.comp[0])));
        }
        a[t][kc] = v;
      } else {
        a[t][kc] = n < C ? ldexp(src[(size_t)n * kNTarget + tcell], l2 * (1 + order_of(n))) : 0.0;
      }
    }
    // D layout: lane holds target cell (x = lane/16, y = (lane%16)/4) of the tile
    obase[t] = (x0 + (lane >> 4) + 6) + kWin * (y0 + ((lane & 15) >> 2) + 6) + kWin * kWin * (wave + 6) +
               slot * kAccStride;
  }
  };
  load_a();

  for (int i = tid; i < 2 * kAccStride; i += kBwdThreads) smem[i] = 0.0;

  // the pairs' output offsets (this lane's half) and, per target plane, the
  // blocks each pair writes, through buffer resources like the tables: waits for
  // them are waits on the vector memory counter, never on the LDS adds
  const __amdgpu_buffer_rsrc_t prs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<int4*>(pairs), (short)0, npairs * 16, 0x00020000);
  const __amdgpu_buffer_rsrc_t trs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(ptouch + wave * npairs), (short)0, npairs * 4, 0x00020000);
  double* out = dM + d.m_off;
  for (int r = 0; r < ROUNDS; ++r) {
    if (!((rounds >> r) & 1u)) continue;
    __syncthreads();
    if (hook.wants(r, ROUNDS)) {
      hook.run(smem);
      __syncthreads();
      for (int i = tid; i < 2 * kAccStride; i += kBwdThreads) smem[i] = 0.0;
      __syncthreads();
      load_a();
    }
    // tables through a buffer resource: a per-pair scalar offset and this lane's
    // fixed byte offset, so no per-pair address registers (reads past the end of
    // the tables would return zeros). Two chunks per 16-byte load, which occupies
    // the texture pipe no longer than 8 bytes (one chunk per load, 2048 sub-grids
    // of p = 3: harmonic 9.85 ms, dense 13.27, now 9.66 and 12.82; 1024 of p = 4
    // 12.05 and 19.25, now 11.7 and 18.5).
    const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(Bp), (short)0, ROUNDS * npairs * KC2 * 256, 0x00020000);
    const int sbase = r * npairs * KC2 * 256;
    const int vboff = (kk * 4 + j) * 16;
    // Three sets (tables, touch mask, products, output offset) rotate over the
    // pairs: at pair q the set of pair q - 1, whose products are issued, takes
    // the tables of pair q + 2 and the output offset of pair q - 1, and a set's
    // products are added into LDS (at that offset) just before the set is
    // multiplied again. Each offset is thus used two pairs after its load and
    // never copied, so no wait on a load younger than the tables in use. After
    // a barrier the sets hold zeros, so those adds change nothing.
    double b0[KC], b1[KC], b2[KC], acc0[TPW], acc1[TPW], acc2[TPW];
    int f0, f1, f2;              // this lane's output offset of the set's pending products
    uint32_t tm0 = 0, tm1 = 0, tm2 = 0;
#pragma unroll
    for (int t = 0; t < TPW; ++t) acc0[t] = acc1[t] = acc2[t] = 0.0;
#define BW_OFFSET(Q) ((int)__builtin_amdgcn_raw_buffer_load_b32(prs, half * 4, max((Q), 0) * 16, 0))
#define BW_LOAD(BS, FS, TS, Q)                                                      \
  {                                                                                 \
    const int q_ = (Q);                                                             \
    const int so_ = sbase + q_ * KC2 * 256;                                         \
    _Pragma("unroll") for (int kc = 0; kc < KC2; ++kc) {                            \
      const double2 b_ = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128( \
                                                         brs, vboff + kc * 256, so_, 0)); \
      BS[2 * kc] = b_.x;                                                            \
      if (2 * kc + 1 < KC) BS[2 * kc + 1] = b_.y;                                   \
    }                                                                               \
    if (!FULL) TS = __builtin_amdgcn_raw_buffer_load_b32(trs, 0, q_ * 4, 0);        \
    FS = BW_OFFSET(q_ - 3);                                                         \
  }
#define BW_FLUSH(AS, FS)                                                            \
  _Pragma("unroll") for (int t = 0; t < TPW; ++t)                                   \
    __hip_atomic_fetch_add(smem + obase[t] + (FS), AS[t], __ATOMIC_RELAXED,         \
                           __HIP_MEMORY_SCOPE_WORKGROUP);
#define BW_MMA(AS, BS)                                                              \
  {                                                                                 \
    _Pragma("unroll") for (int t = 0; t < TPW; ++t) AS[t] = 0.0;                    \
    _Pragma("unroll") for (int kc = 0; kc < KC; ++kc)                               \
      _Pragma("unroll") for (int t = 0; t < TPW; ++t) AS[t] = mfma4(a[t][kc], BS[kc], AS[t]); \
  }
// the loads and the adds are spread through the products
#define BW_INTERLEAVE()                                                             \
  {                                                                                 \
    constexpr int NMF = TPW * KC;                                                   \
    _Pragma("unroll") for (int i_ = 0; i_ < KC2; ++i_) {                            \
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                            \
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            \
    }                                                                               \
    _Pragma("unroll") for (int i_ = 0; i_ < TPW; ++i_) {                            \
      __builtin_amdgcn_sched_group_barrier(0x080, 1, 0);                            \
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                            \
    }                                                                               \
    __builtin_amdgcn_sched_group_barrier(0x008, NMF - TPW - KC2, 0);                     \
  }
// pair Q from set S (products AS, pending products of pair Q - 3 at FS); set N
// (pair Q - 1) takes the tables of Q + 2 and the offset of pair Q - 1
#define BW_STEP(BS, FS, TS, AS, BN, FN, TN, Q)                                      \
  BW_LOAD(BN, FN, TN, min((Q) + 2, npairs - 1));                                    \
  BW_FLUSH(AS, FS);                                                                 \
  if (FULL || (__builtin_amdgcn_readfirstlane(TS) & d.mask) != 0) {                \
    BW_MMA(AS, BS);                                                                 \
    BW_INTERLEAVE();                                                                \
  } else {                                                                          \
    _Pragma("unroll") for (int t = 0; t < TPW; ++t) AS[t] = 0.0;                    \
  }
// at the end of an offset group: every set's products go in (the latest pair of
// each set below QN, whose offset is loaded here), then the barrier
#define BW_PENDING(X, QN) ((QN) - 1 - ((((QN) - 1 - (X)) % 3) + 3) % 3)
#define BW_GROUP_END(QN)                                                            \
  if (__builtin_expect((QN) == gend, 0)) {                                          \
    f0 = BW_OFFSET(BW_PENDING(0, QN));                                              \
    f1 = BW_OFFSET(BW_PENDING(1, QN));                                              \
    f2 = BW_OFFSET(BW_PENDING(2, QN));                                              \
    BW_FLUSH(acc0, f0);                                                             \
    BW_FLUSH(acc1, f1);                                                             \
    BW_FLUSH(acc2, f2);                                                             \
    _Pragma("unroll") for (int t = 0; t < TPW; ++t) acc0[t] = acc1[t] = acc2[t] = 0.0; \
    __syncthreads();   /* the next group writes other planes of other waves */      \
    ++g;                                                                            \
    gend = __builtin_amdgcn_readfirstlane(s_gs[g + 1]);                             \
  }
    BW_LOAD(b0, f0, tm0, 0);
    BW_LOAD(b1, f1, tm1, min(1, npairs - 1));
    int g = 0, gend = __builtin_amdgcn_readfirstlane(s_gs[1]);
#pragma unroll 1
    for (int q = 0; q < npairs; q += 3) {
      BW_STEP(b0, f0, tm0, acc0, b2, f2, tm2, q);
      BW_GROUP_END(q + 1);
      if (__builtin_expect(q + 1 >= npairs, 0)) break;
      BW_STEP(b1, f1, tm1, acc1, b0, f0, tm0, q + 1);
      BW_GROUP_END(q + 2);
      if (__builtin_expect(q + 2 >= npairs, 0)) break;
      BW_STEP(b2, f2, tm2, acc2, b1, f1, tm1, q + 2);
      BW_GROUP_END(q + 3);
    }
#undef BW_OFFSET
#undef BW_LOAD
#undef BW_FLUSH
#undef BW_MMA
#undef BW_INTERLEAVE
#undef BW_STEP
#undef BW_PENDING
#undef BW_GROUP_END
    // write the round's components of dM (whole frame) and clear the accumulators
    if constexpr (HARM) {
      const HOut& ho = hout[r];
      for (int c = tid; c < kNCell; c += kBwdThreads) {
        const int jx = c % kFrame, jy = (c / kFrame) % kFrame, jz = c / (kFrame * kFrame);
        const bool win = jx >= kWin0 && jx < kWin0 + kWin && jy >= kWin0 && jy < kWin0 + kWin &&
                         jz >= kWin0 && jz < kWin0 + kWin;
        const bool pres = win && block_present(d.mask, jx, jy, jz);
        const int wc = (jx - kWin0) + kWin * (jy - kWin0) + kWin * kWin * (jz - kWin0);
        double g0 = 0.0, g1 = 0.0;
        if (win) {
          g0 = smem[wc];
          g1 = smem[kAccStride + wc];
          smem[wc] = 0.0;
          smem[kAccStride + wc] = 0.0;
        }
        for (int e = 0; e < ho.nout; ++e) {
          const int k = ho.comp[e];
          double* o = out + (size_t)k * kNCell + c;
          double v = __builtin_fma(ho.c1[e], g1, ho.c0[e] * g0);
          v = pres ? ldexp(v, l2 * order_of(k)) : 0.0;
          *o = ho.add[e] ? *o + v : v;
        }
      }
      continue;
    }
    const double sc0 = ldexp(1.0, l2 * order_of(2 * r));
    const double sc1 = ldexp(1.0, l2 * order_of(2 * r + 1));
    for (int c = tid; c < kNCell; c += kBwdThreads) {
      const int jx = c % kFrame, jy = (c / kFrame) % kFrame, jz = c / (kFrame * kFrame);
      const bool win = jx >= kWin0 && jx < kWin0 + kWin && jy >= kWin0 && jy < kWin0 + kWin &&
                       jz >= kWin0 && jz < kWin0 + kWin;
      const bool pres = win && block_present(d.mask, jx, jy, jz);
      const int wc = (jx - kWin0) + kWin * (jy - kWin0) + kWin * kWin * (jz - kWin0);
#pragma unroll
      for (int sl = 0; sl < 2; ++sl) {
        const int k = 2 * r + sl;
        double v = 0.0;
        if (win) {
          v = smem[sl * kAccStride + wc];
          smem[sl * kAccStride + wc] = 0.0;
        }
        if (k < C) out[(size_t)k * kNCell + c] = pres ? v * (sl ? sc1 : sc0) : 0.0;
      }
    }
  }
}

// the mass gradients of an earlier item, at the top of round (workgroup index
// mod rounds) of the current one
template <class F>
struct GradHook {
  int prev;
  F grads;
  __device__ bool wants(int r, int rounds) const {
    return prev >= 0 && r == (int)(blockIdx.x % (unsigned)rounds);
  }
  __device__ void run(double* lds) const { grads(prev, lds); }
};

// Work items are sub-grids, or some rounds of one (`part`: a bit per round, 0 for
// all): each round writes output components of its own, so a batch that cannot
// fill the GPU is spread over it by rounds, with the same bits. With a counter
// the workgroups take items from it; without, workgroup i runs item i.
//
// FUSE: the kernel also computes the mass gradients (the P2M adjoint of the
// sub-grid's dM, 8 particles per cell). A workgroup computes them for its
// previous item, whose dM it has written, at the top of round (workgroup index
// mod rounds) of its current item, so that HBM-bound work overlaps the matrix
// work of the other workgroups; its last item's follow after its loop.
template <bool HARM, bool FUSE = false>
__global__ void __launch_bounds__(kBwdThreads) m2l_bwd_kernel(
    const WorkItem* __restrict__ items, int count, unsigned* __restrict__ counter,
    const DevDesc* __restrict__ desc, const double* __restrict__ dL, double* dM,
    const double* __restrict__ B2, const double* __restrict__ B3, const double* __restrict__ B4,
    const int4* __restrict__ pairs, int npairs, const int* __restrict__ gstart,
    const uint32_t* __restrict__ ptouch, const HFold* __restrict__ hf2, const HFold* __restrict__ hf3,
    const HFold* __restrict__ hf4, const HOut* __restrict__ ho2, const HOut* __restrict__ ho3,
    const HOut* __restrict__ ho4, const double* __restrict__ pos = nullptr,
    double* __restrict__ dmass = nullptr) {
  __shared__ double smem[2 * kAccStride];
  __shared__ int s_gs[16];                // first pair of each offset group, and the end
  static_assert(kBwdGroups + 2 <= 16, "the group starts, the end and one read past it");
  __shared__ int s_item;
  static_assert(kP2MAdjRowsLds <= 2 * kAccStride && kBwdThreads == kP2MRowsThreads,
                "the gradient phase fits the accumulator buffer and the workgroup");
  if (threadIdx.x < kBwdGroups + 1) s_gs[threadIdx.x] = gstart[threadIdx.x];
  // the mass gradients of item `it` (its dM complete), with `lds` as staging
  auto grads = [&](int it, double* lds) __attribute__((always_inline)) {
    const DevDesc dp = desc[items[it].sub];
    switch (dp.p) {
      case 2: p2m_adjoint_rows<2>(dp, pos, dM, dmass, lds); break;
      case 3: p2m_adjoint_rows<3>(dp, pos, dM, dmass, lds); break;
      case 4: p2m_adjoint_rows<4>(dp, pos, dM, dmass, lds); break;
      default: break;
    }
  };
  int prev = -1;
  // (LDS operations complete in order; the staged values are read after the
  // barrier at the top of the item loop)
  for (;;) {
    if (counter && threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
    __syncthreads();
    const int item = counter ? s_item : (int)blockIdx.x;
    if (item >= count) {
      // the last of the numbers past the items clears the counter for the next launch
      if (counter && threadIdx.x == 0 && item == count + (int)gridDim.x - 1) *counter = 0u;
      break;
    }
    const DevDesc d = desc[items[item].sub];
    const uint32_t rounds = items[item].part ? (uint32_t)items[item].part : ~0u;
    const bool full = d.mask == kFullMask;
    const auto hook = [&]() {
      if constexpr (FUSE) return GradHook<decltype(grads)>{prev, grads};
      else return NoHook{};
    }();
    switch (d.p) {
      case 2:
        if (full) bwd_subgrid<2, true, HARM>(d, dL, dM, B2, npairs, s_gs, ptouch, smem, pairs, hf2, ho2, hook, rounds);
        else bwd_subgrid<2, false, HARM>(d, dL, dM, B2, npairs, s_gs, ptouch, smem, pairs, hf2, ho2, hook, rounds);
        break;
      case 3:
        if (full) bwd_subgrid<3, true, HARM>(d, dL, dM, B3, npairs, s_gs, ptouch, smem, pairs, hf3, ho3, hook, rounds);
        else bwd_subgrid<3, false, HARM>(d, dL, dM, B3, npairs, s_gs, ptouch, smem, pairs, hf3, ho3, hook, rounds);
        break;
      case 4:
        if (full) bwd_subgrid<4, true, HARM>(d, dL, dM, B4, npairs, s_gs, ptouch, smem, pairs, hf4, ho4, hook, rounds);
        else bwd_subgrid<4, false, HARM>(d, dL, dM, B4, npairs, s_gs, ptouch, smem, pairs, hf4, ho4, hook, rounds);
        break;
      default: break;
    }
    __syncthreads();
    prev = item;
    if (!counter) break;
  }
  if constexpr (FUSE) {
    if (prev >= 0) {
      __syncthreads();
      grads(prev, smem);
    }
  }
}

// ---------------------------------------------------------------------------
// table packing
// ---------------------------------------------------------------------------

// forward: [r][q][c][g][kk*4 + j] = T_{4q+kk}[2r+c][4g+j]
// streamed forward: [r][q][g][kk*4 + j][c], same values
__global__ void pack_fwd_kernel(const double* __restrict__ T, int p, double* __restrict__ out,
                                double* __restrict__ outl) {
  const int C = ncomp(p), NG = (C + 3) / 4, ROUNDS = (C + 1) / 2;
  const int total = ROUNDS * kQuads * 2 * NG * 16;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int j = i & 3, kk = (i >> 2) & 3;
  int rest = i >> 4;
  const int g = rest % NG; rest /= NG;
  const int c = rest % 2; rest /= 2;
  const int q = rest % kQuads;
  const int r = rest / kQuads;
  const int k = 2 * r + c, n = 4 * g + j, s = 4 * q + kk;
  const double v = (k < C && n < C) ? T[((size_t)s * C + k) * C + n] : 0.0;
  out[i] = v;
  outl[((((size_t)r * kQuads + q) * NG + g) * 16 + kk * 4 + j) * 2 + c] = v;
}

// split precision: [r][q][g][kk*4 + j] = the hi and lo parts of component 2r, then of 2r + 1
__global__ void pack_split_kernel(const double* __restrict__ T, int p, int ng, float* __restrict__ out) {
  const int C = ncomp(p), ROUNDS = (C + 1) / 2;
  const int total = ROUNDS * kQuads * ng * 32;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int c = i & 1, jj = (i >> 1) & 15;
  int rest = i >> 5;
  const int g = rest % ng; rest /= ng;
  const int q = rest % kQuads;
  const int r = rest / kQuads;
  const int k = 2 * r + c, n = 4 * g + (jj & 3), s = 4 * q + (jj >> 2);
  const double v = (k < C && n < C) ? T[((size_t)s * C + k) * C + n] : 0.0;
  const float h = (float)v;
  out[2 * (size_t)i] = h;
  out[2 * (size_t)i + 1] = (float)(v - (double)h);
}

// harmonic: [r][q][g][kk*4 + j][c] = T_{4q+kk}[rowk[2r + c]][colk[4g + j]] (0 where a map is -1)
struct HPackMaps {
  int rowk[32];   // full index of each round's folded components, or -1
  int colk[32];   // full index of each harmonic column, or -1 past (p+1)^2
};
__global__ void pack_fwdh_kernel(const double* __restrict__ T, int p, HPackMaps mp, int rounds, int ng,
                                 double* __restrict__ out) {
  const int C = ncomp(p);
  const int total = rounds * kQuads * ng * 32;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int c = i & 1;
  int rest = i >> 1;
  const int jj = rest & 15;
  rest >>= 4;
  const int g = rest % ng;
  rest /= ng;
  const int q = rest % kQuads;
  const int r = rest / kQuads;
  const int s = 4 * q + (jj >> 2);
  const int k = mp.rowk[2 * r + c], n = mp.colk[4 * g + (jj & 3)];
  out[i] = (k >= 0 && n >= 0) ? T[((size_t)s * C + k) * C + n] : 0.0;
}

// harmonic adjoint: [r][pair][kc/2][kk*4 + j][kc%2] = T_{s_(j/2)}[rowk[2r + j%2]][colk[4kc + kk]]
__global__ void pack_bwdh_kernel(const double* __restrict__ T, int p, const int4* __restrict__ pairs,
                                 int npairs, HPackMaps mp, int rounds, int kcn, double* __restrict__ out) {
  const int C = ncomp(p);
  const int total = rounds * npairs * kcn * 16;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int j = i & 3, kk = (i >> 2) & 3;
  int rest = i >> 4;
  const int kc = rest % kcn;
  rest /= kcn;
  const int q = rest % npairs;
  const int r = rest / npairs;
  const int4 pr = pairs[q];
  const int so = (j >> 1) ? pr.w : pr.z;
  const int k = mp.rowk[2 * r + (j & 1)], n = mp.colk[4 * kc + kk];
  out[((((size_t)r * npairs + q) * ((kcn + 1) / 2) + kc / 2) * 16 + (i & 15)) * 2 + kc % 2] =
      (so >= 0 && k >= 0 && n >= 0) ? T[((size_t)so * C + k) * C + n] : 0.0;
}

// adjoint: [r][pair][kc/2][kk*4 + j][kc%2] = T_{s_(j/2)}[2r + j%2][4kc + kk] (0 for a missing offset)
__global__ void pack_bwd_kernel(const double* __restrict__ T, int p, const int4* __restrict__ pairs,
                                int npairs, double* __restrict__ out) {
  const int C = ncomp(p), KC = (C + 3) / 4, ROUNDS = (C + 1) / 2;
  const int total = ROUNDS * npairs * KC * 16;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int j = i & 3, kk = (i >> 2) & 3;
  int rest = i >> 4;
  const int kc = rest % KC; rest /= KC;
  const int q = rest % npairs;
  const int r = rest / npairs;
  const int4 pr = pairs[q];
  const int so = (j >> 1) ? pr.w : pr.z;
  const int k = 2 * r + (j & 1), n = 4 * kc + kk;
  out[((((size_t)r * npairs + q) * ((KC + 1) / 2) + kc / 2) * 16 + (i & 15)) * 2 + kc % 2] =
      (so >= 0 && k < C && n < C) ? T[((size_t)so * C + k) * C + n] : 0.0;
}

size_t fwd_pack_elems(int p) {
  const int C = ncomp(p), NG = (C + 3) / 4, ROUNDS = (C + 1) / 2;
  return (size_t)ROUNDS * kQuads * 2 * NG * 16;
}

int split_groups(int p) {
  return p == 2 ? SplitCols<2>::NG : p == 3 ? SplitCols<3>::NG : SplitCols<4>::NG;
}

// (an odd chunk's pair is half empty)
size_t bwd_table_bytes(int rounds, int npairs, int chunks) {
  return (size_t)rounds * npairs * ((chunks + 1) / 2) * 256;
}

size_t bwd_pack_elems(int p, int npairs) {
  const int C = ncomp(p), KC = (C + 3) / 4, ROUNDS = (C + 1) / 2;
  return (size_t)ROUNDS * npairs * KC * 16;
}

// Offset groups of the adjoint: wave w writes output plane w + 6 + dz, so two
// dz whose difference is at least 8 never make two of the 8 waves write one
// plane, and their offsets can run between the same two barriers. The 13 dz
// values make 8 groups (5 of two dz, 3 of one), 100 to 138 offsets each.
constexpr int kBwdGroupDz[kBwdGroups][2] = {{-6, 2}, {-5, 3}, {-4, 4}, {-3, 5}, {-2, 6},
                                            {-1, -1}, {0, 0}, {1, 1}};

// Offsets of one group paired so that the two never send two cells of a 4x4
// tile to the same output cell (4 cells apart in x or y, or different dz, so
// different planes). The lanes of a tile's add hold 4 x, 4 y, 2 components and
// the 2 offsets of the pair; with the accumulator rows 20 doubles apart and an
// odd component stride, the add takes the fewest LDS cycles when the two
// offsets' x differ by 2 mod 4 (measured: 8.2 cycles for a 64-lane ds_add_f64,
// 16 to 20 for any other difference). So the offsets are first paired by a
// maximum matching among such partners (a bipartite graph: x = 0, 1 mod 4
// against x = 2, 3 mod 4), the rest greedily with any partner 4 cells away,
// and what is left runs alone.
void build_pairs(const std::vector<int>& st, std::vector<int4>* pairs, std::vector<int>* gstart) {
  gstart->clear();
  for (int gi = 0; gi < kBwdGroups; ++gi) {
    gstart->push_back((int)pairs->size());
    std::vector<int> ids;
    for (int i = 0; i < kNStencil; ++i)
      if (st[3 * i + 2] == kBwdGroupDz[gi][0] || st[3 * i + 2] == kBwdGroupDz[gi][1]) ids.push_back(i);
    const int n = (int)ids.size();
    auto dx = [&](int a) { return st[3 * ids[a]]; };
    auto compatible = [&](int a, int b) {
      return st[3 * ids[a] + 2] != st[3 * ids[b] + 2] || std::abs(dx(a) - dx(b)) >= 4 ||
             std::abs(st[3 * ids[a] + 1] - st[3 * ids[b] + 1]) >= 4;
    };
    auto preferred = [&](int a, int b) { return compatible(a, b) && (((dx(a) - dx(b)) % 4) + 4) % 4 == 2; };
    std::vector<int> mate(n, -1);
    std::vector<char> seen(n);
    // augmenting paths from the x = 0, 1 (mod 4) side
    std::function<bool(int)> augment = [&](int a) {
      for (int b = 0; b < n; ++b)
        if (!seen[b] && preferred(a, b)) {
          seen[b] = 1;
          if (mate[b] < 0 || augment(mate[b])) {
            mate[b] = a;
            mate[a] = b;
            return true;
          }
        }
      return false;
    };
    for (int a = 0; a < n; ++a)
      if (((dx(a) % 4) + 4) % 4 < 2) {
        std::fill(seen.begin(), seen.end(), 0);
        augment(a);
      }
    for (int a = 0; a < n; ++a)
      if (mate[a] < 0)
        for (int b = n - 1; b > a; --b)
          if (mate[b] < 0 && compatible(a, b)) {
            mate[a] = b;
            mate[b] = a;
            break;
          }
    for (int a = 0; a < n; ++a) {
      if (mate[a] >= 0 && mate[a] < a) continue;   // listed with its partner
      const int s1 = ids[a], s2 = mate[a] >= 0 ? ids[mate[a]] : -1;
      const int o1 = st[3 * s1] + kWin * st[3 * s1 + 1] + kWin * kWin * st[3 * s1 + 2];
      // an offset without a partner: the second half's tables are zero, so its
      // lanes add zeros; they go to the cells 2 away in x (toward the centre, so
      // into the same row of the same wave's plane), where the add is as cheap
      // as a preferred pair's
      const int o2 = s2 >= 0 ? st[3 * s2] + kWin * st[3 * s2 + 1] + kWin * kWin * st[3 * s2 + 2]
                             : o1 + (st[3 * s1] >= 0 ? -2 : 2);
      pairs->push_back(make_int4(o1, o2, s1, s2));
    }
  }
  gstart->push_back((int)pairs->size());
}

// Forward configurations.
struct Config {
  fmm_precision prec;
  bool stream;          // m2l_fwd_whole_kernel or m2l_fwd_part_kernel; otherwise (FMM_FP64) m2l_fwd_kernel with
  int waves = 8;        //   this many waves per workgroup (16-cell tiles per wave = 32 / waves)
  bool prefetch = false;   // and the table operands of the next offset quad loaded one quad ahead
                           // (not at p = 4 with 8 waves: the registers would spill)
  int same_as = -1;     // runs the same kernel as this entry (not timed by the autotuner)
};
constexpr Config kConfigs[] = {{FMM_FP64, true}, {FMM_FP64, true, 8, false, 0},
                               {FMM_FP64, false, 8, true},  {FMM_FP64, false, 8, false},
                               {FMM_FP64, false, 4, false}, {FMM_FP64, false, 4, true},
                               {FMM_SPLIT_FP32, false}, {FMM_FP64_HARMONIC, true}, {FMM_EXACT_SLICE, false},
                               {FMM_FP64_HARMONIC, true, 8, false, 7}, {FMM_FP64_HARMONIC, true, 8, false, 7}};
constexpr int kNumConfigs = sizeof(kConfigs) / sizeof(kConfigs[0]);

}  // namespace

// What a sub-grid takes against one of its order with every block present (256 alike,
// whole, p = 2 to 4): forward, with a share f of the pairs present, 0.71 to 0.76 at
// f = 0.34, 0.76 to 0.84 at 0.37 to 0.42, 0.86 to 0.93 at 0.52, 0.94 to 1.05 from
// 0.68 on, as its windows are staged all the same and a tile's products skip only
// quads with no present source; the adjoint 1.09 to 1.19 whatever the mask, as nearly
// every pair of offsets meets some present block.
void sort_by_cost(const fmm_subgrid* desc, int64_t nsub, bool harmonic, bool adjoint, WorkItem* out) {
  constexpr int64_t kAll = (int64_t)kNTarget * kNStencil;
  for (int64_t b = 0; b < nsub; ++b) {
    const int p = desc[b].p;
    const int64_t per_pair = harmonic ? (int64_t)(p + 1) * (p + 1) * (p + 1) * (p + 1)
                                      : (int64_t)ncomp(p) * ncomp(p);
    const int64_t pairs = pairs_of_mask(desc[b].mask);
    out[b].sub = (int32_t)b;
    const int64_t counted = !adjoint ? (kAll + pairs) / 2 : desc[b].mask == kFullMask ? kAll : kAll * 9 / 8;
    out[b].part = (int32_t)(per_pair * counted / 4096);   // below 2^18
  }
  std::sort(out, out + nsub, [](const WorkItem& a, const WorkItem& b) {
    return a.part != b.part ? a.part > b.part : a.sub < b.sub;
  });
}

void whole_items(WorkItem* items, int64_t n) {
  for (int64_t i = 0; i < n; ++i) items[i].part = 0;
}

// Time (in cost units) of the items, longest first, on num_cu compute units that
// each take the next one when free (ahead: when they start the one before it), with
// `each` added to every item.
static int64_t makespan(const WorkItem* items, int64_t n, int num_cu, int64_t total, int64_t each, bool ahead = false) {
  constexpr int kMaxUnits = 1024;
  if (n <= num_cu) return items[0].part + each;
  if (items[0].part == items[n - 1].part) return ((n + num_cu - 1) / num_cu) * (items[0].part + each);
  // unlike sub-grids end on short ones: past a few per unit the ends even out
  if (n > 4 * (int64_t)num_cu || num_cu > kMaxUnits) return (total + n * each) / num_cu;
  struct Unit {
    int64_t at, last;   // when it takes another item; ahead: the one it starts then
    bool operator>(const Unit& o) const { return at != o.at ? at > o.at : last > o.last; }
  };
  Unit units[kMaxUnits] = {};   // a min-heap
  for (int64_t i = 0; i < n; ++i) {
    std::pop_heap(units, units + num_cu, std::greater<Unit>());
    Unit& u = units[num_cu - 1];
    const int64_t cost = items[i].part + each;
    u.at += ahead ? u.last : cost;
    u.last = ahead ? cost : 0;
    std::push_heap(units, units + num_cu, std::greater<Unit>());
  }
  int64_t end = 0;
  for (int i = 0; i < num_cu; ++i) end = std::max(end, units[i].at + units[i].last);
  return end;
}

// the longest of the items is over 1.5 times the mean
static bool unlike_items(const WorkItem* items, int64_t n, int64_t total) {
  return n > 0 && 2 * n * items[0].part > 3 * total;
}

// In cost units (p = 3, all blocks present: 28,544 harmonic, 44,600 dense; a
// workgroup takes 0.031 us per unit, so 890 and 1350 us): a batch in parts takes
// 1.04 of its work spread evenly, with 900 units a sub-grid for the windows that its
// parts stage besides, plus a fifth of its longest sub-grid, or less where that one is
// cut finer (512 alike: 2050 us against 1850 whole; 300: 1230 against 1960; 256 of
// p = 2, uneven, harmonic: 565 against 526; 500 mixed, uneven, dense: 3910 against
// 4300). Moments cost 140 us inside a whole sub-grid's launch, where a workgroup also
// takes its next sub-grid when it starts one, and 0.64 us of the whole GPU per sub-grid
// in a launch of their own (harmonic, in one launch against two: 700 of p = 3 3192 and
// 3276 us, 2000 8390 and 8850, 1034 5190 and 4880 in parts; 513 mixed, uneven 3750
// and 3055).
StreamPlan plan_stream(const WorkItem* items, int64_t n, int num_cu) {
  constexpr int64_t kMomentsInside = 4500, kMomentsApart = 5300, kStaged = 900;
  if (n == 0) return StreamPlan{};
  int64_t total = 0;
  for (int64_t i = 0; i < n; ++i) total += items[i].part;
  const int64_t whole = makespan(items, n, num_cu, total, 0);
  const int64_t longest = (unlike_items(items, n, total) ? 8 : 21) * (int64_t)items[0].part;
  const int64_t parts = ((total + n * kStaged) * 104 / num_cu + longest) / 100;
  StreamPlan p;
  p.parts = parts < whole;
  p.fuse = n > num_cu && makespan(items, n, num_cu, total, kMomentsInside, true) <
                             std::min(parts, whole) + n * kMomentsApart / num_cu;
  return p;
}

// The adjoint's units (p = 3: 28,544 harmonic, 44,600 dense, 1230 and 1660 us of a
// workgroup). By rounds, a batch takes its work spread evenly (harmonic: 1.05 of
// it, as each round folds dL anew; dense 0.97) plus about an eighth of its longest
// sub-grid (dense: little where that one is far longer than the others): harmonic
// p = 3, whole against rounds: 1 sub-grid 1160 and 166 us, 256 1379 and
// 1459, 300 2505 and 1760, 512 2631 and 2776, 600 3795 and 3202, 2048 9853 and
// 10307; 256 of p = 4, uneven, 3340 and 3760; 900 of mixed p 6030 and 6300; dense, 19
// of mixed p 5170 and 326, 900 alike 6655 and 5854. Mass gradients cost 130 us inside
// a sub-grid's launch, and 0.98 us of the whole GPU per sub-grid in a launch of their
// own (600 harmonic: 4121 us inside, 3815 apart; 900: 5447 and 5746).
AdjointPlan plan_adjoint(const WorkItem* items, int64_t n, int num_cu, bool harmonic) {
  constexpr int64_t kGradsInside = 3100, kGradsApart = 5800;
  if (n == 0) return AdjointPlan{};
  int64_t total = 0;
  for (int64_t i = 0; i < n; ++i) total += items[i].part;
  const int64_t whole = makespan(items, n, num_cu, total, 0);
  const int64_t longest = (!unlike_items(items, n, total) ? 13 : harmonic ? 12 : 4) * (int64_t)items[0].part;
  const int64_t split = (total * (harmonic ? 105 : 97) / num_cu + longest) / 100;
  AdjointPlan p;
  p.rounds = split < whole && n <= kMaxRoundSubgrids;
  p.fuse = n > num_cu && makespan(items, n, num_cu, total, kGradsInside) <
                             (p.rounds ? split : whole) + n * kGradsApart / num_cu;
  return p;
}

// Where the levels' lines lie (costs c in sub-grids, harmonic p = 3, 256 compute
// units, us): a sub-grid goes in eighths while a quarter of it on a compute unit
// of its own takes longer than the whole batch on a full GPU. 32 alike: 288 in
// quarters, 188 in eighths; 43 alike 293 and 302; 100 alike 514 and 559. A batch
// of unlike sub-grids, whose longest would set the time, gains further up: 64
// mixed orders 956 and 701, 128 1102 and 958, 200 1390 and 1349; those with absent
// blocks, whose parts skip more than the whole does, a little less far (200 mixed
// and uneven, dense, the partly present ones of p = 4 in quarters: 1770 against 1905,
// 260 2200 against 2435). Tiles, which
// stage more window and use the matrix cores less well, only where eighths cannot
// reach every compute unit: 8 alike 266 in quarters, 158 in eighths, 118 in tiles;
// 24 alike 279, 180, 269.
int64_t split_items(const fmm_subgrid* desc, WorkItem* items, int64_t n, int num_cu) {
  int64_t total = 0, extra = 0;
  for (int64_t i = 0; i < n; ++i) total += items[i].part;
  const bool unlike = unlike_items(items, n, total);
  for (int64_t i = 0; i < n; ++i) {
    const int64_t c = (int64_t)items[i].part * num_cu;
    int level = 0;
    const int64_t tenths = !unlike ? 6 : desc[items[i].sub].mask == kFullMask ? 20 : 16;
    if (c * tenths / 10 > 4 * total) level = 1;
    if (c * 6 / 10 > 8 * total) level = 2;
    if (extra + kLevelParts[level] - kLevelParts[0] > kMaxExtraItems) level = 0;
    extra += kLevelParts[level] - kLevelParts[0];
    items[i].part = level;
  }
  // in place, from the back: an item's parts land at or after it
  const int64_t parts = n * kLevelParts[0] + extra;
  int64_t to = parts;
  for (int64_t i = n - 1; i >= 0; --i) {
    const WorkItem w = items[i];
    for (int k = kLevelParts[w.part] - 1; k >= 0; --k) items[--to] = WorkItem{w.sub, w.part | k << 4};
  }
  return parts;
}

namespace {
// blocks touched by the 8x8 target plane z shifted by offset o
uint32_t plane_blocks(const std::vector<int>& st, int z, int o) {
  const int dx = st[3 * o], dy = st[3 * o + 1], dz = st[3 * o + 2];
  const int bz = (8 + z + dz) / 8;
  uint32_t m = 0;
  for (int bx = (8 + dx) / 8; bx <= (15 + dx) / 8; ++bx)
    for (int by = (8 + dy) / 8; by <= (15 + dy) / 8; ++by) m |= 1u << (bx + 3 * by + 9 * bz);
  return m;
}
// blocks touched by target tile `tile` (4 plane + 2 y + x in the plane's 2 x 2 tiles) shifted by offset o
uint32_t tile_blocks(const std::vector<int>& st, int tile, int o) {
  const int x0 = 8 + 4 * (tile & 1) + st[3 * o], y0 = 8 + 4 * ((tile >> 1) & 1) + st[3 * o + 1];
  const int bz = (8 + (tile >> 2) + st[3 * o + 2]) / 8;
  uint32_t m = 0;
  for (int bx = x0 / 8; bx <= (x0 + 3) / 8; ++bx)
    for (int by = y0 / 8; by <= (y0 + 3) / 8; ++by) m |= 1u << (bx + 3 * by + 9 * bz);
  return m;
}

// Rows of the streamed forward's windows (WindowCells): of two target planes, of
// one, and those one tile of that one reaches (tile row 0, then 1).
std::vector<int> window_row_table() {
  std::vector<int> t;
  auto rows = [&](int nz, int y0, int span) {
    for (int w = 0, base = 0; w < nz + 12; ++w) {
      const int reach = window_reach(nz, w);
      for (int y = y0 - reach; y < y0 + span + reach; ++y) t.push_back(y | w << 8 | (base + y - (6 - reach)) << 16);
      base += 8 + 2 * reach;
    }
  };
  rows(2, 6, 8);
  rows(1, 6, 8);
  rows(1, 6, 4);
  rows(1, 10, 4);
  for (int w = 0; w < kWin; ++w)   // a whole sub-grid's window keeps its full planes in LDS
    for (int y = 6 - window_reach(8, w); y < 14 + window_reach(8, w); ++y) t.push_back(y | w << 8 | (y + kWin * w) << 16);
  return t;
}

// LDS offsets of the stencil offsets in those windows: from either target plane
// of two, from the one, and in a whole sub-grid's window.
std::vector<short> window_offsets(const std::vector<int>& st) {
  std::vector<short> v;
  for (int k = 0; k < 4; ++k)
    for (int i = 0; i < kNStencil; ++i) {
      const int dz = st[3 * i + 2];
      const int plane = k == 3 ? kWin * kWin * dz : k == 2 ? window_base(1, dz + 6) : window_base(2, dz + 6 + k);
      v.push_back((short)(plane + kWin * st[3 * i + 1] + st[3 * i]));
    }
  return v;
}

// ---- harmonic form: fold, round plan and expansion (host)

struct MI3 {
  int x, y, z;
};

std::vector<MI3> graded_indices(int p) {
  std::vector<MI3> v;
  for (int n = 0; n <= p; ++n)
    for (int kx = n; kx >= 0; --kx)
      for (int ky = n - kx; ky >= 0; --ky) v.push_back({kx, ky, n - kx - ky});
  return v;
}

int index_of(const std::vector<MI3>& v, int a, int b, int c) {
  for (size_t i = 0; i < v.size(); ++i)
    if (v[i].x == a && v[i].y == b && v[i].z == c) return (int)i;
  return -1;
}

// T(a,b,c) = -T(a+2,b,c-2) - T(a,b+2,c-2) for a family harmonic in its index,
// applied until the z-index is 0 or 1: coefficients over the kz <= 1 indices
void fold_into(const std::vector<MI3>& hs, int a, int b, int c, double coef, std::vector<double>* row) {
  if (c <= 1) {
    (*row)[index_of(hs, a, b, c)] += coef;
    return;
  }
  fold_into(hs, a + 2, b, c - 2, -coef, row);
  fold_into(hs, a, b + 2, c - 2, -coef, row);
}

struct HostHarmonic {
  std::vector<HRound> rounds;
  std::vector<HExp> exps;
  std::vector<HFold> folds;   // per harmonic column: the components folding onto it
  std::vector<HOut> outs;     // per round: the output components written from it
  HPackMaps maps;
  int ng = 0;
};

// The folded components are staged two per round; pairs that share moment
// components are formed first (largest overlap first), so each moment
// component is read as few times as possible.
bool build_harmonic(int p, HostHarmonic* out) {
  const std::vector<MI3> ks = graded_indices(p);
  std::vector<MI3> hs;
  for (const MI3& k : ks)
    if (k.z <= 1) hs.push_back(k);
  const int C = (int)ks.size(), CR = (int)hs.size();
  std::vector<std::vector<double>> F(C, std::vector<double>(CR, 0.0));   // F[k][k']
  for (int k = 0; k < C; ++k) fold_into(hs, ks[k].x, ks[k].y, ks[k].z, 1.0, &F[k]);
  std::vector<std::vector<int>> sup(CR);
  for (int h = 0; h < CR; ++h)
    for (int k = 0; k < C; ++k)
      if (F[k][h] != 0.0) sup[h].push_back(k);
  auto shared = [&](int a, int b) {
    int n = 0;
    for (int x : sup[a])
      for (int y : sup[b]) n += x == y;
    return n;
  };
  std::vector<std::pair<int, int>> pairs;
  std::vector<bool> used(CR, false);
  for (int best = CR; best >= 1; --best)
    for (int a = 0; a < CR; ++a)
      for (int b = a + 1; b < CR; ++b)
        if (!used[a] && !used[b] && shared(a, b) == best) {
          used[a] = used[b] = true;
          pairs.push_back({a, b});
        }
  std::vector<int> rest;
  for (int h = 0; h < CR; ++h)
    if (!used[h]) rest.push_back(h);
  for (size_t i = 0; i < rest.size(); i += 2)
    pairs.push_back({rest[i], i + 1 < rest.size() ? rest[i + 1] : -1});
  out->ng = (CR + 3) / 4;
  if ((int)pairs.size() * 2 > 32 || out->ng * 4 > 32) return false;
  for (int i = 0; i < 32; ++i) out->maps.rowk[i] = out->maps.colk[i] = -1;
  for (size_t r = 0; r < pairs.size(); ++r) {
    const int h0 = pairs[r].first, h1 = pairs[r].second;
    std::vector<int> u = sup[h0];
    if (h1 >= 0)
      for (int k : sup[h1])
        if (std::find(u.begin(), u.end(), k) == u.end()) u.push_back(k);
    std::sort(u.begin(), u.end());
    if ((int)u.size() > kHMaxSup) return false;
    HRound rd{};
    rd.nsup = (int)u.size();
    rd.ord0 = hs[h0].x + hs[h0].y + hs[h0].z;
    rd.ord1 = h1 >= 0 ? hs[h1].x + hs[h1].y + hs[h1].z : -1;
    for (size_t i = 0; i < u.size(); ++i) {
      rd.comp[i] = u[i];
      rd.c0[i] = F[u[i]][h0];
      rd.c1[i] = h1 >= 0 ? F[u[i]][h1] : 0.0;
    }
    out->rounds.push_back(rd);
    out->maps.rowk[2 * r] = index_of(ks, hs[h0].x, hs[h0].y, hs[h0].z);
    out->maps.rowk[2 * r + 1] = h1 >= 0 ? index_of(ks, hs[h1].x, hs[h1].y, hs[h1].z) : -1;
  }
  for (int h = 0; h < CR; ++h) out->maps.colk[h] = index_of(ks, hs[h].x, hs[h].y, hs[h].z);
  // adjoint: the fold of dL onto each harmonic column
  for (int h = 0; h < CR; ++h) {
    if ((int)sup[h].size() > kHMaxSup) return false;
    HFold f{};
    f.nterm = (int)sup[h].size();
    for (size_t i = 0; i < sup[h].size(); ++i) {
      f.comp[i] = sup[h][i];
      f.coef[i] = F[sup[h][i]][h];
    }
    out->folds.push_back(f);
  }
  // adjoint: dM_k = sum_k' F[k][k'] Gh_k', written from each round holding some k'
  std::vector<bool> written(C, false);
  out->outs.assign(pairs.size(), HOut{});
  for (size_t r = 0; r < pairs.size(); ++r) {
    const int h0 = pairs[r].first, h1 = pairs[r].second;
    HOut& o = out->outs[r];
    for (int k = 0; k < C; ++k) {
      const double c0 = F[k][h0], c1 = h1 >= 0 ? F[k][h1] : 0.0;
      if (c0 == 0.0 && c1 == 0.0) continue;
      if (o.nout == kHMaxOut) return false;
      o.comp[o.nout] = k;
      o.add[o.nout] = written[k] ? 1 : 0;
      o.c0[o.nout] = c0;
      o.c1[o.nout] = c1;
      ++o.nout;
      written[k] = true;
    }
  }
  for (int k = 0; k < C; ++k)
    if (!written[k]) return false;
  for (int k = 0; k < C; ++k) {
    HExp ex{};
    for (int h = 0; h < CR; ++h)
      if (F[k][h] != 0.0) {
        if (ex.nterm == kHMaxExp) return false;
        ex.col[ex.nterm] = h;
        ex.coef[ex.nterm] = F[k][h];
        ++ex.nterm;
      }
    out->exps.push_back(ex);
  }
  return true;
}

}  // namespace

int adjoint_round_sets(int p, bool harmonic, uint32_t sets[kMaxRounds]) {
  if (!harmonic) {
    const int n = (ncomp(p) + 1) / 2;
    for (int r = 0; r < n; ++r) sets[r] = 1u << r;
    return n;
  }
  // rounds that add to a component of an earlier round go with it, in order
  static const std::vector<std::vector<uint32_t>> all = [] {
    std::vector<std::vector<uint32_t>> v(kMaxP + 1);
    for (int q = 2; q <= kMaxP; ++q) {
      HostHarmonic hh;
      if (!build_harmonic(q, &hh)) continue;
      for (size_t r = 0; r < hh.outs.size(); ++r) {
        uint32_t set = 1u << r;
        for (size_t e = 0; e < v[q].size();) {
          bool shares = false;
          for (size_t o = 0; o < r; ++o)
            if ((v[q][e] >> o) & 1u)
              for (int a = 0; a < hh.outs[r].nout; ++a)
                for (int b = 0; b < hh.outs[o].nout; ++b) shares |= hh.outs[r].comp[a] == hh.outs[o].comp[b];
          if (shares) {
            set |= v[q][e];
            v[q].erase(v[q].begin() + e);
          } else {
            ++e;
          }
        }
        v[q].push_back(set);
      }
    }
    return v;
  }();
  for (size_t i = 0; i < all[p].size(); ++i) sets[i] = all[p][i];
  return (int)all[p].size();
}

bool harmonic_rounds_host(int p, std::vector<HRound>* rounds) {
  HostHarmonic hh;
  if (!build_harmonic(p, &hh)) return false;
  *rounds = hh.rounds;
  return true;
}

bool harmonic_plan_maps(int p, int32_t rowk[32], int32_t colk[32], int* nrounds) {
  HostHarmonic hh;
  if (!build_harmonic(p, &hh)) return false;
  for (int i = 0; i < 32; ++i) {
    rowk[i] = hh.maps.rowk[i];
    colk[i] = hh.maps.colk[i];
  }
  *nrounds = (int)hh.rounds.size();
  return true;
}

hipError_t mfma_tables_create(MfmaTables* t, double* const* d_T, const int* d_stencil,
                              hipStream_t s) {
  hipError_t e;
  t->stencil = d_stencil;
  int dev = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&t->num_cu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  const std::vector<int>& st = stencil_host();
  // forward: LDS offsets of the offsets, blocks each quad touches per target plane
  std::vector<int> off(kNStencil);
  for (int i = 0; i < kNStencil; ++i) off[i] = st[3 * i] + kWin * st[3 * i + 1] + kWin * kWin * st[3 * i + 2];
  std::vector<uint32_t> touch(8 * kQuads, 0u);
  for (int z = 0; z < 8; ++z)
    for (int q = 0; q < kQuads; ++q)
      for (int o = 4 * q; o < 4 * q + 4; ++o) touch[z * kQuads + q] |= plane_blocks(st, z, o);
  std::vector<uint32_t> ttouch(32 * kQuads, 0u);
  for (int tile = 0; tile < 32; ++tile)
    for (int q = 0; q < kQuads; ++q)
      for (int o = 4 * q; o < 4 * q + 4; ++o) ttouch[tile * kQuads + q] |= tile_blocks(st, tile, o);
  const std::vector<int> rowtab = window_row_table();
  const std::vector<short> woff = window_offsets(st);
  if (rowtab.size() != (size_t)(kWinRows2 + kWinRows1 + 2 * kWinRowsTile + kWinRows8)) return hipErrorInvalidValue;
  // adjoint: offset pairs grouped by dz, blocks each pair writes per target plane
  std::vector<int4> pairs;
  std::vector<int> gstart;
  build_pairs(st, &pairs, &gstart);
  if ((int)pairs.size() > kMaxPairs || gstart.size() != kBwdGroups + 1) return hipErrorInvalidValue;
  t->npairs = (int)pairs.size();
  std::vector<uint32_t> ptouch(8 * pairs.size(), 0u);
  for (int z = 0; z < 8; ++z)
    for (size_t q = 0; q < pairs.size(); ++q) {
      uint32_t m = plane_blocks(st, z, pairs[q].z);
      if (pairs[q].w >= 0) m |= plane_blocks(st, z, pairs[q].w);
      ptouch[z * pairs.size() + q] = m;
    }
  if ((e = hipMalloc(&t->lds_off, off.size() * sizeof(int))) != hipSuccess) return e;
  if ((e = hipMalloc(&t->touch, touch.size() * sizeof(uint32_t))) != hipSuccess) return e;
  if ((e = hipMalloc(&t->pairs, pairs.size() * sizeof(int4))) != hipSuccess) return e;
  if ((e = hipMalloc(&t->gstart, gstart.size() * sizeof(int))) != hipSuccess) return e;
  if ((e = hipMalloc(&t->ptouch, ptouch.size() * sizeof(uint32_t))) != hipSuccess) return e;
  if ((e = hipMalloc(&t->ttouch, ttouch.size() * sizeof(uint32_t))) != hipSuccess) return e;
  if ((e = hipMalloc(&t->rowtab, rowtab.size() * sizeof(int))) != hipSuccess) return e;
  if ((e = hipMalloc(&t->woff, woff.size() * sizeof(short))) != hipSuccess) return e;
  // synchronous copies: the host vectors die at return
  if ((e = hipMemcpy(t->ttouch, ttouch.data(), ttouch.size() * sizeof(uint32_t), hipMemcpyHostToDevice)) != hipSuccess) return e;
  if ((e = hipMemcpy(t->rowtab, rowtab.data(), rowtab.size() * sizeof(int), hipMemcpyHostToDevice)) != hipSuccess) return e;
  if ((e = hipMemcpy(t->woff, woff.data(), woff.size() * sizeof(short), hipMemcpyHostToDevice)) != hipSuccess) return e;
  if ((e = hipMemcpy(t->lds_off, off.data(), off.size() * sizeof(int), hipMemcpyHostToDevice)) != hipSuccess) return e;
  if ((e = hipMemcpy(t->touch, touch.data(), touch.size() * sizeof(uint32_t), hipMemcpyHostToDevice)) != hipSuccess) return e;
  if ((e = hipMemcpy(t->pairs, pairs.data(), pairs.size() * sizeof(int4), hipMemcpyHostToDevice)) != hipSuccess) return e;
  if ((e = hipMemcpy(t->gstart, gstart.data(), gstart.size() * sizeof(int), hipMemcpyHostToDevice)) != hipSuccess) return e;
  if ((e = hipMemcpy(t->ptouch, ptouch.data(), ptouch.size() * sizeof(uint32_t), hipMemcpyHostToDevice)) != hipSuccess) return e;
  for (int p = 2; p <= kMaxP; ++p) {
    const size_t nf = fwd_pack_elems(p), nb = bwd_pack_elems(p, t->npairs);
    if ((e = hipMalloc(&t->fwd[p], nf * sizeof(double))) != hipSuccess) return e;
    if ((e = hipMalloc(&t->fwdl[p], (nf + kTablePad) * sizeof(double))) != hipSuccess) return e;
    const int ngs = split_groups(p), ns = (ncomp(p) + 1) / 2 * kQuads * ngs * 32;
    if ((e = hipMalloc(&t->fwds[p], (ns + kTablePad) * 2 * sizeof(float))) != hipSuccess) return e;
    if ((e = hipMalloc(&t->bwd[p], bwd_table_bytes((ncomp(p) + 1) / 2, t->npairs, (ncomp(p) + 3) / 4))) != hipSuccess) return e;
    hipLaunchKernelGGL(pack_fwd_kernel, dim3((unsigned)((nf + 255) / 256)), dim3(256), 0, s, d_T[p], p,
                       t->fwd[p], t->fwdl[p]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(pack_split_kernel, dim3((unsigned)((ns + 255) / 256)), dim3(256), 0, s, d_T[p], p, ngs,
                       t->fwds[p]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(pack_bwd_kernel, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, d_T[p], p,
                       t->pairs, t->npairs, t->bwd[p]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    HostHarmonic hh;
    if (!build_harmonic(p, &hh)) return hipErrorInvalidValue;
    for (const HRound& rd : hh.rounds)
      if (rd.nsup > harmonic_sup(p)) return hipErrorInvalidValue;
    const size_t nh = hh.rounds.size() * (size_t)kQuads * hh.ng * 32;
    if ((e = hipMalloc(&t->fwdh[p], (nh + kTablePad) * sizeof(double))) != hipSuccess) return e;
    if ((e = hipMalloc(&t->hround[p], hh.rounds.size() * sizeof(HRound))) != hipSuccess) return e;
    if ((e = hipMalloc(&t->hexp[p], hh.exps.size() * sizeof(HExp))) != hipSuccess) return e;
    if ((e = hipMemcpy(t->hround[p], hh.rounds.data(), hh.rounds.size() * sizeof(HRound),
                       hipMemcpyHostToDevice)) != hipSuccess) return e;
    if ((e = hipMemcpy(t->hexp[p], hh.exps.data(), hh.exps.size() * sizeof(HExp),
                       hipMemcpyHostToDevice)) != hipSuccess) return e;
    hipLaunchKernelGGL(pack_fwdh_kernel, dim3((unsigned)((nh + 255) / 256)), dim3(256), 0, s, d_T[p], p,
                       hh.maps, (int)hh.rounds.size(), hh.ng, t->fwdh[p]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const size_t nbh = hh.rounds.size() * (size_t)t->npairs * hh.ng * 16;   // ng = n'-chunks of 4
    if ((e = hipMalloc(&t->bwdh[p], bwd_table_bytes((int)hh.rounds.size(), t->npairs, hh.ng))) != hipSuccess) return e;
    if ((e = hipMalloc(&t->hfold[p], hh.folds.size() * sizeof(HFold))) != hipSuccess) return e;
    if ((e = hipMalloc(&t->hout[p], hh.outs.size() * sizeof(HOut))) != hipSuccess) return e;
    if ((e = hipMemcpy(t->hfold[p], hh.folds.data(), hh.folds.size() * sizeof(HFold),
                       hipMemcpyHostToDevice)) != hipSuccess) return e;
    if ((e = hipMemcpy(t->hout[p], hh.outs.data(), hh.outs.size() * sizeof(HOut),
                       hipMemcpyHostToDevice)) != hipSuccess) return e;
    hipLaunchKernelGGL(pack_bwdh_kernel, dim3((unsigned)((nbh + 255) / 256)), dim3(256), 0, s, d_T[p], p,
                       t->pairs, t->npairs, hh.maps, (int)hh.rounds.size(), hh.ng, t->bwdh[p]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

void mfma_tables_destroy(MfmaTables* t) {
  for (int p = 0; p <= kMaxP; ++p) {
    if (t->fwd[p]) (void)hipFree(t->fwd[p]);
    if (t->fwdl[p]) (void)hipFree(t->fwdl[p]);
    t->fwdl[p] = nullptr;
    if (t->fwds[p]) (void)hipFree(t->fwds[p]);
    if (t->bwd[p]) (void)hipFree(t->bwd[p]);
    if (t->fwdh[p]) (void)hipFree(t->fwdh[p]);
    if (t->hround[p]) (void)hipFree(t->hround[p]);
    if (t->hexp[p]) (void)hipFree(t->hexp[p]);
    if (t->bwdh[p]) (void)hipFree(t->bwdh[p]);
    if (t->hfold[p]) (void)hipFree(t->hfold[p]);
    if (t->hout[p]) (void)hipFree(t->hout[p]);
    t->bwdh[p] = nullptr;
    t->hfold[p] = nullptr;
    t->hout[p] = nullptr;
    t->fwdh[p] = nullptr;
    t->hround[p] = nullptr;
    t->hexp[p] = nullptr;
    t->fwd[p] = t->bwd[p] = nullptr;
    t->fwds[p] = nullptr;
  }
  if (t->lds_off) (void)hipFree(t->lds_off);
  if (t->touch) (void)hipFree(t->touch);
  if (t->ttouch) (void)hipFree(t->ttouch);
  if (t->rowtab) (void)hipFree(t->rowtab);
  if (t->woff) (void)hipFree(t->woff);
  t->ttouch = nullptr;
  t->rowtab = nullptr;
  t->woff = nullptr;
  if (t->pairs) (void)hipFree(t->pairs);
  if (t->gstart) (void)hipFree(t->gstart);
  if (t->ptouch) (void)hipFree(t->ptouch);
  t->lds_off = nullptr;
  t->touch = nullptr;
  t->pairs = nullptr;
  t->gstart = nullptr;
  t->ptouch = nullptr;
}

int mfma_num_configs() { return kNumConfigs; }

bool mfma_config_supports(int cfg, fmm_precision prec) {
  return cfg >= 0 && cfg < kNumConfigs && kConfigs[cfg].prec == prec;
}

int mfma_default_config(fmm_precision prec) {
  for (int c = 0; c < kNumConfigs; ++c)
    if (kConfigs[c].prec == prec) return c;
  return 0;
}

bool mfma_config_streams(int cfg) { return cfg >= 0 && cfg < kNumConfigs && kConfigs[cfg].stream; }

bool mfma_config_distinct(int cfg) { return kConfigs[cfg].same_as < 0; }

hipError_t launch_m2l_stream(const MfmaTables& t, const WorkList& w, const DevDesc* d_desc, const double* M,
                             double* L, bool harmonic, hipStream_t s, const double* pos, const double* mass, double* Mw) {
  if (w.count == 0) return hipSuccess;
  if (pos && (mass == nullptr || Mw != M || w.parts)) return hipErrorInvalidValue;
  const HRound* const nr[3] = {};
  const HExp* const ne[3] = {};
  const HRound* const hr[3] = {t.hround[2], t.hround[3], t.hround[4]};
  const HExp* const he[3] = {t.hexp[2], t.hexp[3], t.hexp[4]};
#define STREAM_LAUNCH(KERNEL, GRID, NT, COUNTER, B, HR, HE, ...)                                                  \
  hipLaunchKernelGGL(KERNEL, dim3(GRID), dim3(NT), 0, s, w.items, w.count, COUNTER, d_desc, M, L, B[2], B[3], B[4], \
                     t.woff, t.ttouch, t.rowtab, HR[0], HR[1], HR[2], HE[0], HE[1], HE[2], ##__VA_ARGS__)
  if (w.parts) {
    const int grid = std::min(2 * t.num_cu, w.count);
    // no more items than workgroups: each takes its own, without the counter
    unsigned* counter = w.count > grid ? w.counter : nullptr;
    if (harmonic) STREAM_LAUNCH((m2l_fwd_part_kernel<true>), grid, kPartThreads, counter, t.fwdh, hr, he);
    else STREAM_LAUNCH((m2l_fwd_part_kernel<false>), grid, kPartThreads, counter, t.fwdl, nr, ne);
    return hipGetLastError();
  }
  const int grid = std::min(t.num_cu, w.count);
  if (harmonic && pos) STREAM_LAUNCH((m2l_fwd_whole_kernel<true, true>), grid, kWholeThreads, w.counter, t.fwdh, hr, he, pos, mass, Mw);
  else if (harmonic) STREAM_LAUNCH((m2l_fwd_whole_kernel<true, false>), grid, kWholeThreads, w.counter, t.fwdh, hr, he, pos, mass, Mw);
  else if (pos) STREAM_LAUNCH((m2l_fwd_whole_kernel<false, true>), grid, kWholeThreads, w.counter, t.fwdl, nr, ne, pos, mass, Mw);
  else STREAM_LAUNCH((m2l_fwd_whole_kernel<false, false>), grid, kWholeThreads, w.counter, t.fwdl, nr, ne, pos, mass, Mw);
#undef STREAM_LAUNCH
  return hipGetLastError();
}

hipError_t launch_m2l_split(const MfmaTables& t, const WorkList& w, const DevDesc* d_desc, const double* M,
                            double* L, hipStream_t s) {
  if (w.count == 0) return hipSuccess;
  if (w.parts) return hipErrorInvalidValue;
  const float4* B[3];
  for (int p = 2; p <= 4; ++p) B[p - 2] = reinterpret_cast<const float4*>(t.fwds[p]);
  // Eighths while all of them run at once: 1 sub-grid (p = 3) 350 us in eighths, 548
  // in quarters; 30 402 and 585, 50 of mixed p 1237 and 1870; 64 704 and 663, 100
  // 1266 and 1126, 1024 9087 and 8459.
  const int level = w.count * (int)kLevelParts[1] < 2 * t.num_cu ? 1 : 0;
  const int count = w.count * (int)kLevelParts[level];
  const int grid = std::min(2 * t.num_cu, count);
  unsigned* counter = count > grid ? w.counter : nullptr;
#define SPLIT_LAUNCH(LEVEL)                                                                              \
  hipLaunchKernelGGL(m2l_fwd_split_kernel<LEVEL>, dim3(grid), dim3(kPartThreads), 0, s, w.items, count,  \
                     counter, d_desc, M, L, B[0], B[1], B[2], t.woff, t.ttouch, t.rowtab)
  if (level == 1) SPLIT_LAUNCH(1);
  else SPLIT_LAUNCH(0);
#undef SPLIT_LAUNCH
  return hipGetLastError();
}

hipError_t launch_m2l_mfma(const MfmaTables& t, const WorkList& w, const DevDesc* d_desc,
                           const double* M, double* L, fmm_precision prec, int cfg, hipStream_t s) {
  if (w.count == 0) return hipSuccess;
  // (the per-wave FMM_FP64 configurations; the others have launches of their own)
  if (!mfma_config_supports(cfg, prec) || prec != FMM_FP64 || mfma_config_streams(cfg)) return hipErrorInvalidValue;
  const Config& c = kConfigs[cfg];
  const int grid = std::min(t.num_cu, w.count);
  hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(1), 0, s, w.counter);
#define FWD_LAUNCH(W, PFV)                                                                         \
  hipLaunchKernelGGL((m2l_fwd_kernel<W, PFV>), dim3(grid), dim3(W * 64), 0, s, w.items, w.count,   \
                     w.counter, d_desc, M, L, t.fwd[2], t.fwd[3], t.fwd[4], t.lds_off, t.touch)
  if (c.waves == 8 && c.prefetch) FWD_LAUNCH(8, true);
  else if (c.waves == 4 && c.prefetch) FWD_LAUNCH(4, true);
  else if (c.waves == 8) FWD_LAUNCH(8, false);
  else if (c.waves == 4) FWD_LAUNCH(4, false);
  else return hipErrorInvalidValue;
#undef FWD_LAUNCH
  return hipGetLastError();
}

hipError_t launch_m2l_mfma_backward(const MfmaTables& t, const WorkList& w, const DevDesc* d_desc,
                                    const double* dL, double* dM, bool harmonic, hipStream_t s,
                                    const double* pos, double* dmass) {
  if (w.count == 0) return hipSuccess;
  if ((pos == nullptr) != (dmass == nullptr) || (pos && w.parts)) return hipErrorInvalidValue;
  const int grid = std::min(t.num_cu, w.count);
  unsigned* counter = w.count > grid ? w.counter : nullptr;
  const HFold* nf = nullptr;
  const HOut* no = nullptr;
#define BWD_LAUNCH(HARMV, FUSEV, B, HF0, HF1, HF2, HO0, HO1, HO2)                                  \
  hipLaunchKernelGGL((m2l_bwd_kernel<HARMV, FUSEV>), dim3(grid), dim3(kBwdThreads), 0, s, w.items,  \
                     w.count, counter, d_desc, dL, dM, B[2], B[3], B[4], t.pairs, t.npairs,         \
                     t.gstart, t.ptouch, HF0, HF1, HF2, HO0, HO1, HO2, pos, dmass)
  if (harmonic && pos)
    BWD_LAUNCH(true, true, t.bwdh, t.hfold[2], t.hfold[3], t.hfold[4], t.hout[2], t.hout[3], t.hout[4]);
  else if (harmonic)
    BWD_LAUNCH(true, false, t.bwdh, t.hfold[2], t.hfold[3], t.hfold[4], t.hout[2], t.hout[3], t.hout[4]);
  else if (pos)
    BWD_LAUNCH(false, true, t.bwd, nf, nf, nf, no, no, no);
  else
    BWD_LAUNCH(false, false, t.bwd, nf, nf, nf, no, no, no);
#undef BWD_LAUNCH
  return hipGetLastError();
}

}  // namespace fmm
