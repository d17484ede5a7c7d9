// Gridding path of the measurement operator (paper Sect. 5.2: the adjoint and
// forward as type-1 / type-2 non-uniform FFTs).
//
// Adjoint (Eq. adjoint-phi) as four launches:
//   spread   sorted visibilities -> fine-grid band, one wave per work item
//            and output tile (kTile x kTile cells), accumulated in registers
//            by matrix instructions in FP32 (SpreadM) and in LDS in FP64
//            (SpreadCfg); every band tile is written exactly once (no global
//            atomics, no zero-fill pass).  Hot tiles are split into several
//            work items writing partial tiles.
//   fold     sums the partial tiles of split tiles, in a fixed order.
//   pass A   per band row: inverse FFT of length M along u, keeping the n
//            central frequencies (input pruned to the band, output pruned).
//   pass B   per pair of image rows: inverse FFT along v of the pass-A
//            columns, keeping n frequencies, then the apodisation and
//            1/n(l, m) correction, the image write and a fused max |eta|.
// Coplanar plans hold the half plane v >= 0 of the band only, and two real
// image rows come out of one complex transform (PairGeom).  The transforms
// run through LDS (fft_lds.h), or, at fine grids 4096 ... 16384 in FP32, in
// registers (reg_passA, reg_passB).
// Forward by interpolation (type-2): the same passes transposed with the
// opposite sign, then a w x w gather per visibility.
//
// Non-coplanar baselines (Sect. 2.1, Eq. phi-plane): the adjoint is
// w-stacked (planes and their kernel in the WStack comment), a group of
// planes at a time.  One small kernel weights the visibilities by the planes'
// kernel values (zero beyond their reach), the spread, fold and pass A run on
// all planes of the group in one launch each, and pass B rotates each output
// pixel by the planes' phases exp(2 pi i w_j c') and adds the real parts into
// the image; a last kernel divides by Psi(dw c') and takes the maximum.
#include <algorithm>
#include <cstring>
#include <memory>
#include <type_traits>

#include "common.h"
#include "es_kernel.h"
#include "fft_lds.h"
#include "half_plane.h"

namespace pc {

// Exponential of semicircle in FP64, exp(beta (sqrt(1 - z^2) - 1)) on |z| < 1
// (FP32: es_tap).
__device__ __forceinline__ double es_kernel(double z, double beta) {
  const double t = 1.0 - z * z;
  return t > 0.0 ? exp(beta * (sqrt(t) - 1.0)) : 0.0;
}

// A cell relative to an output tile's origin, in (-W, M - W] in periodic (wrap)
// mode.
__device__ __forceinline__ int tile_base(int c, int origin, int M, int W, int wrap) {
  int b = c - origin;  // in (-M, M): both are cells of the periodic grid
  if (wrap) {
    if (b < 0) b += M;
    if (b > M - W) b -= M;
  }
  return b;
}

// Spreading layout: one wave per work item owns the output tile in LDS
// (planar re/im, row stride kTile + BS).  Its lanes cover a BS x BS window of
// cells (BS = 8 for kernel widths up to 8, else W): the union of the
// footprints of every visibility whose first cell lies in one RB x RB block
// (RB = BS - W + 1; 3 x 3 first cells for W = 6).  Visibilities are sorted by
// that block, so a run of them shares the window: each lane adds its cell's
// weight times the value into a register, and the sums go to LDS (a plain
// read-add-write: the lanes of one instruction address distinct cells and a
// wave's LDS operations complete in order) only when the block changes.  The
// wave stages 64 visibilities at a time, one per lane: the block key, the
// value, and the kernel weights already shifted onto the window's rows and
// columns (zero outside the visibility's own footprint), so that in the
// accumulation loop a lane reads its two weights at fixed offsets and spends
// one multiply and two FMAs per visibility.  No LDS atomics (whose per-lane
// serialisation made them the bottleneck), and each cell receives its
// contributions in a fixed order, so the result is bitwise reproducible.
// Hot tiles are split across work items upstream.
template <typename R, int W>
struct SpreadCfg {
  static constexpr int BS = spread_span(W);      // window side (cells)
  static constexpr int RB = spread_block(W);     // block side (first cells)
  static constexpr int NPASS = (BS * BS + 63) / 64;
  static constexpr int S = kTile + BS;           // LDS row stride
  static constexpr int TILE = kTile * S;         // reals per plane
  static constexpr int REC = 2 * BS + 4;         // wy[BS], wx[BS], re, im, key, pad
  static constexpr int STG = 64 * REC;
  static constexpr int U = 16;                   // visibilities per inner step
  static constexpr size_t lds_bytes = sizeof(R) * (2 * TILE + STG);
};

// Block key of a window origin (bu, bv) relative to the tile, both in
// (-BS, kTile): one integer, so that a run test is a single comparison.
__device__ __forceinline__ int block_key(int bu, int bv) { return ((bv + 64) << 8) | (bu + 64); }
constexpr int kNoBlock = -1;

// Adds a run's per-cell register sums into the LDS tile and clears them.
// single_u: the periodic grid is one tile wide along u, so window cells left of
// the tile wrap onto its other end (FP64 plans are coplanar: no wrap along v).
template <typename R, int W>
__device__ __forceinline__ void spread_flush(int lane, int key, bool single_u,
                                             R (&accr)[SpreadCfg<R, W>::NPASS],
                                             R (&acci)[SpreadCfg<R, W>::NPASS], R* tre,
                                             R* tim) {
  using C = SpreadCfg<R, W>;
  if (key != kNoBlock) {
    const int bu = (key & 0xff) - 64, bv = (key >> 8) - 64;
#pragma unroll
    for (int ps = 0; ps < C::NPASS; ++ps) {
      const int tap = lane + 64 * ps;
      const int a = tap / C::BS, b = tap - (tap / C::BS) * C::BS;
      const int y = bv + a;
      int x = bu + b;
      if (single_u) x &= kTile - 1;
      if ((C::BS * C::BS % 64 == 0 || tap < C::BS * C::BS) && (unsigned)y < (unsigned)kTile &&
          (unsigned)x < (unsigned)kTile) {
        tre[y * C::S + x] += accr[ps];
        tim[y * C::S + x] += acci[ps];
      }
    }
  }
#pragma unroll
  for (int ps = 0; ps < C::NPASS; ++ps) {
    accr[ps] = R(0);
    acci[ps] = R(0);
  }
}

// One staged visibility as fetched from global memory.
template <typename R>
struct VisIn {
  uint32_t cell;
  R su, sv;
  cpx<R> val;
};

// Position in the sorted arrays of the q-th visibility of a work item whose
// four ranges have cumulative lengths c1 <= c2 <= c3 and offsets b0..b3
// (plain values, so that no reference is selected at run time).
__device__ __forceinline__ int chunk_index(int q, int c1, int c2, int c3, int b0, int b1, int b2,
                                           int b3) {
  const int add = q < c1 ? b0 : (q < c2 ? b1 : (q < c3 ? b2 : b3));
  return q + add;
}

// End (cumulative) of the range that position q of a work item falls in.
__device__ __forceinline__ int range_end(int q, int c1, int c2, int c3, int total) {
  return q < c1 ? c1 : (q < c2 ? c2 : (q < c3 ? c3 : total));
}

template <typename R>
__device__ __forceinline__ VisIn<R> fetch_vis(int s, const uint32_t* __restrict__ cell,
                                              const R* __restrict__ off,
                                              const cpx<R>* __restrict__ vals,
                                              const int32_t* __restrict__ perm) {
  VisIn<R> v;
  v.cell = cell[s];
  v.su = off[2 * s];
  v.sv = off[2 * s + 1];
  v.val = perm ? vals[perm[s]] : vals[s];
  return v;
}

template <typename R, int W>
__device__ __forceinline__ void spread_body(
    const GridGeom& g, const SpreadChunk& ch, const uint32_t* __restrict__ cell,
    const R* __restrict__ off, const cpx<R>* __restrict__ vals, const int32_t* __restrict__ perm,
    cpx<R>* __restrict__ grid, cpx<R>* __restrict__ partials) {
  using C = SpreadCfg<R, W>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int lane = threadIdx.x;
  R* tre = reinterpret_cast<R*>(smem_raw);
  R* tim = tre + C::TILE;
  R* stg = tim + C::TILE;  // [64][REC]
  const int tv = ch.tile / g.ntu, tu = ch.tile - tv * g.ntu;
  const int ov = g.v0 + tv * kTile, ou = g.u0 + tu * kTile;
  const bool single_u = g.wrap && g.M == kTile;
  const R inv = R(2) / R(W);
  const R beta = g.beta64;
  // cumulative range boundaries
  const int c1 = ch.end[0] - ch.beg[0];
  const int c2 = c1 + ch.end[1] - ch.beg[1];
  const int c3 = c2 + ch.end[2] - ch.beg[2];
  const int total = c3 + ch.end[3] - ch.beg[3];
  const int b0 = ch.beg[0], b1 = ch.beg[1] - c1, b2 = ch.beg[2] - c2, b3 = ch.beg[3] - c3;
  constexpr int NPASS = C::NPASS;
  constexpr int U = C::U;
  // The first batch's global loads go out before the tile is cleared; each
  // later batch's before the current batch's accumulation loop.
  VisIn<R> nx{0u, R(0), R(0), {R(0), R(0)}};
  if (lane < total)
    nx = fetch_vis<R>(chunk_index(lane, c1, c2, c3, b0, b1, b2, b3), cell, off, vals, perm);
  for (int i = lane; i < C::TILE; i += 64) {
    tre[i] = R(0);
    tim[i] = R(0);
  }
  // per-lane window cell (row a, column b) for each pass
  int ia[NPASS], ib[NPASS];
#pragma unroll
  for (int ps = 0; ps < NPASS; ++ps) {
    const int tap = lane + 64 * ps;
    const bool ok = C::BS * C::BS % 64 == 0 || tap < C::BS * C::BS;
    ia[ps] = ok ? tap / C::BS : 0;
    ib[ps] = ok ? C::BS + tap - (tap / C::BS) * C::BS : C::BS;  // wx row follows wy
  }
  int ckey = kNoBlock;
  R accr[NPASS], acci[NPASS];
#pragma unroll
  for (int ps = 0; ps < NPASS; ++ps) accr[ps] = acci[ps] = R(0);
#pragma unroll 1
  for (int base = 0; base < total; base += 64) {
    // stage one visibility per lane: weights shifted onto the window
    const int q = base + lane;
    R* my = stg + lane * C::REC;
    if (q < total) {
      const int cu = cell_u(nx.cell), cv = cell_v(nx.cell);
      const int du = cu % C::RB, dv = cv % C::RB;
      const int bu = tile_base(cu - du, ou, g.M, C::BS, g.wrap);
      const int bv = cv - dv - ov;
      // the W taps of each axis land at window positions d .. d + W - 1
      // (d = dv or du < RB); the other BS - W positions are zero
#pragma unroll
      for (int j = 0; j < C::BS; ++j) my[j] = my[C::BS + j] = R(0);
#pragma unroll
      for (int t = 0; t < W; ++t) {
        my[dv + t] = es_kernel((nx.sv + R(t)) * inv, beta);
        my[C::BS + du + t] = es_kernel((nx.su + R(t)) * inv, beta);
      }
      my[2 * C::BS] = nx.val.x;
      my[2 * C::BS + 1] = nx.cell & kFlip ? -nx.val.y : nx.val.y;
      *reinterpret_cast<int*>(&my[2 * C::BS + 2]) = block_key(bu, bv);  // in the R-sized slot
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (q + 64 < total)
      nx = fetch_vis<R>(chunk_index(q + 64, c1, c2, c3, b0, b1, b2, b3), cell, off, vals, perm);
    const int nb = total - base < 64 ? total - base : 64;
#pragma unroll 1
    for (int v0 = 0; v0 < nb; v0 += U) {
      int key[U];
      R vr[U], vi[U], wg[U][NPASS];
#pragma unroll
      for (int u = 0; u < U; ++u) {  // issue all LDS reads of the step first
        const R* kw = stg + (v0 + u) * C::REC;
        // records past the batch end hold a stale key and stale weights:
        // their key is replaced by kNoBlock below and their weights unused
        key[u] = *reinterpret_cast<const int*>(&kw[2 * C::BS + 2]);
        vr[u] = kw[2 * C::BS];
        vi[u] = kw[2 * C::BS + 1];
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps) wg[u][ps] = kw[ia[ps]] * kw[ib[ps]];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (v0 + u < nb) {
          const int k = __builtin_amdgcn_readfirstlane(key[u]);
          if (k != ckey) {  // same for every lane of the wave
            spread_flush<R, W>(lane, ckey, single_u, accr, acci, tre, tim);
            ckey = k;
          }
#pragma unroll
          for (int ps = 0; ps < NPASS; ++ps) {
            accr[ps] = fma(wg[u][ps], vr[u], accr[ps]);
            acci[ps] = fma(wg[u][ps], vi[u], acci[ps]);
          }
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  spread_flush<R, W>(lane, ckey, single_u, accr, acci, tre, tim);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  cpx<R>* dst;
  size_t stride;
  if (ch.slot < 0) {
    dst = grid + (size_t)(tv * kTile) * g.nu + tu * kTile;
    stride = g.nu;
  } else {
    dst = partials + (size_t)ch.slot * kTile * kTile;
    stride = kTile;
  }
  for (int i = lane; i < kTile * kTile; i += 64) {
    const int y = i / kTile, x = i - y * kTile;
    dst[(size_t)y * stride + x] = {tre[y * C::S + x], tim[y * C::S + x]};
  }
}

// FP32 spreading on the matrix cores.
//
// A tile's sum over its visibilities, tile[y][x] = sum_k wy_k[y] (wx_k[x] v_k),
// is a product of a 32 x K and a K x 64 matrix (re and im of each column): the
// wave keeps the whole 32 x 32 complex tile in 2 x 4 accumulator blocks of 16
// rows by 8 complex columns, and v_mfma_f32_16x16x4_f32 adds four
// visibilities to one block.  Only the blocks that the footprints of a step's
// visibilities reach are computed (about two of the eight: the plan sorts a
// tile's visibilities by the blocks they reach), so sparse and dense tiles
// cost the same per visibility, and nothing is flushed between visibilities.
//
// The factors are staged in LDS, BATCH visibilities at a time: the tables
// wy[y][j] and wx[x][j], zero outside visibility j's W taps, and the values.
// Lanes 0-31 evaluate the row weights of one visibility each, lanes 32-63 its
// column weights, and write the W taps; after the batch they write zeros over
// them.  The row stride of 34 floats makes the operand reads conflict-free.
// Taps outside the tile (visibilities spilling from a neighbour) go to row 32,
// which no operand reads.  FP32 products and sums; deterministic (each cell
// receives its terms in a fixed order).
//
// Against the register window of SpreadCfg in FP32 (spread alone): 13.7 -> 5.6 us
// for 3,968 visibilities on a 256^2 fine grid, 29 -> 22 for 424,800 on 2048^2,
// 89 -> 63 for 2,088,960 on 8192^2; 8,372,224 on 16384^2 with the fold 255 -> 232.
// Of 208 us there (plan-order input) 46 go with the matrix instructions, 20
// with the weights' exponentials and 11 with the clearing, each left out
// alone: bound by the issue of the staging and the loads together.
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct SpreadM {
  static constexpr int BATCH = 32;              // visibilities per staged batch
  static constexpr int S = kTile + 2;           // tile row stride (complex cells)
  static constexpr int RS = 34;                 // table row stride (floats)
  static constexpr int TAB_F = kTile * RS + BATCH;  // floats per table, with the discard row
  static constexpr int WAVE_F = 2 * TAB_F + 2 * BATCH;  // 9,216 bytes
  static_assert(2 * kTile * S <= WAVE_F, "the finished tile overlays the tables");
  static constexpr size_t lds_bytes = kSpreadQuad * sizeof(float) * WAVE_F;
};

__device__ __forceinline__ void lds_order() {  // a wave's own LDS writes before its reads
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Accumulates one work item and leaves its tile in the wave's LDS region
// (complex cells, row stride S); the caller writes it out.
// perm: NULL when vals is in plan order, else the plan -> caller map.
template <int W>
__device__ __forceinline__ void spread_group_accumulate(
    const GridGeom& g, const SpreadChunk& ch, const uint32_t* __restrict__ cell,
    const float* __restrict__ off, const cpx<float>* __restrict__ vals,
    const int32_t* __restrict__ perm, float* __restrict__ region, int lane) {
  using C = SpreadM;
  static_assert(W >= 2 && W <= kMaxWidth, "kernel widths");
  float* tab = region + (lane >= 32 ? C::TAB_F : 0);  // this lane's table: wy, wx [33][RS]
  float* tval = region + 2 * C::TAB_F;                // Re v [32], Im v [32]
  const int j = lane & 31;
  const bool cols = lane >= 32;
  const int tv = ch.tile / g.ntu, tu = ch.tile - tv * g.ntu;
  const int origin = cols ? g.u0 + tu * kTile : g.v0 + tv * kTile;
  const int wrap = cols ? g.wrap : g.wrapv;
  const bool single = g.M == kTile && wrap;  // the periodic grid is one tile wide
  const bool periodic = (g.wrap | g.wrapv) != 0;
  const int bside = cols ? 8 : 16;           // the axis's block side
  const int c1n = ch.end[0] - ch.beg[0];
  const int c2n = c1n + ch.end[1] - ch.beg[1];
  const int c3n = c2n + ch.end[2] - ch.beg[2];
  const int total = c3n + ch.end[3] - ch.beg[3];
  const int b0 = ch.beg[0], b1 = ch.beg[1] - c1n, b2 = ch.beg[2] - c2n, b3 = ch.beg[3] - c3n;
  f32x4 acc[2][4];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[rb][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Loads run ahead through three record buffers (batch k uses buffer k mod 3).
  // The cell, offset and source index of batch k + 3 and the value of batch
  // k + 2 are issued while batch k is staged and summed; the value of a
  // caller-order input needs its source index, which was issued a batch
  // earlier, so no load waits on one issued just before it.  Lanes past the
  // end load the last record again, and both ways of forming the index issue
  // the same loads, so that each wait covers exactly the batch it consumes.
  struct Raw {
    uint32_t cell;
    float off;
    uint32_t ld, sidx;  // the loaded index, and the record's plan position
    cpx<float> val;
  };
  // (for a plan-order input the index load reads the cell array instead and
  // is discarded, so that every path issues the same loads)
  const uint32_t* src_arr = perm ? reinterpret_cast<const uint32_t*>(perm) : cell;
  const uint32_t j1 = (uint32_t)j, j2 = 2 * j1 + (cols ? 0u : 1u);
  auto load_pre = [&](Raw& rw, int q0) {
    // a batch inside one of the four ranges has a scalar base for all lanes
    const int end = range_end(q0, c1n, c2n, c3n, total);
    const uint32_t s0 = (uint32_t)chunk_index(q0, c1n, c2n, c3n, b0, b1, b2, b3);
    if (q0 + C::BATCH <= end) {
      rw.cell = (cell + s0)[j1];
      rw.off = (off + 2 * (size_t)s0)[j2];
      rw.ld = (src_arr + s0)[j1];
      rw.sidx = s0 + j1;
    } else {
      const int q = q0 + j;
      const uint32_t sidx =
          (uint32_t)chunk_index(q < total ? q : total - 1, c1n, c2n, c3n, b0, b1, b2, b3);
      rw.cell = cell[sidx];
      rw.off = off[2 * (size_t)sidx + (j2 & 1u)];
      rw.ld = src_arr[sidx];
      rw.sidx = sidx;
    }
  };
  // (the choice between them is made here, a batch after the index load; row
  // lanes need no value: they read the first one rather than repeat the
  // column lanes' gather)
  auto load_val = [&](Raw& rw) { rw.val = vals[cols ? (perm ? rw.ld : rw.sidx) : 0u]; };
  // Operand addresses of this lane: row (lane & 15) of a row block, column
  // (lane & 15) / 2 of a column block and part (lane & 1) of the values.  The
  // two products of a step of eight visibilities take its even and odd ones:
  // lane group lane / 16 holds visibilities 2 (lane / 16) and the next.
  const int k2 = 2 * (lane >> 4);
  const float* pa = region + (lane & 15) * C::RS + k2;
  const float* pb = region + C::TAB_F + ((lane & 15) >> 1) * C::RS + k2;
  const float* pv = tval + (lane & 1) * C::BATCH + k2;
  // One batch: stage from rk (batch k), reload rk with batch k + 3 and the
  // value of rk2 (batch k + 2), then sum.
  auto batch = [&](int base, Raw& rk, Raw& rk2) {
    const bool valid = base + j < total;
    int lo = (cols ? cell_u(rk.cell) : cell_v(rk.cell)) - origin;
    if (periodic) lo = tile_base(lo, 0, g.M, W, wrap);
    const int hi = lo + W - 1;
    float w[W];
#pragma unroll
    for (int t = 0; t < W; ++t) w[t] = es_tap<W>(rk.off, t);
    // lanes past the end stage values of zero and reach no block
    const float vr = valid ? rk.val.x : 0.f;
    const float vi = valid ? __uint_as_float(__float_as_uint(rk.val.y) ^ (rk.cell & kFlip)) : 0.f;
    load_pre(rk, base + 3 * C::BATCH);
    load_val(rk2);
    // which of the batch's visibilities reach each block of 16 rows (lanes
    // 0-31) or 8 columns (lanes 32-63): lo <= last cell and hi >= first cell
    const int left = total - base;
    const unsigned live = left >= C::BATCH ? ~0u : (left > 0 ? (1u << left) - 1u : 0u);
    unsigned rows[2], cls[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned long long r =
          __builtin_amdgcn_ballot_w64((unsigned)(hi - q * bside) < (unsigned)(W - 1 + bside)) |
          (periodic && g.M == kTile ? ~0ull : 0ull);  // (one tile wide: taps wrap inside it)
      if (q < 2) rows[q] = (unsigned)r & live;
      cls[q] = (unsigned)(r >> 32) & live;
    }
    // taps inside the tile for the whole wave: constant strides
    const bool inside = __builtin_amdgcn_ballot_w64((unsigned)lo > (unsigned)(kTile - W)) == 0;
    auto stage = [&](auto value) {
      if (inside) {
        float* p = tab + lo * C::RS + j;
#pragma unroll
        for (int t = 0; t < W; ++t) p[t * C::RS] = value(t);
      } else {
        int l = lo;
        asm volatile("" : "+v"(l));  // this path's addresses are formed here, not ahead of the branch
#pragma unroll
        for (int t = 0; t < W; ++t) {
          unsigned r = (unsigned)(l + t);
          if (single) r &= kTile - 1;
          tab[(r < (unsigned)kTile ? r : (unsigned)kTile) * C::RS + j] = value(t);
        }
      }
    };
    stage([&](int t) { return w[t]; });
    if (cols) {
      tval[j] = vr;
      tval[C::BATCH + j] = vi;
    }
    lds_order();
#pragma unroll
    for (int st = 0; st < C::BATCH / 8; ++st) {
      const unsigned m = 0xffu << (8 * st);
      const unsigned r0 = rows[0] & m, r1 = rows[1] & m;
      const float2 a0 = *reinterpret_cast<const float2*>(pa + 8 * st);
      const float2 a1 = *reinterpret_cast<const float2*>(pa + 16 * C::RS + 8 * st);
      const float2 v = *reinterpret_cast<const float2*>(pv + 8 * st);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (cls[q] & m) {
          const float2 x = *reinterpret_cast<const float2*>(pb + 8 * q * C::RS + 8 * st);
          const float bx = x.x * v.x, by = x.y * v.y;
          if (r0) {
            acc[0][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.x, bx, acc[0][q], 0, 0, 0);
            acc[0][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.y, by, acc[0][q], 0, 0, 0);
          }
          if (r1) {
            acc[1][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.x, bx, acc[1][q], 0, 0, 0);
            acc[1][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.y, by, acc[1][q], 0, 0, 0);
          }
        }
    }
    lds_order();
    stage([&](int) { return 0.f; });
  };
  if (total > 0) {
    // (issued in the order of the loop's steady state)
    Raw rb0, rb1, rb2;
    load_pre(rb0, 0);
    load_pre(rb1, C::BATCH);
    {
      float4* t4 = reinterpret_cast<float4*>(region);
      for (int i = lane; i < C::WAVE_F / 4; i += 64) t4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    lds_order();
    load_val(rb0);
    load_pre(rb2, 2 * C::BATCH);
    load_val(rb1);
#pragma unroll 1
    for (int base = 0;; base += 3 * C::BATCH) {
      batch(base, rb0, rb2);
      if (base + C::BATCH >= total) break;
      batch(base + C::BATCH, rb1, rb0);
      if (base + 2 * C::BATCH >= total) break;
      batch(base + 2 * C::BATCH, rb2, rb1);
      if (base + 3 * C::BATCH >= total) break;
    }
    lds_order();
  }
  // accumulator r of block (rb, q) holds row 16 rb + 4 (lane / 16) + r, float
  // 16 q + lane % 16 of the tile row
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        region[(16 * rb + 4 * (lane >> 4) + r) * 2 * C::S + 16 * q + (lane & 15)] = acc[rb][q][r];
}

// Output address of a work item's tile: the band tile itself, or its
// partial slot.
__device__ __forceinline__ cpx<float>* spread_dst(const GridGeom& g, const SpreadChunk& ch,
                                                  cpx<float>* grid, cpx<float>* partials,
                                                  size_t& stride) {
  if (ch.slot < 0) {
    const int tv = ch.tile / g.ntu, tu = ch.tile - tv * g.ntu;
    stride = g.nu;
    return grid + (size_t)(tv * kTile) * g.nu + tu * kTile;
  }
  stride = kTile;
  return partials + (size_t)ch.slot * kTile * kTile;
}

// A workgroup of kSpreadQuad waves over as many work items (see
// SpreadChunk): each wave accumulates its item into its own LDS tile;
// independent items are written by their own wave, the shares of a combined
// tile are added in wave order and written once by the whole workgroup.
template <int W>
__device__ __forceinline__ void spread_quad_body(
    const GridGeom& g, const SpreadChunk* __restrict__ quad, const uint32_t* __restrict__ cell,
    const float* __restrict__ off, const cpx<float>* __restrict__ vals,
    const int32_t* __restrict__ perm, cpx<float>* __restrict__ grid,
    cpx<float>* __restrict__ partials) {
  using C = SpreadM;
  constexpr int WAVE_F = C::WAVE_F;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // (the wave's index as a scalar: its work item then sits in scalar registers)
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  float* region = reinterpret_cast<float*>(smem_raw);
  const SpreadChunk ch = quad[w];
  const bool combine = quad[0].combine != 0;  // the same for every wave
  if (ch.tile >= 0)
    spread_group_accumulate<W>(g, ch, cell, off, vals, perm, region + w * WAVE_F, lane);
  size_t stride;
  if (!combine) {
    if (ch.tile < 0) return;
    lds_order();
    cpx<float>* dst = spread_dst(g, ch, grid, partials, stride);
    const float4* t4 = reinterpret_cast<const float4*>(region + w * WAVE_F);
    for (int i = lane; i < kTile * kTile / 2; i += 64) {  // two cells per lane and step
      const int y = i / (kTile / 2), x2 = i - y * (kTile / 2);
      *reinterpret_cast<float4*>(dst + (size_t)y * stride + 2 * x2) = t4[(y * C::S) / 2 + x2];
    }
    return;
  }
  __syncthreads();
  cpx<float>* dst = spread_dst(g, quad[0], grid, partials, stride);
  for (int i = threadIdx.x; i < kTile * kTile / 2; i += 64 * kSpreadQuad) {
    const int y = i / (kTile / 2), x2 = i - y * (kTile / 2);
    const int o = (y * C::S) / 2 + x2;
    float4 v = reinterpret_cast<const float4*>(region)[o];
#pragma unroll
    for (int k = 1; k < kSpreadQuad; ++k) {
      const float4 t = reinterpret_cast<const float4*>(region + k * WAVE_F)[o];
      v.x += t.x;
      v.y += t.y;
      v.z += t.z;
      v.w += t.w;
    }
    *reinterpret_cast<float4*>(dst + (size_t)y * stride + 2 * x2) = v;
  }
}

// Element strides between the buffers of w-planes worked on together
// (blockIdx.y, or blockIdx.z of the fold, is the plane; one plane otherwise).
struct PlaneStride {
  size_t vals, grid, partials, H;
};

template <int W>
__global__ __launch_bounds__(64 * kSpreadQuad) void spread_quad_kernel(
    GridGeom g, const SpreadChunk* __restrict__ chunks, const uint32_t* __restrict__ cell,
    const float* __restrict__ off, const cpx<float>* __restrict__ vals,
    const int32_t* __restrict__ perm, cpx<float>* __restrict__ grid,
    cpx<float>* __restrict__ partials, unsigned long long* __restrict__ maxkey,
    PlaneStride ps) {
  // the image maximum that the last pass accumulates starts from zero
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *maxkey = 0ull;
  spread_quad_body<W>(g, chunks + (size_t)kSpreadQuad * blockIdx.x, cell, off,
                      vals + blockIdx.y * ps.vals, perm, grid + blockIdx.y * ps.grid,
                      partials + blockIdx.y * ps.partials);
}

// One launch over the workgroups of several plans: items[b] = (job, group).
template <int W>
__global__ __launch_bounds__(64 * kSpreadQuad) void spread_quad_batch_kernel(
    const AdjJob* __restrict__ jobs, const int2* __restrict__ items) {
  const int2 it = items[blockIdx.x];
  const AdjJob& J = jobs[it.x];
  if (it.y == 0 && threadIdx.x == 0) *J.maxkey = 0ull;  // every job has a group 0
  spread_quad_body<W>(J.g, J.chunks + (size_t)kSpreadQuad * it.y, J.cell, J.off, J.vals, J.perm,
                      J.grid, J.partials);
}

template <typename R, int W>
__global__ __launch_bounds__(64) void spread_kernel(
    GridGeom g, const SpreadChunk* __restrict__ chunks, const uint32_t* __restrict__ cell,
    const R* __restrict__ off, const cpx<R>* __restrict__ vals, const int32_t* __restrict__ perm,
    cpx<R>* __restrict__ grid, cpx<R>* __restrict__ partials,
    unsigned long long* __restrict__ maxkey) {
  // the image maximum that the last pass accumulates starts from zero (reset
  // here rather than by a launch of its own; the pass runs later on the stream)
  if (blockIdx.x == 0 && threadIdx.x == 0) *maxkey = 0ull;
  spread_body<R, W>(g, chunks[blockIdx.x], cell, off, vals, perm, grid, partials);
}

// Fold of a split tile: 64 cells per workgroup, kFoldSub threads per cell
// each summing every kFoldSub-th partial (kFoldBurst loads in flight), then the
// sub-sums are added in a fixed order (bitwise reproducible).
constexpr int kFoldSub = 8;
constexpr int kFoldBurst = 4;  // loads in flight per thread

template <typename R>
__device__ __forceinline__ void fold_body(const GridGeom& g, const FoldItem& it,
                                          const cpx<R>* __restrict__ partials,
                                          cpx<R>* __restrict__ grid) {
  __shared__ R sx[kFoldSub][64], sy[kFoldSub][64];
  const int c = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int i = blockIdx.y * 64 + c;
  const cpx<R>* src = partials + (size_t)it.first * kTile * kTile + i;
  R ax = 0, ay = 0;
  int q = sub;
  for (; q + (kFoldBurst - 1) * kFoldSub < it.count; q += kFoldBurst * kFoldSub) {
    cpx<R> v[kFoldBurst];
#pragma unroll
    for (int u = 0; u < kFoldBurst; ++u) v[u] = src[(size_t)(q + u * kFoldSub) * kTile * kTile];
#pragma unroll
    for (int u = 0; u < kFoldBurst; ++u) {
      ax += v[u].x;
      ay += v[u].y;
    }
  }
  for (; q < it.count; q += kFoldSub) {
    const cpx<R> v = src[(size_t)q * kTile * kTile];
    ax += v.x;
    ay += v.y;
  }
  sx[sub][c] = ax;
  sy[sub][c] = ay;
  __syncthreads();
  if (sub == 0) {
    R tx = 0, ty = 0;
#pragma unroll
    for (int k = 0; k < kFoldSub; ++k) {
      tx += sx[k][c];
      ty += sy[k][c];
    }
    const int tv = it.tile / g.ntu, tu = it.tile - tv * g.ntu;
    cpx<R>* dst = grid + (size_t)(tv * kTile) * g.nu + tu * kTile;
    const int y = i / kTile, x = i - y * kTile;
    dst[(size_t)y * g.nu + x] = {tx, ty};
  }
}

template <typename R>
__global__ __launch_bounds__(64 * kFoldSub) void fold_kernel(GridGeom g,
                                                           const FoldItem* __restrict__ items,
                                                           const cpx<R>* __restrict__ partials,
                                                           cpx<R>* __restrict__ grid,
                                                           PlaneStride ps) {
  fold_body<R>(g, items[blockIdx.x], partials + blockIdx.z * ps.partials,
               grid + blockIdx.z * ps.grid);
}

__global__ __launch_bounds__(64 * kFoldSub) void fold_batch_kernel(
    const AdjJob* __restrict__ jobs, const int2* __restrict__ items) {
  const int2 it = items[blockIdx.x];
  const AdjJob& J = jobs[it.x];
  fold_body<float>(J.g, J.fold[it.y], J.partials, J.grid);
}

// v exp(+2 pi i q / RAD) for a runtime q >= 0 and RAD = 2 or 4: half turns as
// sign changes, quarter turns as a swap of the parts plus sign changes, all
// as selects (the pruned first stage's outputs are band values rotated so).
// Exact; a zero v may come out as -0.
template <typename R, int RAD>
__device__ __forceinline__ cpx<R> turns_pos(cpx<R> v, int q) {
  static_assert(RAD == 2 || RAD == 4, "half or quarter turns");
  if constexpr (RAD == 2) {
    const bool neg = (q & 1) != 0;
    return {neg ? -v.x : v.x, neg ? -v.y : v.y};
  } else {
    q &= 3;
    const bool sw = (q & 1) != 0;
    const R a = sw ? v.y : v.x, b = sw ? v.x : v.y;
    const bool na = ((q + 1) & 2) != 0, nb = (q & 2) != 0;  // q = 1, 2 and q = 2, 3
    return {na ? -a : a, nb ? -b : b};
  }
}

// Pass-A output layout: columns grouped in blocks of KHB, each block stored
// row-major over the band rows; h_col is the element of a column at band row
// 0, its rows are KHB apart.  Columns 2k and 2k + 1 stay adjacent (pass B reads
// them together).  At the 16384 fine grid, whose pass A stores a thread's
// columns 4k, 4k + 1 and 4k + 2, 4k + 3 at different times, the pairs of each
// kind are grouped apart, so that neighbouring lanes fill a block's row at
// once (half-filled lines cost pass A 82 -> 115 us there).
constexpr int kSplitGrid = 16384;
template <int M>
constexpr int khb_for() {
  return M == kSplitGrid ? 4 : 8;
}
template <int M>
__device__ __forceinline__ size_t h_col(int col, int nv) {
  constexpr int KHB = khb_for<M>();
  const int c = M == kSplitGrid ? ((col >> 1) & 1) * (M / 4) + ((col >> 2) << 1) + (col & 1) : col;
  return (size_t)(c / KHB) * nv * KHB + (c % KHB);
}
template <int M>
__device__ __forceinline__ size_t h_index(int row, int col, int nv) {
  return h_col<M>(col, nv) + (size_t)row * khb_for<M>();
}

// Workgroups are dispatched to the 8 XCDs (each with its own L2) in turn:
// workgroup b runs on XCD b mod 8.  Renumbering so that each XCD receives a
// contiguous range of logical indices keeps neighbouring work (rows that
// share cache lines of the pass-A buffer) inside one L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_local(int b, int n) {
  const int q = n / kXcds, r = n % kXcds;
  const int x = b % kXcds, k = b / kXcds;
  return x < r ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

// Row masks (see RowMask): copied into LDS by the passes that test a row per
// element; the whole-row passes test their workgroup's rows once.  The pass
// kernels carry a MASKED flag only so that launches with a mask appear under
// their own symbols in traces: the code reads the mask pointer at run time in
// both, exactly as the batched passes do.
__device__ __forceinline__ bool row_set(const uint32_t* bits, int i) {
  return (bits[i >> 5] >> (i & 31)) & 1u;
}
template <int NB>
__device__ __forceinline__ bool any_row_set(const uint32_t* __restrict__ bits, int i0) {
  bool any = false;
#pragma unroll
  for (int b = 0; b < NB; ++b) any |= row_set(bits, i0 + b);
  return any;
}
template <int NT>
__device__ __forceinline__ void rows_to_lds(uint32_t* smask, const uint32_t* __restrict__ bits,
                                            int n) {
  if (bits)
    for (int i = threadIdx.x; i < (n + 31) / 32; i += NT) smask[i] = bits[i];
}

// Pass A of the adjoint: rows of the band grid (fixed v), FFT along u.
// Element m of a row sits at LDS position pidx(b M + m); a thread's elements
// are NT apart, so their positions advance by padded(NT).  The occupancy
// flags of the workgroup's tile rows are read once into LDS: tiles without
// data were never written and are read as zeros.
constexpr int kMaxTileCols = 512;  // fine grids up to 16384 cells per side
template <typename R, int M, int NB, int NT>
__device__ __forceinline__ void passA_adj_body(const GridGeom& g, const cpx<R>* __restrict__ grid,
                                               const uint8_t* __restrict__ tile_flags,
                                               cpx<R>* __restrict__ H,
                                               const cpx<R>* __restrict__ tw, int rowblock,
                                               const uint32_t* __restrict__ rows = nullptr) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<R>* buf = reinterpret_cast<cpx<R>*>(smem_raw);
  __shared__ cpx<R> tws[tw_count(M)];
  constexpr int TR = (NB + kTile - 1) / kTile + 1;  // tile rows a row block can touch
  __shared__ uint8_t sflag[TR][kMaxTileCols];
  __shared__ uint32_t smask[kMaxRowWords];
  rows_to_lds<NT>(smask, rows, g.n);
  constexpr int n = M / 2;
  const int row0 = rowblock * NB;
  const int tr0 = row0 / kTile;
  for (int i = threadIdx.x; i < TR * g.ntu; i += NT) {
    const int r = i / g.ntu, c = i - r * g.ntu;
    sflag[r][c] = (tr0 + r < g.ntv) ? tile_flags[(tr0 + r) * g.ntu + c] : 0;
  }
  load_twiddles<R, M, NT>(tws, tw);  // ends with a barrier
  static_assert((NB * M) % NT == 0 && NT % 16 == 0, "pass-A gather layout");
  // Input pruning as in pass B: with a first radix of 2 or 4 and a band no
  // wider than M / radix columns, the first stage is applied while loading.
  constexpr int RAD0 = first_radix(M);
  constexpr int NBF0 = M / RAD0;
  bool pruned = false;
  if constexpr (RAD0 <= 4) {
    if (g.nu <= NBF0) {  // uniform
      pruned = true;
      constexpr int ITJ = (NB * NBF0 + NT - 1) / NT;
      cpx<R> t[ITJ];
      int rr[ITJ];
#pragma unroll
      for (int it = 0; it < ITJ; ++it) {
        const int e = (int)threadIdx.x + it * NT;
        const int b = e / NBF0, j = e - b * NBF0;
        const int row = row0 + b;
        const int d = g.u0 - j;
        const int r = d > 0 ? (d + NBF0 - 1) / NBF0 : 0;  // first input at or past u0
        const int rel = j + r * NBF0 - g.u0;
        const bool ok = e < NB * NBF0 && row < g.nv && r < RAD0 && (unsigned)rel < (unsigned)g.nu &&
                        sflag[row / kTile - tr0][rel / kTile] != 0;
        const cpx<R> v = grid[ok ? (size_t)row * g.nu + rel : 0];
        t[it] = ok ? v : cpx<R>{R(0), R(0)};
        rr[it] = ok ? r : 0;
      }
#pragma unroll
      for (int it = 0; it < ITJ; ++it) {
        const int e = (int)threadIdx.x + it * NT;
        if ((NB * NBF0) % NT == 0 || e < NB * NBF0) {
          const int b = e / NBF0, j = e - b * NBF0;
#pragma unroll
          for (int s = 0; s < RAD0; ++s)
            buf[pidx(b * M + j * RAD0 + s)] = turns_pos<R, RAD0>(t[it], rr[it] * s);
        }
      }
    }
  }
  if (!pruned) {
    constexpr int IT = NB * M / NT;
    cpx<R> t[IT];
    bool ok[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int idx = (int)threadIdx.x + it * NT;
      const int b = idx / M, m = idx - b * M;
      const int row = row0 + b, rel = m - g.u0;
      ok[it] = row < g.nv && (unsigned)rel < (unsigned)g.nu &&
               sflag[row / kTile - tr0][rel / kTile] != 0;
      t[it] = grid[ok[it] ? (size_t)row * g.nu + rel : 0];
    }
    const int p0 = pidx((int)threadIdx.x);
#pragma unroll
    for (int it = 0; it < IT; ++it)
      buf[p0 + it * padded(NT)] = ok[it] ? t[it] : cpx<R>{R(0), R(0)};
  }
  __syncthreads();
  // the n central frequencies f in [-n/2, n/2) go to H column i = f + n/2,
  // stored from the last stage's registers
  auto keep = [](int, int f) { return 4 * f < M || 4 * f >= 3 * M; };
  // (with a row mask, only the columns of the image rows set)
  auto store = [&](int b, int f, cpx<R> v) {
    const int row = row0 + b;
    const int i = f < n / 2 ? f + n / 2 : f - M + n / 2;
    if (row < g.nv && (!rows || row_set(smask, i))) H[h_index<M>(row, i, g.nv)] = v;
  };
  // a last-stage butterfly j (outputs j + r M/16) keeps the columns
  // i = j + t M/16, t = 0..7: with a row mask, one whose eight columns are all
  // cleared is skipped whole
  auto need = [&](int j) {
    if (!rows) return true;
    bool any = false;
#pragma unroll
    for (int t = 0; t < 8; ++t) any |= row_set(smask, j + t * (M / 16));
    return any;
  };
  if constexpr (RAD0 <= 4) {
    if (pruned)
      lds_fft_store<R, M, NB, NT, +1, RAD0>(buf, tws, keep, store, need);
    else
      lds_fft_store<R, M, NB, NT, +1>(buf, tws, keep, store, need);
  } else {
    lds_fft_store<R, M, NB, NT, +1>(buf, tws, keep, store, need);
  }
}

template <typename R, int M, int NB, int NT, bool MASKED>
__global__ __launch_bounds__(NT) void passA_adj_kernel(GridGeom g, const cpx<R>* __restrict__ grid,
                                                        const uint8_t* __restrict__ tile_flags,
                                                        cpx<R>* __restrict__ H,
                                                        const cpx<R>* __restrict__ tw,
                                                        const uint32_t* __restrict__ rows,
                                                        PlaneStride ps) {
  passA_adj_body<R, M, NB, NT>(g, grid + blockIdx.y * ps.grid, tile_flags, H + blockIdx.y * ps.H,
                               tw, xcd_local(blockIdx.x, gridDim.x), rows);
}

// Pass A of the adjoint by register-held transforms (FP32, M = 4096 S): one
// band row per workgroup, the band within the window of 4096 slots centred on
// M / 2 (reg_window).  Outputs f = S t + s + 256 S k3 are the columns
// i = S t + s + 256 S q, q = (k3 + 4) mod 16 < 8; the S residues of a thread
// are adjacent columns, written two at a time.  Four workgroups share a compute
// unit, so that one's LDS exchanges run under another's arithmetic (the
// full-length transform's single 1024-thread workgroup alternated): 82 -> 72 us
// at 16384 (its bytes at the copy rate: 40), 78 -> 51 with a row mask; 31 -> 25 us
// at 8192, 17 -> 15 at 4096.
__host__ __device__ constexpr bool reg_window(int M, int lo, int hi) {  // slots [lo, hi)
  return M == kRegN ||
         (M > kRegN && M <= 4 * kRegN && lo >= M / 2 - kRegN / 2 && hi <= M / 2 + kRegN / 2);
}

template <int S>
__device__ __forceinline__ void passA_reg_body(const GridGeom& g, const c32* __restrict__ grid,
                                               const uint8_t* __restrict__ tile_flags,
                                               c32* __restrict__ H, const c32* __restrict__ tw,
                                               int row, const uint32_t* __restrict__ rows) {
  constexpr int M = kRegN * S;
  static_assert(S * kRegN == M && (S == 1 || S == 2 || S == 4), "register-held pass sizes");
  __shared__ c32 buf[kRegBuf];
  __shared__ c32 tws[tw_count(M)];
  __shared__ uint8_t sflag[kMaxTileCols];
  __shared__ uint32_t smask[kMaxRowWords];
  const int t = (int)threadIdx.x;
  rows_to_lds<kRegT>(smask, rows, g.n);
  for (int c = t; c < g.ntu; c += kRegT) sflag[c] = tile_flags[(row / kTile) * g.ntu + c];
  load_twiddles<float, M, kRegT>(tws, tw);  // ends with a barrier
  c32 x[16];
  bool ok[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int c = t + kRegT * r;
    const int rel = (S == 1 ? c : M / 2 + (r < 8 ? c : c - kRegN)) - g.u0;
    ok[r] = (unsigned)rel < (unsigned)g.nu && sflag[rel / kTile] != 0;
    x[r] = grid[ok[r] ? (size_t)row * g.nu + rel : 0];
  }
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (!ok[r]) x[r] = {0.f, 0.f};
  constexpr int KHB = khb_for<M>();
  auto set = [&](int i) { return !rows || row_set(smask, i); };
  if constexpr (S == 1) {
    c32 y[16];
    reg_fft<1, 0, +1>(x, y, buf, tws);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int i = t + kRegT * q;
      if (set(i)) H[h_index<M>(row, i, g.nv)] = y[(q + 12) & 15];
    }
  } else {
    auto pair = [&](auto s0) {
      c32 y0[16], y1[16];
      if constexpr (s0 > 0) __syncthreads();
      reg_fft<S, s0, +1>(x, y0, buf, tws);
      __syncthreads();
      reg_fft<S, s0 + 1, +1>(x, y1, buf, tws);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int i = S * (t + kRegT * q) + s0, k3 = (q + 12) & 15;
        c32* h = H + h_index<M>(row, i, g.nv);  // columns i, i + 1: 16 bytes
        if (!rows)
          *reinterpret_cast<cpair<float>*>(h) = cpair<float>{y0[k3], y1[k3]};
        else {
          if (row_set(smask, i)) h[0] = y0[k3];
          if (row_set(smask, i + 1)) h[1] = y1[k3];
        }
      }
    };
    pair(std::integral_constant<int, 0>{});
    if constexpr (S == 4) pair(std::integral_constant<int, 2>{});
  }
}

template <int S, bool MASKED>
__global__ __launch_bounds__(kRegT, 4) void passA_adj_reg_kernel(
    GridGeom g, const c32* __restrict__ grid, const uint8_t* __restrict__ tile_flags,
    c32* __restrict__ H, const c32* __restrict__ tw, const uint32_t* __restrict__ rows,
    PlaneStride ps) {
  passA_reg_body<S>(g, grid + blockIdx.y * ps.grid, tile_flags, H + blockIdx.y * ps.H, tw,
                    xcd_local(blockIdx.x, gridDim.x), rows);
}

template <int S>
__global__ __launch_bounds__(kRegT, 4) void passA_reg_batch_kernel(const AdjJob* __restrict__ jobs,
                                                                   const int2* __restrict__ items) {
  const int2 it = items[xcd_local(blockIdx.x, gridDim.x)];
  const AdjJob& J = jobs[it.x];
  passA_reg_body<S>(J.g, J.grid, J.flags, J.H, J.tw, it.y, J.rows);
}

template <int M, int NB, int NT>
__global__ __launch_bounds__(NT) void passA_batch_kernel(const AdjJob* __restrict__ jobs,
                                                          const int2* __restrict__ items) {
  const int2 it = items[xcd_local(blockIdx.x, gridDim.x)];
  const AdjJob& J = jobs[it.x];
  passA_adj_body<float, M, NB, NT>(J.g, J.grid, J.flags, J.H, J.tw, it.y, J.rows);
}

__device__ __forceinline__ unsigned long long max_key(float a, int idx) {
  return ((unsigned long long)__float_as_uint(a) << 32) | (unsigned long long)(0xffffffffu - (unsigned)idx);
}

// Consecutive w-planes of the w-stacked adjoint: the position of the first,
// the spacing, the phase reference c_mid, their number, the stride of their
// pass-A buffers, and whether the first of them is the first of all (which
// writes instead of adding).
struct WPlane {
  double w0, dw, cmid;
  int first, count;
  size_t H;
};

template <typename R, int M, int NB, int NT>
__device__ __forceinline__ void passB_adj_w_plane(const GridGeom& g, const cpx<R>* __restrict__ H,
                                                  R* __restrict__ image, cpx<R>* buf,
                                                  const cpx<R>* tws, const R* __restrict__ corr,
                                                  R scale, int i0, double wj, double cmid,
                                                  bool first) {
  constexpr int n = M / 2;
  // element (m, b): band row m - v0 of column i0 + b of the pass-A buffer,
  // whose KHB-wide column blocks are row-major over the band rows
  static_assert((NB & (NB - 1)) == 0 && NT % NB == 0, "pass-B layout");
  constexpr int IT = (NB * M + NT - 1) / NT;
  constexpr int MSTEP = NT / NB;  // a thread's m advances by this per element
  const int b = (int)threadIdx.x & (NB - 1), m0 = (int)threadIdx.x / NB;
  const int col = i0 + b;
  constexpr int KHB = khb_for<M>();
  const cpx<R>* hcol = H + h_col<M>(col, g.nv);
  // Input pruning: with a first radix of 2 or 4 and a band no longer than
  // M / radix, each first-stage butterfly (inputs j + r M / radix) holds at
  // most one band row, so the stage is applied while loading: output s of
  // butterfly j is that row rotated by r s quarter (or half) turns, exactly
  // what the full stage computes.  The remaining stages follow as usual.
  constexpr int RAD0 = first_radix(M);
  constexpr int NBF0 = M / RAD0;
  bool pruned = false;
  if constexpr (RAD0 <= 4) {
    if (g.nv <= NBF0) {  // uniform
      pruned = true;
      constexpr int ITJ = (NBF0 + MSTEP - 1) / MSTEP;
      cpx<R> t[ITJ];
      int rr[ITJ];
#pragma unroll
      for (int it = 0; it < ITJ; ++it) {
        const int j = m0 + it * MSTEP;
        const int d = g.v0 - j;
        const int r = d > 0 ? (d + NBF0 - 1) / NBF0 : 0;  // first input at or past v0
        const int rel = j + r * NBF0 - g.v0;
        const bool ok = j < NBF0 && r < RAD0 && (unsigned)rel < (unsigned)g.nv;
        const cpx<R> v = hcol[ok ? (size_t)rel * KHB : 0];
        t[it] = ok ? v : cpx<R>{R(0), R(0)};
        rr[it] = ok ? r : 0;
      }
#pragma unroll
      for (int it = 0; it < ITJ; ++it) {
        const int j = m0 + it * MSTEP;
        if (NBF0 % MSTEP == 0 || j < NBF0) {
#pragma unroll
          for (int s = 0; s < RAD0; ++s)
            buf[pidx(b * M + j * RAD0 + s)] = turns_pos<R, RAD0>(t[it], rr[it] * s);
        }
      }
    }
  }
  if (!pruned) {
    cpx<R> t[IT];
    bool ok[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int m = m0 + it * MSTEP;
      const int rel = m - g.v0;
      ok[it] = m < M && (unsigned)rel < (unsigned)g.nv;
      t[it] = hcol[ok[it] ? (size_t)rel * KHB : 0];
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int m = m0 + it * MSTEP;
      if ((NB * M) % NT == 0 || m < M) buf[pidx(b * M + m)] = ok[it] ? t[it] : cpx<R>{R(0), R(0)};
    }
  }
  __syncthreads();
  const R dl = (R)g.dl;
  // pixel (i, j) from frequency f = j - n/2 (mod M) of column i, stored from
  // the last stage's registers: Re(exp(2 pi i w_j c') v), c' = n - 1 - c_mid,
  // phase in FP64
  auto keep = [](int, int f) { return 4 * f < M || 4 * f >= 3 * M; };
  auto store = [&](int bb, int f, cpx<R> v) {
    const int i = i0 + bb;
    const int j = f < n / 2 ? f + n / 2 : f - M + n / 2;
    const R l = (R)(i - n / 2) * dl, mm = (R)(j - n / 2) * dl;
    const R inv_n = __builtin_amdgcn_rsqf(R(1) - l * l - mm * mm);
    double th = wj * (n_minus_one((double)(i - n / 2) * g.dl, (double)(j - n / 2) * g.dl) -
                         cmid);
    th -= rint(th);
    const R sn = (R)__builtin_amdgcn_sinf((float)th), cs = (R)__builtin_amdgcn_cosf((float)th);
    const R val = (v.x * cs - v.y * sn) * (corr[i] * scale) * corr[j] * inv_n;
    R* dst = image + (size_t)i * n + j;
    *dst = first ? val : *dst + val;
  };
  if constexpr (RAD0 <= 4) {
    if (pruned)
      lds_fft_store<R, M, NB, NT, +1, RAD0>(buf, tws, keep, store);
    else
      lds_fft_store<R, M, NB, NT, +1>(buf, tws, keep, store);
  } else {
    lds_fft_store<R, M, NB, NT, +1>(buf, tws, keep, store);
  }
}

// Pass B of w-planes: NB image rows i; for each plane in order, FFT along v of
// H[:, i] (the whole plane: the rotation makes the transform's outputs
// complex), correction, rotation by the plane's phase, and the real part added
// into the image rows in memory (each pixel read and written per plane, by the
// same thread each time).
template <typename R, int M, int NB, int NT>
__device__ __forceinline__ void passB_adj_w_body(const GridGeom& g, const cpx<R>* __restrict__ H,
                                                 R* __restrict__ image,
                                                 const cpx<R>* __restrict__ tw,
                                                 const R* __restrict__ corr, R scale, int iblock,
                                                 WPlane wp) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<R>* buf = reinterpret_cast<cpx<R>*>(smem_raw);
  __shared__ cpx<R> tws[tw_count(M)];
  constexpr int n = M / 2;
  const int i0 = iblock * NB;
  load_twiddles<R, M, NT>(tws, tw);
  for (int plane = 0; plane < wp.count; ++plane) {
    if (plane > 0) __syncthreads();  // the last plane's reads of the buffer
    passB_adj_w_plane<R, M, NB, NT>(g, H + plane * wp.H, image, buf, tws, corr, scale, i0,
                                    wp.w0 + plane * wp.dw, wp.cmid, wp.first && plane == 0);
  }
}

// Pass-B workgroups whose transforms (of `total` elements) have few radix-16
// butterflies: their pixels go through LDS, one per thread and step.  From a
// butterfly's registers a few lanes would handle 16 pixels each of both rows,
// one after the other, and that chain is what such a launch waits for.
// Adjoint at fine grids 128, 256 and 512: 6.5, 6.9 and 7.2 -> 5.5, 5.6 and 6.3
// us; forward at 128 and 256: 4.9 and 6.4 -> 4.1 and 4.5 (8.0 -> 4.8 with cold
// caches), and no faster at 512.
constexpr bool few_butterflies(bool adjoint, int total) {
  return total / 16 < (adjoint ? 64 : 32);
}

// Pass B of the adjoint (coplanar plans): NB pairs of image rows; FFT along v
// of each pair's completed column; correction; both image rows written; fused
// max |eta| (max(eta, 0) with ``positive``, the positivity-constrained solve)
// with lowest-index ties.
template <typename R, int M, int NB, int NT>
__device__ __forceinline__ void passB_adj_body(const GridGeom& g, const cpx<R>* __restrict__ H,
                                               R* __restrict__ image,
                                               const cpx<R>* __restrict__ tw,
                                               const R* __restrict__ corr, R scale,
                                               unsigned long long* __restrict__ maxkey,
                                               int positive, int iblock,
                                               const uint32_t* __restrict__ rows = nullptr) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<R>* buf = reinterpret_cast<cpx<R>*>(smem_raw);
  __shared__ cpx<R> tws[tw_count(M)];
  constexpr int n = M / 2;
  const int i0 = iblock * NB * 2;
  // with a row mask: workgroups without a row set return at once, the others
  // store only their rows that are set
  static_assert(NB <= 8, "row bits");
  unsigned rowbits = (1u << (2 * NB)) - 1u;
  if (rows) {
    rowbits = 0;
#pragma unroll
    for (int b = 0; b < 2 * NB; ++b) rowbits |= (unsigned)row_set(rows, i0 + b) << b;
    if (rowbits == 0) return;  // the whole workgroup
  }
  load_twiddles<R, M, NT>(tws, tw);
  // slot m of pair b, whose KHB-wide column blocks are row-major over the
  // band rows
  static_assert((NB & (NB - 1)) == 0 && NT % NB == 0, "pass-B layout");
  constexpr int IT = (NB * M + NT - 1) / NT;
  constexpr int MSTEP = NT / NB;  // a thread's m advances by this per element
  const int b = (int)threadIdx.x & (NB - 1), m0 = (int)threadIdx.x / NB;
  const int col = i0 + 2 * b;
  constexpr int KHB = khb_for<M>();
  const cpx<R>* hcol = H + h_col<M>(col, g.nv);
  auto load = [&](int rel) {
    return *reinterpret_cast<const cpair<R>*>(hcol + (size_t)rel * KHB);
  };
  const PairGeom q{M, g.v0, g.nv};
  // Input pruning: the completed column occupies the slots within E of M/2;
  // with a first radix of 2 or 4 and those no more than M / radix, each
  // first-stage butterfly (inputs j + r M / radix) holds at most one, so the
  // stage is applied while loading: output s of butterfly j is that value
  // rotated by r s quarter (or half) turns, exactly what the full stage
  // computes.  The remaining stages follow as usual.
  constexpr int RAD0 = first_radix(M);
  constexpr int NBF0 = M / RAD0;
  const int E = g.v0 + g.nv - 1 - M / 2 > M / 2 - g.v0 ? g.v0 + g.nv - 1 - M / 2 : M / 2 - g.v0;
  bool pruned = false;
  if constexpr (RAD0 <= 4) {
    if (2 * E + 1 <= NBF0) {  // uniform
      pruned = true;
      constexpr int ITJ = (NBF0 + MSTEP - 1) / MSTEP;
      cpair<R> t[ITJ];
      int cc[ITJ];  // the slot, or -1
      auto slot = [&](int j) {
        const int d = M / 2 - E - j;
        const int r = d > 0 ? (d + NBF0 - 1) / NBF0 : 0;  // first input in the support
        return (j < NBF0 && r < RAD0 && j + r * NBF0 <= M / 2 + E) ? j + r * NBF0 : -1;
      };
#pragma unroll
      for (int it = 0; it < ITJ; ++it) {
        const int c = slot(m0 + it * MSTEP);
        bool conj, ok;
        const int rel = pair_main(q, c < 0 ? 0 : c, conj, ok);
        ok = ok && c >= 0;
        t[it] = load(ok ? rel : 0);
        cc[it] = ok ? c : -1;
      }
#pragma unroll
      for (int it = 0; it < ITJ; ++it) {
        const int j = m0 + it * MSTEP;
        if (NBF0 % MSTEP == 0 || j < NBF0) {
          cpx<R> z{R(0), R(0)};
          if (cc[it] >= 0) {
            z = pair_z<R>(t[it], 2 * cc[it] < M);
            if (pair_edge(q, cc[it])) {
              const cpx<R> e = pair_rest<R>(q, cc[it], load);
              z = {z.x + e.x, z.y + e.y};
            }
          }
          const int r = cc[it] >= 0 ? cc[it] / NBF0 : 0;
#pragma unroll
          for (int s = 0; s < RAD0; ++s)
            buf[pidx(b * M + j * RAD0 + s)] = turns_pos<R, RAD0>(z, r * s);
        }
      }
    }
  }
  if (!pruned) {
    cpair<R> t[IT];
    bool ok[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int m = m0 + it * MSTEP;
      bool conj;
      const int rel = pair_main(q, m < M ? m : 0, conj, ok[it]);
      ok[it] = ok[it] && m < M;
      t[it] = load(ok[it] ? rel : 0);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int m = m0 + it * MSTEP;
      if ((NB * M) % NT == 0 || m < M) {
        cpx<R> z{R(0), R(0)};
        if (ok[it]) z = pair_z<R>(t[it], 2 * m < M);
        if (pair_edge(q, m)) {
          const cpx<R> e = pair_rest<R>(q, m, load);
          z = {z.x + e.x, z.y + e.y};
        }
        buf[pidx(b * M + m)] = z;
      }
    }
  }
  __syncthreads();
  unsigned long long best = 0;
  const R dl = (R)g.dl;
  // pixels (i, j) and (i + 1, j) from frequency f = j - n/2 (mod M) of the
  // pair, stored from the last stage's registers with the correction (and the
  // completion's 1/2) and the max key
  auto keep = [](int, int f) { return 4 * f < M || 4 * f >= 3 * M; };
  auto store = [&](int bb, int f, cpx<R> v) {
    const int j = f < n / 2 ? f + n / 2 : f - M + n / 2;
    const R mm = (R)(j - n / 2) * dl;
    const R cj = corr[j];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!((rowbits >> (2 * bb + h)) & 1u)) continue;
      const int i = i0 + 2 * bb + h;
      const R l = (R)(i - n / 2) * dl;
      R inv_n;
      if constexpr (sizeof(R) == 4) {
        inv_n = __builtin_amdgcn_rsqf(R(1) - l * l - mm * mm);
      } else {
        inv_n = R(1) / sqrt(R(1) - l * l - mm * mm);
      }
      const R val = (h ? v.y : v.x) * (corr[i] * (R(0.5) * scale)) * cj * inv_n;
      image[(size_t)i * n + j] = val;
      // positive part: +0 for every val <= 0 (never -0, whose bits would win)
      const float kv = positive ? (val > R(0) ? (float)val : 0.0f) : (float)fabs(val);
      const unsigned long long key = max_key(kv, i * n + j);
      best = key > best ? key : best;
    }
  };
  auto finish = [&](auto ns) {
    if constexpr (few_butterflies(true, NB * M)) {
      fft_stages<R, M, NB, NT, +1, ns>(buf, tws);  // ends with a barrier
      for (int e = (int)threadIdx.x; e < NB * n; e += NT) {
        const int bb = e / n, f = (e - bb * n - n / 2) & (M - 1);
        store(bb, f, buf[pidx(bb * M + f)]);
      }
    } else {
      lds_fft_store<R, M, NB, NT, +1, ns>(buf, tws, keep, store);
    }
  };
  if constexpr (RAD0 <= 4) {
    if (pruned)
      finish(std::integral_constant<int, RAD0>{});
    else
      finish(std::integral_constant<int, 1>{});
  } else {
    finish(std::integral_constant<int, 1>{});
  }
  // block max
  for (int o = 32; o > 0; o >>= 1) {
    unsigned long long other = __shfl_xor(best, o, 64);
    best = other > best ? other : best;
  }
  __shared__ unsigned long long wbest[NT / 64];
  __syncthreads();
  if ((threadIdx.x & 63) == 0) wbest[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0 && maxkey) {
    unsigned long long m = 0;
    for (int w = 0; w < NT / 64; ++w) m = wbest[w] > m ? wbest[w] : m;
    atomicMax(maxkey, m);
  }
}

template <typename R, int M, int NB, int NT, bool MASKED>
__global__ __launch_bounds__(NT) void passB_adj_kernel(GridGeom g, const cpx<R>* __restrict__ H,
                                                        R* __restrict__ image,
                                                        const cpx<R>* __restrict__ tw,
                                                        const R* __restrict__ corr, R scale,
                                                        unsigned long long* __restrict__ maxkey,
                                                        int positive,
                                                        const uint32_t* __restrict__ rows) {
  passB_adj_body<R, M, NB, NT>(g, H, image, tw, corr, scale, maxkey, positive,
                               xcd_local(blockIdx.x, gridDim.x), rows);
}

// Adjacent pixels of a caller's image, at a float's alignment.
typedef float image2 __attribute__((ext_vector_type(2), aligned(4)));
typedef float image4 __attribute__((ext_vector_type(4), aligned(4)));

// Pass B of the adjoint by register-held transforms (FP32, M = 4096 S): one
// pair of image rows per workgroup, the completed column within the window of
// 4096 slots centred on M / 2.  Thread t holds the pixels j = S t + s + 256 S q
// (q < 8), stored two adjacent ones at a time, or four at 16384, where two pairs
// stored apart left the L2 as half lines (523 MB written for 268): 231 -> 178 us
// there, and 136 in fours (its bytes at the copy rate: 85); 55 -> 42 at 8192,
// 33 -> 28 at 4096; bound by the transforms' arithmetic.
template <int S>
__device__ __forceinline__ void passB_reg_body(const GridGeom& g, const c32* __restrict__ H,
                                               float* __restrict__ image,
                                               const c32* __restrict__ tw,
                                               const float* __restrict__ corr, float scale,
                                               unsigned long long* __restrict__ maxkey,
                                               int positive, int pairno,
                                               const uint32_t* __restrict__ rows) {
  constexpr int M = kRegN * S, n = M / 2;
  __shared__ c32 buf[kRegBuf];
  __shared__ c32 tws[tw_count(M)];
  const int t = (int)threadIdx.x, i0 = 2 * pairno;
  // with a row mask: pairs without a row set return at once, the others
  // store only their rows that are set
  const bool set0 = !rows || row_set(rows, i0), set1 = !rows || row_set(rows, i0 + 1);
  if (!set0 && !set1) return;  // the whole workgroup
  load_twiddles<float, M, kRegT>(tws, tw);
  constexpr int KHB = khb_for<M>();
  const c32* hcol = H + h_col<M>(i0, g.nv);
  auto load = [&](int rel) {
    return *reinterpret_cast<const cpair<float>*>(hcol + (size_t)rel * KHB);
  };
  const PairGeom pg{M, g.v0, g.nv};
  c32 x[16];
  {
    cpair<float> h[16];
    auto cell = [&](int r) {  // the slot's cell in [0, M)
      const int c = t + kRegT * r;
      return S == 1 ? c : M / 2 + (r < 8 ? c : c - kRegN);
    };
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      bool conj, ok;
      const int rel = pair_main(pg, cell(r), conj, ok);
      h[r] = load(ok ? rel : 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      bool conj, ok;
      pair_main(pg, cell(r), conj, ok);
      x[r] = pair_z<float>(h[r], conj);
      if (!ok) x[r] = {0.f, 0.f};
      if (pair_edge(pg, cell(r))) {
        const c32 e = pair_rest<float>(pg, cell(r), load);
        x[r] = {x[r].x + e.x, x[r].y + e.y};
      }
    }
  }
  // the largest |eta| (by its bits, so that a NaN wins) of each row and its j,
  // lowest on ties: pixels come in ascending j within a residue pair
  unsigned best[2];
  int at[2];
  auto begin = [&](int s0) {  // (an all-zero row reports its first pixel)
    best[0] = best[1] = 0u;
    at[0] = at[1] = S * t + s0;
  };
  unsigned long long key = 0;
  const float dl = (float)g.dl;
  const float l0 = (float)(i0 - n / 2) * dl, l1 = (float)(i0 + 1 - n / 2) * dl;
  const float ci0 = corr[i0] * (0.5f * scale), ci1 = corr[i0 + 1] * (0.5f * scale);
  auto pixel = [&](c32 v, int j, float cj, float& p0, float& p1) {
    const float mm = (float)(j - n / 2) * dl;
    p0 = v.x * ci0 * cj * __builtin_amdgcn_rsqf(1.0f - l0 * l0 - mm * mm);
    p1 = v.y * ci1 * cj * __builtin_amdgcn_rsqf(1.0f - l1 * l1 - mm * mm);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float p = h ? p1 : p0;
      // positive part: +0 for every value <= 0 (never -0, whose bits would win)
      const unsigned b = __float_as_uint(positive ? (p > 0.f ? p : 0.0f) : fabsf(p));
      const bool up = b > best[h];
      best[h] = up ? b : best[h];
      at[h] = up ? j : at[h];
    }
  };
  auto fold = [&]() {  // the rows' maxima so far into the key (only rows stored count)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned long long k = max_key(__uint_as_float(best[h]), (i0 + h) * n + at[h]);
      if ((h ? set1 : set0) && k > key) key = k;
    }
  };
  float* row0 = image + (size_t)i0 * n;
  float* row1 = row0 + n;
  if constexpr (S == 1) {
    c32 y[16];
    reg_fft<1, 0, +1>(x, y, buf, tws);
    begin(0);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = t + kRegT * q;
      float p0, p1;
      pixel(y[(q + 12) & 15], j, corr[j], p0, p1);
      if (set0) row0[j] = p0;
      if (set1) row1[j] = p1;
    }
    fold();
  } else {
    float2 e0[8], e1[8];  // S = 4: the first two pixels of four, until all are formed
    auto pair = [&](auto s0) {
      c32 y0[16], y1[16];
      if constexpr (s0 > 0) __syncthreads();
      reg_fft<S, s0, +1>(x, y0, buf, tws);
      __syncthreads();
      reg_fft<S, s0 + 1, +1>(x, y1, buf, tws);
      begin(s0);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int j = S * (t + kRegT * q) + s0, k3 = (q + 12) & 15;
        const float2 cj = *reinterpret_cast<const float2*>(corr + j);
        float2 p0, p1;
        pixel(y0[k3], j, cj.x, p0.x, p1.x);
        pixel(y1[k3], j + 1, cj.y, p0.y, p1.y);
        if constexpr (S == 2) {
          if (set0) *reinterpret_cast<image2*>(row0 + j) = image2{p0.x, p0.y};
          if (set1) *reinterpret_cast<image2*>(row1 + j) = image2{p1.x, p1.y};
        } else if constexpr (s0 == 0) {
          e0[q] = p0;
          e1[q] = p1;
        } else {
          if (set0)
            *reinterpret_cast<image4*>(row0 + j - 2) = image4{e0[q].x, e0[q].y, p0.x, p0.y};
          if (set1)
            *reinterpret_cast<image4*>(row1 + j - 2) = image4{e1[q].x, e1[q].y, p1.x, p1.y};
        }
      }
      fold();
    };
    pair(std::integral_constant<int, 0>{});
    if constexpr (S == 4) pair(std::integral_constant<int, 2>{});
  }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(key, o, 64);
    key = other > key ? other : key;
  }
  __shared__ unsigned long long wbest[kRegT / 64];
  if ((t & 63) == 0) wbest[t >> 6] = key;
  __syncthreads();
  if (t == 0 && maxkey) {
    unsigned long long m = 0;
    for (int w = 0; w < kRegT / 64; ++w) m = wbest[w] > m ? wbest[w] : m;
    atomicMax(maxkey, m);
  }
}

template <int S, bool MASKED>
__global__ __launch_bounds__(kRegT, S == 4 ? 3 : 4) void passB_adj_reg_kernel(
    GridGeom g, const c32* __restrict__ H, float* __restrict__ image, const c32* __restrict__ tw,
    const float* __restrict__ corr, float scale, unsigned long long* __restrict__ maxkey,
    int positive, const uint32_t* __restrict__ rows) {
  passB_reg_body<S>(g, H, image, tw, corr, scale, maxkey, positive,
                    xcd_local(blockIdx.x, gridDim.x), rows);
}

template <int S>
__global__ __launch_bounds__(kRegT, S == 4 ? 3 : 4) void passB_reg_batch_kernel(const AdjJob* __restrict__ jobs,
                                                                   const int2* __restrict__ items) {
  const int2 it = items[xcd_local(blockIdx.x, gridDim.x)];
  const AdjJob& J = jobs[it.x];
  passB_reg_body<S>(J.g, J.H, J.image, J.tw, J.corr, J.scale, J.maxkey, J.positive, it.y, J.rows);
}

template <typename R, int M, int NB, int NT>
__global__ __launch_bounds__(NT) void passB_adj_w_kernel(GridGeom g, const cpx<R>* __restrict__ H,
                                                          R* __restrict__ image,
                                                          const cpx<R>* __restrict__ tw,
                                                          const R* __restrict__ corr, R scale,
                                                          WPlane wp) {
  passB_adj_w_body<R, M, NB, NT>(g, H, image, tw, corr, scale,
                                 xcd_local(blockIdx.x, gridDim.x), wp);
}

// Visibility weights of the w-planes w_j = w0 + j dw, j < count (plan order):
// h_k exp(2 pi i w_k c_mid) psi((w_k - w_j) / dw) within the kernel's reach
// |w_k - w_j| <= (W/2) dw, zero beyond it; a visibility with w_k < 0 enters as
// its conjugate at -w_k (the plan grids it at (-u, -v)).  perm: NULL when h is
// in plan order.  One thread forms a visibility's values for every plane:
// its w and value are read once per group (5 -> 1.6 us per plane at 424,800
// visibilities).
__global__ __launch_bounds__(256) void wplane_kernel(int64_t L, const double* __restrict__ Cw,
                                                     const cpx<float>* __restrict__ h,
                                                     const int32_t* __restrict__ perm, WPlane wp,
                                                     double inv_dw, float R2, float inv_R, float c,
                                                     cpx<float>* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= L) return;
  const double wk = fabs(Cw[k]);
  const float t0 = (float)((wk - wp.w0) * inv_dw);
  cpx<float> v{0.f, 0.f};
  // (a margin for the rounding of the plane's own distance below)
  const float reach = __builtin_amdgcn_sqrtf(R2) + 1e-3f;
  if (t0 >= -reach && t0 <= (float)(wp.count - 1) + reach) {
    const cpx<float> x = h[perm ? perm[k] : k];
    const float y = Cw[k] < 0.0 ? -x.y : x.y;
    double ph = wk * wp.cmid;
    ph -= rint(ph);
    const float sn = __builtin_amdgcn_sinf((float)ph), cs = __builtin_amdgcn_cosf((float)ph);
    v = {x.x * cs - y * sn, x.x * sn + y * cs};
  }
  for (int j = 0; j < wp.count; ++j) {
    const float t = (float)((wk - (wp.w0 + j * wp.dw)) * inv_dw);
    cpx<float> o{0.f, 0.f};
    if (t * t <= R2) {
      const float z = t * inv_R;
      const float psi = es_from_q(fmaf(-z, z, 1.0f), c);
      o = {psi * v.x, psi * v.y};
    }
    out[(size_t)j * L + k] = o;
  }
}

// Last step of the w-stacked adjoint: image /= Psi(dw c') per pixel, and
// the fused maximum key.  Psi(xi) = sum_q W w_q phi(z_q) cos(pi W z_q xi)
// (the quadrature of the kernel's Fourier integral) is evaluated as its
// Chebyshev series in 4 xi (xi = dw (c' - c_mid) lies in [-1/4, 1/4]):
// cheb[k], k < kPsiCheb, by Clenshaw's recurrence in FP64.
__global__ __launch_bounds__(256) void wfinal_kernel(GridGeom g, WStack ws,
                                                     const double* __restrict__ cheb,
                                                     float* __restrict__ image,
                                                     unsigned long long* __restrict__ maxkey,
                                                     int positive) {
  // a grid-stride loop over a capped grid: one atomic per workgroup on the
  // single key, so few workgroups (thousands contending for one address
  // took most of the kernel's time)
  const int n = g.n;
  unsigned long long best = 0;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < (int64_t)n * n;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(idx / n), j = (int)(idx - (int64_t)i * n);
    const double xi =
        ws.dw * (n_minus_one((double)(i - n / 2) * g.dl, (double)(j - n / 2) * g.dl) - ws.cmid);
    const double x = fmin(fmax(4.0 * xi, -1.0), 1.0);
    double b1 = 0.0, b2 = 0.0;
#pragma unroll
    for (int k = kPsiCheb - 1; k >= 1; --k) {
      const double b0 = fma(2.0 * x, b1, cheb[k] - b2);
      b2 = b1;
      b1 = b0;
    }
    const double psi = fma(x, b1, cheb[0] - b2);
    const float val = (float)((double)image[idx] / psi);
    image[idx] = val;
    const float kv = positive ? (val > 0.f ? val : 0.0f) : fabsf(val);
    const unsigned long long key = max_key(kv, (int)idx);
    best = key > best ? key : best;
  }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o, 64);
    best = other > best ? other : best;
  }
  __shared__ unsigned long long wbest[4];
  if ((threadIdx.x & 63) == 0) wbest[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long m = 0;
    for (int w = 0; w < 4; ++w) m = wbest[w] > m ? wbest[w] : m;
    atomicMax(maxkey, m);
  }
}

template <int M, int NB, int NT>
__global__ __launch_bounds__(NT) void passB_batch_kernel(const AdjJob* __restrict__ jobs,
                                                          const int2* __restrict__ items) {
  const int2 it = items[xcd_local(blockIdx.x, gridDim.x)];
  const AdjJob& J = jobs[it.x];
  passB_adj_body<float, M, NB, NT>(J.g, J.H, J.image, J.tw, J.corr, J.scale, J.maxkey,
                                   J.positive, it.y, J.rows);
}

// First stage of a forward transform whose input is the n = M/2 central
// frequencies of each sequence (slot m holds frequency m for m < M/4 and
// m - M for m >= 3M/4; the slots between are zero), applied while loading.
// Butterfly j of the first stage (radix RAD0, inputs j + r M/RAD0) then has
// fixed nonzero inputs: for RAD0 >= 4 the r < RAD0/4 and r >= 3 RAD0/4, for
// RAD0 = 2 exactly one (r = 0 when j < M/4, else r = 1).  load(b, c) returns
// the value at central index c = f + n/2 of sequence b; outputs go where the
// full stage writes them (b M + j RAD0 + s).  All loads of a thread are issued
// before the first is used.
template <typename R, int M, int NB, int NT, int SIGN, typename Load>
__device__ __forceinline__ void central_first_stage(cpx<R>* buf, Load load) {
  constexpr int RAD0 = first_radix(M);
  constexpr int NBF0 = M / RAD0;
  constexpr int TOT = NB * NBF0;
  constexpr int IT = (TOT + NT - 1) / NT;
  constexpr int NZ = RAD0 >= 4 ? RAD0 / 2 : 1;  // nonzero inputs per butterfly
  static_assert(M >= 32, "central first stage layout");
  cpx<R> t[IT][NZ];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int e = (int)threadIdx.x + it * NT;
    const int ee = (TOT % NT == 0 || e < TOT) ? e : 0;  // a valid element for spare lanes
    const int b = ee / NBF0, j = ee - b * NBF0;
    if constexpr (RAD0 == 2) {
      t[it][0] = load(b, j < M / 4 ? j + M / 4 : j - M / 4);
    } else {
#pragma unroll
      for (int q = 0; q < NZ; ++q) {
        const int r = q < RAD0 / 4 ? q : q + RAD0 / 2;   // r in [0, RAD0/4) u [3 RAD0/4, RAD0)
        const int m = j + r * NBF0;
        t[it][q] = load(b, r < RAD0 / 4 ? m + M / 4 : m - 3 * (M / 4));
      }
    }
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int e = (int)threadIdx.x + it * NT;
    if (TOT % NT == 0 || e < TOT) {
      const int b = e / NBF0, j = e - b * NBF0;
      const int p0 = b * M + j * RAD0;
      if constexpr (RAD0 == 2) {
        const cpx<R> v = t[it][0];
        buf[pidx(p0)] = v;
        buf[pidx(p0 + 1)] = j < M / 4 ? v : cpx<R>{-v.x, -v.y};
      } else if constexpr (RAD0 == 4) {
        // X_s = x_0 + x_3 w^(3 s)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const cpx<R> u = rot<R, 4, SIGN>(t[it][1], (3 * s) & 3);
          buf[pidx(p0 + s)] = {t[it][0].x + u.x, t[it][0].y + u.y};
        }
      } else {
        cpx<R> x[RAD0];
#pragma unroll
        for (int r = 0; r < RAD0; ++r) x[r] = {R(0), R(0)};
#pragma unroll
        for (int q = 0; q < NZ; ++q) x[q < RAD0 / 4 ? q : q + RAD0 / 2] = t[it][q];
        dft<R, RAD0, SIGN>(x);
#pragma unroll
        for (int s = 0; s < RAD0; ++s) buf[pidx(p0 + s)] = x[s];
      }
    }
  }
}

// Forward pass B^T: NB pairs of image rows, pre-correct, FFT along v (sign
// -1), keep the band rows: H[v_rel][i] (the pass-A layout).  The rows 2k and
// 2k + 1 of the real image are the real and imaginary parts of one sequence
// (see pair_main); its transform Z is taken apart as H_2k(c) =
// (Z(c) + conj Z(-c)) / 2 and H_2k+1(c) = (Z(c) - conj Z(-c)) / 2i at the band
// cells c.  The first stage is applied while loading (a row's n pixels are
// the central frequencies).
template <typename R, int M, int NB, int NT>
__device__ __forceinline__ void passB_fwd_body(const GridGeom& g, const R* __restrict__ image,
                                               cpx<R>* __restrict__ H,
                                               const cpx<R>* __restrict__ tw,
                                               const R* __restrict__ corr, int iblock,
                                               const uint32_t* __restrict__ rows) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<R>* buf = reinterpret_cast<cpx<R>*>(smem_raw);
  __shared__ cpx<R> tws[tw_count(M)];
  constexpr int n = M / 2;
  const int i0 = iblock * NB * 2;
  // with a row mask, workgroups of zero rows write nothing (pass A reads
  // those columns of H as zeros), and the rows cleared are not read
  if (rows && !any_row_set<2 * NB>(rows, i0)) return;
  const R dl = (R)g.dl;
  auto pixel = [&](int b, int j) -> cpx<R> {
    R x[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = i0 + 2 * b + h;
      const R l = (R)(i - n / 2) * dl, mm = (R)(j - n / 2) * dl;
      R inv_n;
      if constexpr (sizeof(R) == 4) {
        inv_n = __builtin_amdgcn_rsqf(R(1) - l * l - mm * mm);
      } else {
        inv_n = R(1) / sqrt(R(1) - l * l - mm * mm);
      }
      x[h] = (!rows || row_set(rows, i)) ? image[(size_t)i * n + j] * corr[i] * corr[j] * inv_n
                                         : R(0);
    }
    return {x[0], x[1]};
  };
  if constexpr (few_butterflies(false, NB * M)) {
    for (int e = (int)threadIdx.x; e < NB * M; e += NT) {
      const int b = e / M, m = e - b * M, j = (m + n / 2) & (M - 1);  // (0 <= j < n: a pixel)
      buf[pidx(e)] = j < n ? pixel(b, j) : cpx<R>{R(0), R(0)};
    }
    load_twiddles<R, M, NT>(tws, tw);  // ends with a barrier
    fft_stages<R, M, NB, NT, -1, 1>(buf, tws);  // the same
  } else {
    load_twiddles<R, M, NT>(tws, tw);
    central_first_stage<R, M, NB, NT, -1>(buf, pixel);
    __syncthreads();
    fft_stages<R, M, NB, NT, -1, first_radix(M)>(buf, tws);  // ends with a barrier
  }
  constexpr int KHB = khb_for<M>();
  const int v0 = g.v0, nv = g.nv;
  for (int e = (int)threadIdx.x; e < NB * nv; e += NT) {
    const int b = e & (NB - 1), rel = e / NB;
    const int c = v0 + rel;
    const cpx<R> z = buf[pidx(b * M + (c & (M - 1)))];
    const cpx<R> w = buf[pidx(b * M + ((M - c) & (M - 1)))];
    *reinterpret_cast<cpair<R>*>(H + h_index<M>(rel, i0 + 2 * b, nv)) =
        cpair<R>{{R(0.5) * (z.x + w.x), R(0.5) * (z.y - w.y)},
                 {R(0.5) * (z.y + w.y), R(0.5) * (w.x - z.x)}};
  }
}

template <typename R, int M, int NB, int NT, bool MASKED>
__global__ __launch_bounds__(NT) void passB_fwd_kernel(GridGeom g, const R* __restrict__ image,
                                                        cpx<R>* __restrict__ H,
                                                        const cpx<R>* __restrict__ tw,
                                                        const R* __restrict__ corr,
                                                        const uint32_t* __restrict__ rows) {
  passB_fwd_body<R, M, NB, NT>(g, image, H, tw, corr, xcd_local(blockIdx.x, gridDim.x), rows);
}

// Forward pass A^T: NB band rows v; FFT along u (sign -1) of H[v][:] placed
// at the n central frequencies (first stage applied while loading); the band
// columns stored from the last stage's registers.
template <typename R, int M, int NB, int NT, bool MASKED>
__global__ __launch_bounds__(NT) void passA_fwd_kernel(GridGeom g, const cpx<R>* __restrict__ H,
                                                        cpx<R>* __restrict__ grid,
                                                        const cpx<R>* __restrict__ tw,
                                                        const uint32_t* __restrict__ rows) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cpx<R>* buf = reinterpret_cast<cpx<R>*>(smem_raw);
  __shared__ cpx<R> tws[tw_count(M)];
  __shared__ uint32_t smask[kMaxRowWords];
  rows_to_lds<NT>(smask, rows, g.n);
  load_twiddles<R, M, NT>(tws, tw);  // (its barrier also covers the mask)
  const int row0 = xcd_local(blockIdx.x, gridDim.x) * NB;
  constexpr int KHB = khb_for<M>();
  const int nv = g.nv;
  central_first_stage<R, M, NB, NT, -1>(buf, [&](int b, int c) -> cpx<R> {
    const int row = row0 + b;
    // H column c is image row c: zero, and not read, when the mask clears it;
    // rows past the band (last workgroup) read row 0 and are never stored
    if (rows && !row_set(smask, c)) return {R(0), R(0)};
    return H[h_index<M>(row < nv ? row : 0, c, nv)];
  });
  __syncthreads();
  const int u0 = g.u0, nu = g.nu;
  auto keep = [&](int, int f) { return (unsigned)(f - u0) < (unsigned)nu; };
  auto store = [&](int b, int f, cpx<R> v) {
    const int row = row0 + b;
    if (row < nv) grid[(size_t)row * nu + (f - u0)] = v;
  };
  lds_fft_store<R, M, NB, NT, -1, first_radix(M)>(buf, tws, keep, store);
}

// The forward passes by register-held transforms (FP32, M = 4096 S), for the
// bands of the adjoint's: pass B^T one pair of image rows per workgroup, its
// completed spectrum taken apart through LDS; pass A^T one band row.
template <int S, int E, typename Load>  // E residues at a time; x[e][q]: residue
__device__ __forceinline__ void reg_central_all(  // s0 + e of k + 1024 = t + 256 q
    c32 (&acc)[16], c32* __restrict__ buf, const c32* __restrict__ tws, Load load) {
  auto group = [&](auto s0) {
    c32 x[E][8];
    load(x, (int)s0);
    if constexpr (s0 > 0) __syncthreads();
    reg_fft_central<S, s0, -1>(x[0], acc, buf, tws);
    if constexpr (E == 2) {
      __syncthreads();
      reg_fft_central<S, s0 + 1, -1>(x[1], acc, buf, tws);
    }
  };
  group(std::integral_constant<int, 0>{});
  if constexpr (S > 1 && E == 1) group(std::integral_constant<int, 1>{});
  if constexpr (S == 4) group(std::integral_constant<int, 2>{});
  if constexpr (S == 4 && E == 1) group(std::integral_constant<int, 3>{});
}

template <int S, bool MASKED>
__global__ __launch_bounds__(kRegT, 4) void passB_fwd_reg_kernel(
    GridGeom g, const float* __restrict__ image, c32* __restrict__ H, const c32* __restrict__ tw,
    const float* __restrict__ corr, const uint32_t* __restrict__ rows) {
  constexpr int M = kRegN * S, n = M / 2;
  __shared__ c32 buf[kRegBuf];
  __shared__ c32 tws[tw_count(M)];
  const int t = (int)threadIdx.x, i0 = 2 * xcd_local(blockIdx.x, gridDim.x);
  // with a row mask, pairs of zero rows write nothing (pass A reads those
  // columns of H as zeros), and the rows cleared are not read
  const bool set0 = !rows || row_set(rows, i0), set1 = !rows || row_set(rows, i0 + 1);
  if (!set0 && !set1) return;  // the whole workgroup
  load_twiddles<float, M, kRegT>(tws, tw);
  const float dl = (float)g.dl;
  const float l0 = (float)(i0 - n / 2) * dl, l1 = (float)(i0 + 1 - n / 2) * dl;
  const float c0 = corr[i0], c1 = corr[i0 + 1];
  const float* row0 = image + (size_t)i0 * n;
  const float* row1 = row0 + n;
  auto two = [](const float* at) {
    const image2 v = *reinterpret_cast<const image2*>(at);
    return float2{v.x, v.y};
  };
  auto pixel = [&](float a, float b, float cj, int j) {
    const float mm = (float)(j - n / 2) * dl;
    return c32{a * c0 * cj * __builtin_amdgcn_rsqf(1.0f - l0 * l0 - mm * mm),
               b * c1 * cj * __builtin_amdgcn_rsqf(1.0f - l1 * l1 - mm * mm)};
  };
  c32 acc[16];
  constexpr int E = S == 1 ? 1 : 2;
  reg_central_all<S, E>(acc, buf, tws, [&](c32 (&x)[E][8], int s0) {
    float2 a[8], b[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = S * (t + kRegT * q) + s0;
      a[q] = b[q] = make_float2(0.f, 0.f);
      if constexpr (S == 1) {
        if (set0) a[q].x = row0[j];
        if (set1) b[q].x = row1[j];
      } else {
        if (set0) a[q] = two(row0 + j);
        if (set1) b[q] = two(row1 + j);
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = S * (t + kRegT * q) + s0;
      x[0][q] = pixel(a[q].x, b[q].x, corr[j], j);
      if constexpr (S > 1) x[1][q] = pixel(a[q].y, b[q].y, corr[j + 1], j + 1);
    }
  });
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) buf[pidx(t + kRegT * k)] = acc[k];
  __syncthreads();
  c32* hcol = H + h_col<M>(i0, g.nv);
  for (int rel = t; rel < g.nv; rel += kRegT) {
    const int c = g.v0 + rel;
    const c32 z = buf[pidx(c & (kRegN - 1))], w = buf[pidx(-c & (kRegN - 1))];
    *reinterpret_cast<cpair<float>*>(hcol + (size_t)rel * khb_for<M>()) =
        cpair<float>{{0.5f * (z.x + w.x), 0.5f * (z.y - w.y)},
                     {0.5f * (z.y + w.y), 0.5f * (w.x - z.x)}};
  }
}

template <int S, bool MASKED>
__global__ __launch_bounds__(kRegT, 4) void passA_fwd_reg_kernel(
    GridGeom g, const c32* __restrict__ H, c32* __restrict__ grid, const c32* __restrict__ tw,
    const uint32_t* __restrict__ rows) {
  constexpr int M = kRegN * S;
  __shared__ c32 buf[kRegBuf];
  __shared__ c32 tws[tw_count(M)];
  __shared__ uint32_t smask[kMaxRowWords];
  rows_to_lds<kRegT>(smask, rows, g.n);
  load_twiddles<float, M, kRegT>(tws, tw);  // (its barrier also covers the mask)
  const int t = (int)threadIdx.x, row = xcd_local(blockIdx.x, gridDim.x), nv = g.nv;
  // H column i is image row i: zero, and not read, when the mask clears it
  auto set = [&](int i) { return !rows || row_set(smask, i); };
  c32 acc[16];
  reg_central_all<S, 1>(acc, buf, tws, [&](c32 (&x)[1][8], int s0) {
    // columns 256 S apart are a constant stride apart.  One residue at a time,
    // and (opaque) its loads behind the transforms of the one before: more in
    // flight leaves too few registers.
    const c32* col = H;
    asm volatile("" : "+s"(col));
    const size_t lane = h_index<M>(row, S * t + s0, nv), step = (size_t)(S == 1 ? 256 : 512) * nv;
    bool ok[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      ok[q] = set(S * (t + kRegT * q) + s0);
      x[0][q] = col[ok[q] ? lane + q * step : 0];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (!ok[q]) x[0][q] = {0.f, 0.f};
  });
  const int u0 = g.u0, nu = g.nu;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int c = t + kRegT * k;
    const int rel = (S == 1 ? c : M / 2 + (k < 8 ? c : c - kRegN)) - u0;
    if ((unsigned)rel < (unsigned)nu) grid[(size_t)row * nu + rel] = acc[k];
  }
}

// Interpolation: V_k = sum of w x w taps of the fine grid (type-2 gather).
// Coplanar plans only, whose band never wraps along v.
template <typename R, int W>
__global__ __launch_bounds__(256) void interp_kernel(GridGeom g, int64_t L,
                                                     const uint32_t* __restrict__ cell,
                                                     const R* __restrict__ off,
                                                     const cpx<R>* __restrict__ grid,
                                                     const int32_t* __restrict__ perm,
                                                     cpx<R>* __restrict__ out) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= L) return;
  const uint32_t c = cell[s];
  const int cu = cell_u(c), cv = cell_v(c);
  const R su = off[2 * s], sv = off[2 * s + 1];
  const R inv = R(2) / R(W);
  const R beta = g.beta64;
  R ku[W];
#pragma unroll
  for (int t = 0; t < W; ++t) ku[t] = es_kernel((su + R(t)) * inv, beta);
  R ax = 0, ay = 0;
  // rows: not fully unrolled (W^2 loads in flight would exhaust registers for
  // wide kernels); the row weight is evaluated in the loop
#pragma unroll 2
  for (int a = 0; a < W; ++a) {
    const R kva = es_kernel((sv + R(a)) * inv, beta);
    const int y = cv + a - g.v0;
    R rx = 0, ry = 0;
#pragma unroll
    for (int b = 0; b < W; ++b) {
      int x = cu + b - g.u0;
      if (g.wrap && x >= g.M) x -= g.M;
      const cpx<R> v = grid[(size_t)y * g.nu + x];
      rx += v.x * ku[b];
      ry += v.y * ku[b];
    }
    ax += rx * kva;
    ay += ry * kva;
  }
  const int64_t d = perm ? perm[s] : s;
  out[d] = {ax, c & kFlip ? -ay : ay};
}

// Interpolation from LDS (FP32, kernel widths up to 16): one workgroup of
// kInterpThreads per work item (InterpItem), a plan-order range of
// visibilities whose first cells lie in one tile.  The workgroup copies the
// tile and the W - 1 cells past its right and lower edges, all that its
// visibilities' footprints reach, into LDS (cells outside the band as zeros;
// with a periodic band, wrapped), then each thread sums the W x W taps of one
// visibility at a time from there, rows of taps in the same order as
// interp_kernel.  With base (plan-order output), the output is base - Phi x:
// the residual, in the same FP32 subtraction a separate pass would do.  base is
// in plan order, or with base_perm in caller order: the gather is a load per
// visibility issued ahead of its taps.  It is bound by its random 64-byte
// sectors all the same: 8,372,224 visibilities take 75 us without it and 189
// with it, 35 less than with a pass of its own.  With stats as well, each work item also writes its sums of
// |r|^2 and Re(conj(base) r) in FP64 to stats[2 item], [2 item + 1] (threads
// combined in a fixed order).
constexpr int kInterpThreads = 256;
template <int W>
struct InterpCfg {
  static constexpr int S = kTile + W - 1;  // region side (cells)
  static constexpr int SP = S | 1;         // row stride (odd)
};

template <int W>
__global__ __launch_bounds__(kInterpThreads) void interp_lds_kernel(GridGeom g,
                                                        const InterpItem* __restrict__ items,
                                                        const uint32_t* __restrict__ cell,
                                                        const float* __restrict__ off,
                                                        const c32* __restrict__ grid,
                                                        const int32_t* __restrict__ perm,
                                                        const c32* __restrict__ base,
                                                        const int32_t* __restrict__ base_perm,
                                                        c32* __restrict__ out,
                                                        double* __restrict__ stats) {
  using C = InterpCfg<W>;
  __shared__ float2 reg[C::S * C::SP];
  const InterpItem it = items[blockIdx.x];
  const int tid = (int)threadIdx.x;
  const int tv = it.tile / g.ntu, tu = it.tile - tv * g.ntu;
  const int rv0 = tv * kTile, ru0 = tu * kTile;  // region origin in the band
  for (int e = tid; e < C::S * C::S; e += kInterpThreads) {
    const int y = e / C::S, x = e - y * C::S;
    const int rv = rv0 + y;
    int ru = ru0 + x;
    float2 v = make_float2(0.f, 0.f);
    if (g.wrap && ru >= g.M) ru -= g.M;
    if (rv < g.nv && ru < g.nu) {
      const c32 c = grid[(size_t)rv * g.nu + ru];
      v = make_float2(c.x, c.y);
    }
    reg[y * C::SP + x] = v;
  }
  __syncthreads();
  const int ou = g.u0 + ru0, ov = g.v0 + rv0;
  double r2 = 0.0, vr = 0.0;
  // a caller-order base's source index one visibility ahead of its use
  int src = base_perm && it.beg + tid < it.end ? base_perm[it.beg + tid] : 0;
  for (int sidx = it.beg + tid; sidx < it.end; sidx += kInterpThreads) {
    const uint32_t c = cell[sidx];
    c32 v{0.f, 0.f};
    if (base) v = base[base_perm ? src : sidx];
    if (base_perm && sidx + kInterpThreads < it.end) src = base_perm[sidx + kInterpThreads];
    const int x = cell_u(c) - ou, y = cell_v(c) - ov;  // in [0, kTile)
    const float2 o = reinterpret_cast<const float2*>(off)[sidx];
    float ku[W];
#pragma unroll
    for (int t = 0; t < W; ++t) ku[t] = es_tap<W>(o.x, t);
    float ax = 0.f, ay = 0.f;
    const float2* rp = reg + y * C::SP + x;
#pragma unroll
    for (int a = 0; a < W; ++a) {
      const float kva = es_tap<W>(o.y, a);
      float rx = 0.f, ry = 0.f;
#pragma unroll
      for (int b = 0; b < W; ++b) {
        const float2 v = rp[a * C::SP + b];
        rx += v.x * ku[b];
        ry += v.y * ku[b];
      }
      ax += rx * kva;
      ay += ry * kva;
    }
    ay = __uint_as_float(__float_as_uint(ay) ^ (c & kFlip));  // conjugate if flipped
    if (base) {
      const c32 r = {v.x - ax, v.y - ay};
      out[sidx] = r;
      r2 += (double)r.x * r.x + (double)r.y * r.y;
      vr += (double)v.x * r.x + (double)v.y * r.y;
    } else {
      out[perm ? perm[sidx] : sidx] = {ax, ay};
    }
  }
  if (stats) {
    constexpr int NW = kInterpThreads / 64;
    __shared__ double wsum[2][NW];
    for (int o = 32; o > 0; o >>= 1) {
      r2 += __shfl_xor(r2, o, 64);
      vr += __shfl_xor(vr, o, 64);
    }
    if ((tid & 63) == 0) {
      wsum[0][tid >> 6] = r2;
      wsum[1][tid >> 6] = vr;
    }
    __syncthreads();
    if (tid == 0) {
      double a = 0.0, b = 0.0;
      for (int w = 0; w < NW; ++w) {
        a += wsum[0][w];
        b += wsum[1][w];
      }
      stats[2 * (size_t)blockIdx.x] = a;
      stats[2 * (size_t)blockIdx.x + 1] = b;
    }
  }
}

// Pass B evaluated directly for an active set (the APGD's gridded
// operators).  Its atoms lie on few image rows, a row holding one or two, so
// instead of a length-M transform per row the needed values are sums over
// the atoms or over the band rows with phases e^{-/+2 pi i f q / M} (f = j -
// n/2 the atom's centred column, q = v0 + band row), the product f q reduced
// mod M exactly in integers and the angle (in turns, |t| <= 1/2) taken by the
// hardware sine and cosine.  The apodisation and 1/n factors are applied in
// the order the transform's loading (forward) and epilogue (adjoint) apply
// them.
__device__ __forceinline__ float turns_mod(int f, int q, int M) {
  int t = (f * q) & (M - 1);  // f q mod M (two's complement), f q < 2^31
  if (t >= M / 2) t -= M;
  return (float)t / (float)M;  // exact: M is a power of two
}

__device__ __forceinline__ float inv_n_f32(const GridGeom& g, int i, int j) {
  const float dl = (float)g.dl;
  const float l = (float)(i - g.n / 2) * dl, mm = (float)(j - g.n / 2) * dl;
  return __builtin_amdgcn_rsqf(1.0f - l * l - mm * mm);
}

// Forward: H[band row][i] = sum over the atoms of row i of c e^{-2 pi i f q / M}
// for each occupied row i (rowlist: row, first atom, end), atoms sorted by
// pixel with FP64 weights w.
template <int M>
__global__ __launch_bounds__(256) void rows_fwd_direct_kernel(GridGeom g,
                                                              const int3* __restrict__ rowlist,
                                                              const int32_t* __restrict__ pix,
                                                              const double* __restrict__ w,
                                                              const float* __restrict__ corr,
                                                              c32* __restrict__ H) {
  const int3 rl = rowlist[blockIdx.y];
  const int i = rl.x, n = g.n;
  for (int rel = (int)(blockIdx.x * blockDim.x + threadIdx.x); rel < g.nv;
       rel += (int)(gridDim.x * blockDim.x)) {
    const int q = g.v0 + rel;
    float hx = 0.f, hy = 0.f;
    for (int a = rl.y; a < rl.z; ++a) {
      const int j = pix[a] - i * n;
      const float c = (float)w[a] * corr[i] * corr[j] * inv_n_f32(g, i, j);
      const float tt = turns_mod(j - n / 2, q, g.M);
      hx += c * __builtin_amdgcn_cosf(tt);
      hy -= c * __builtin_amdgcn_sinf(tt);
    }
    H[h_index<M>(rel, i, g.nv)] = {hx, hy};
  }
}

// Adjoint at the atoms: one 256-thread workgroup per atom, g = Re(sum over
// band rows of H[band row][i] e^{+2 pi i f q / M}) times the corrections, in
// FP64 out (thread sums combined in a fixed order).
template <int M>
__global__ __launch_bounds__(256) void atoms_adj_direct_kernel(GridGeom g,
                                                               const int32_t* __restrict__ pix,
                                                               const c32* __restrict__ H,
                                                               const float* __restrict__ corr,
                                                               double* __restrict__ gout) {
  const int a = (int)blockIdx.x, t = (int)threadIdx.x;
  const int pp = pix[a], n = g.n;
  const int i = pp / n, j = pp - i * n;
  float acc = 0.f;
  for (int rel = t; rel < g.nv; rel += 256) {
    const float tt = turns_mod(j - n / 2, g.v0 + rel, g.M);
    const c32 h = H[h_index<M>(rel, i, g.nv)];
    acc += h.x * __builtin_amdgcn_cosf(tt) - h.y * __builtin_amdgcn_sinf(tt);
  }
  double d = acc;
  for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
  __shared__ double wsum[4];
  if ((t & 63) == 0) wsum[t >> 6] = d;
  __syncthreads();
  if (t == 0) {
    const double sum = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
    const float v = (float)sum * corr[i] * corr[j] * inv_n_f32(g, i, j);
    gout[a] = (double)v;
  }
}

// ----------------------------------------------------------------------------
// Host launchers
// ----------------------------------------------------------------------------
// Algorithmic bytes of one spread: each visibility's value and its two
// sub-cell offsets read once (4 reals), each band cell written once.
static double spread_bytes(const pc_plan* p, double rb) {
  return p->L * 4.0 * rb + 2.0 * rb * p->g.nu * p->g.nv;
}

static PlaneStride plane_stride(const pc_plan* p) {
  const GridGeom& g = p->g;
  return PlaneStride{(size_t)p->L, (size_t)g.nu * g.nv, (size_t)p->n_partials * kTile * kTile,
                     (size_t)g.nv * g.n};
}

template <typename R, int W>
static void launch_spread_w(pc_plan* p, const cpx<R>* vals, const int32_t* perm, hipStream_t s,
                            int planes) {
  const double rb = sizeof(R);
  ProfScope ps(p, s, "spread", planes * spread_bytes(p, rb), planes * (double)p->L);
  if constexpr (sizeof(R) == 4) {
    if (!p->spread_quads) fail(PC_ERR_DEVICE, "spread: the plan's work list is not grouped");
    constexpr size_t lds = SpreadM::lds_bytes;
    static_assert(lds <= 64 * 1024, "grouped spread LDS budget");
    hipLaunchKernelGGL((spread_quad_kernel<W>), dim3((unsigned)(p->n_chunks / kSpreadQuad), (unsigned)planes),
                       dim3(64 * kSpreadQuad), lds, s, p->g, p->chunks, p->cell,
                       (const float*)p->off, vals, perm, (c32*)p->grid, (c32*)p->partials,
                       p->maxkey, plane_stride(p));
  } else {
    constexpr size_t lds = SpreadCfg<R, W>::lds_bytes;
    static_assert(lds <= 160 * 1024, "spread LDS budget");
    if (p->spread_quads) fail(PC_ERR_DEVICE, "spread: the plan's work list is grouped");
    if (lds > 64 * 1024)
      PC_HIP(hipFuncSetAttribute((const void*)spread_kernel<R, W>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((spread_kernel<R, W>), dim3((unsigned)p->n_chunks), dim3(64), lds, s, p->g,
                       p->chunks, p->cell, (const R*)p->off, vals, perm, (cpx<R>*)p->grid,
                       (cpx<R>*)p->partials, p->maxkey);
  }
  PC_LAUNCH_CHECK("spread");
}

template <typename R>
static void launch_spread(pc_plan* p, const cpx<R>* vals, const int32_t* perm, hipStream_t s,
                          int planes = 1) {
  switch (p->g.W) {
#define PC_W(w) \
  case w:       \
    launch_spread_w<R, w>(p, vals, perm, s, planes); \
    break;
    PC_W(2) PC_W(3) PC_W(4) PC_W(5) PC_W(6) PC_W(7) PC_W(8) PC_W(9) PC_W(10) PC_W(11) PC_W(12)
    PC_W(13) PC_W(14) PC_W(15) PC_W(16)
#undef PC_W
    default:
      fail(PC_ERR_UNSUPPORTED, "kernel width");
  }
  if (p->n_fold > 0) {
    const double tb = 2.0 * sizeof(R) * kTile * kTile;
    ProfScope ps(p, s, "fold", planes * tb * (p->n_partials + p->n_fold),
                 planes * (double)p->n_partials);
    hipLaunchKernelGGL((fold_kernel<R>),
                       dim3((unsigned)p->n_fold, kTile * kTile / 64, (unsigned)planes),
                       dim3(64 * kFoldSub), 0, s, p->g, p->fold,
                       (const cpx<R>*)p->partials, (cpx<R>*)p->grid, plane_stride(p));
    PC_LAUNCH_CHECK("fold");
  }
}

template <typename R, int W>
static void launch_interp_w(pc_plan* p, const int32_t* perm, cpx<R>* out, hipStream_t s,
                            const cpx<R>* base, const int32_t* base_perm, double* stats) {
  const double rb = sizeof(R);
  ProfScope ps(p, s, "interp", p->L * (4 + 4 * rb + (base ? 2 * rb : 0)) +
                                   2 * rb * p->g.nu * p->g.nv, (double)p->L);
  if constexpr (sizeof(R) == 4) {
    hipLaunchKernelGGL((interp_lds_kernel<W>), dim3((unsigned)p->n_interp), dim3(kInterpThreads),
                       0, s, p->g,
                       p->interp, p->cell, (const float*)p->off, (const c32*)p->grid, perm,
                       (const c32*)base, base_perm, (c32*)out, base ? stats : nullptr);
  } else {
    if (base) fail(PC_ERR_UNSUPPORTED, "FP64 interpolation with a base");
    const unsigned nb = (unsigned)((p->L + 255) / 256);
    hipLaunchKernelGGL((interp_kernel<R, W>), dim3(nb), dim3(256), 0, s, p->g, p->L, p->cell,
                       (const R*)p->off, (const cpx<R>*)p->grid, perm, out);
  }
  PC_LAUNCH_CHECK("interp");
}

template <typename R>
static void launch_interp(pc_plan* p, const int32_t* perm, cpx<R>* out, hipStream_t s,
                          const cpx<R>* base = nullptr, const int32_t* base_perm = nullptr,
                          double* stats = nullptr) {
  switch (p->g.W) {
#define PC_W(w) \
  case w:       \
    launch_interp_w<R, w>(p, perm, out, s, base, base_perm, stats); \
    break;
    PC_W(2) PC_W(3) PC_W(4) PC_W(5) PC_W(6) PC_W(7) PC_W(8) PC_W(9) PC_W(10) PC_W(11) PC_W(12)
    PC_W(13) PC_W(14) PC_W(15) PC_W(16)
#undef PC_W
    default:
      fail(PC_ERR_UNSUPPORTED, "kernel width");
  }
}

// Launch shapes per fine-grid size: NB sequences per workgroup, NT threads.
// Pass A keeps about 64 KB (FP32) of LDS per workgroup; pass B up to 128 KB.
template <typename R>
struct Shapes {
  static constexpr int lds_a = 64 * 1024;
  static constexpr int lds_b = 64 * 1024;
};

static void set_lds(const void* kernel, size_t bytes) {
  if (bytes > 64 * 1024)
    PC_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
}

// Sequences per pass-B workgroup (pairs of image rows; single rows for a
// w-plane): so many that a launch has >= 256 workgroups, capped by the LDS
// budget.
template <typename R, int M, int ROWS = 2>
constexpr int nb_passB() {
  constexpr int CB = sizeof(cpx<R>);
  constexpr int lim = (M * CB >= Shapes<R>::lds_b) ? 1 : Shapes<R>::lds_b / (M * CB);
  constexpr int want = (M / 2) / ROWS / 256 < 1 ? 1 : (M / 2) / ROWS / 256;
  return want < lim ? want : lim;
}

template <int TOTAL_BUTTERFLIES>
constexpr int nt_for() {
  return TOTAL_BUTTERFLIES >= 1024 ? 1024 : (TOTAL_BUTTERFLIES >= 512 ? 512 : 256);
}

// The register-held passes take FP32 plans of fine grids 4096 ... 16384 whose
// band (pass A), or completed column (pass B), fits their window; wider bands
// and the other sizes go through the full-length LDS transforms.
constexpr bool reg_size(int M) { return M == kRegN || M == 2 * kRegN || M == 4 * kRegN; }
// Fine grid 4096 fits its window whole: FP32 plans need no other passes there.
template <typename R, int M>
constexpr bool reg_always = sizeof(R) == 4 && M == kRegN;
static bool reg_passA(const GridGeom& g) {
  return reg_size(g.M) && reg_window(g.M, g.u0, g.u0 + g.nu);
}
static bool reg_passB(const GridGeom& g) {
  const int hi = g.v0 + g.nv;  // cells [v0, hi) and their mirror images M - c
  const int lo = std::min(g.v0, g.M + 1 - hi);
  return reg_size(g.M) && reg_window(g.M, lo, g.M + 1 - lo);
}

template <typename R, int M>
static void run_passes_adj(pc_plan* p, R* image, R scale, hipStream_t s,
                           const WPlane* wp = nullptr, const RowMask* rows = nullptr,
                           bool pass_b = true) {
  constexpr int CB = sizeof(cpx<R>);
  constexpr int NBA = (M * CB >= Shapes<R>::lds_a) ? 1 : Shapes<R>::lds_a / (M * CB);
  constexpr int NTA = nt_for<NBA * M / 16>();
  constexpr int NBB = nb_passB<R, M>();
  constexpr int NTB = nt_for<NBB * M / 16>();
  const GridGeom& g = p->g;
  const size_t lda = (size_t)padded(NBA * M) * CB, ldb = (size_t)padded(NBB * M) * CB;
  const double nvn = (double)g.nv * g.n * CB;
  // with a row mask: the H columns and image rows of the rows set (the
  // passes appear under names of their own)
  const uint32_t* bits = rows ? rows->bits : nullptr;
  const uint32_t* cols = rows ? rows->pair_bits : nullptr;
  const double nr = rows ? (double)rows->count : (double)g.n;
  const double nvr = (double)g.nv * nr * CB;
  {
    const unsigned planes = wp ? (unsigned)wp->count : 1u;
    ProfScope ps(p, s, rows ? "passA_adj_rows" : "passA_adj",
                 planes * ((double)g.nv * g.nu * CB + nvr), planes * (double)g.nv * M);
    bool passA_done = false;
    if constexpr (sizeof(R) == 4 && reg_size(M)) {
      if (reg_passA(g)) {
        constexpr int S = M / kRegN;
        if (rows)
          hipLaunchKernelGGL((passA_adj_reg_kernel<S, true>), dim3(g.nv), dim3(kRegT), 0, s, g,
                             (const c32*)p->grid, p->tile_flags, (c32*)p->H,
                             (const c32*)p->twiddle, cols, plane_stride(p));
        else
          hipLaunchKernelGGL((passA_adj_reg_kernel<S, false>), dim3(g.nv, planes), dim3(kRegT), 0,
                             s, g, (const c32*)p->grid, p->tile_flags, (c32*)p->H,
                             (const c32*)p->twiddle, nullptr, plane_stride(p));
        passA_done = true;
      }
    }
    if constexpr (!reg_always<R, M>) {
#define PC_PASS_A(MASKED)                                                                     \
  set_lds((const void*)passA_adj_kernel<R, M, NBA, NTA, MASKED>, lda);                        \
  hipLaunchKernelGGL((passA_adj_kernel<R, M, NBA, NTA, MASKED>),                              \
                     dim3((g.nv + NBA - 1) / NBA, planes), dim3(NTA), lda, s, g,              \
                     (const cpx<R>*)p->grid, p->tile_flags, (cpx<R>*)p->H,                    \
                     (const cpx<R>*)p->twiddle, cols, plane_stride(p))
      if (passA_done) {
      } else if (rows) {
        PC_PASS_A(true);
      } else {
        PC_PASS_A(false);
      }
#undef PC_PASS_A
    }
    PC_LAUNCH_CHECK("passA_adj");
  }
  if (!pass_b) return;  // (the caller evaluates pass B itself)
  if (wp) {  // one w-plane: rotate, add into the image
    if constexpr (sizeof(R) == 4) {
      constexpr int NBW = nb_passB<R, M, 1>();
      constexpr int NTW = nt_for<NBW * M / 16>();
      const size_t ldw = (size_t)padded(NBW * M) * CB;
      set_lds((const void*)passB_adj_w_kernel<R, M, NBW, NTW>, ldw);
      ProfScope ps(p, s, "passB_adj_w",
                   wp->count * nvn +
                       (double)g.n * g.n * sizeof(R) * (2 * wp->count - (wp->first ? 1 : 0)),
                   wp->count * (double)g.n * M);
      hipLaunchKernelGGL((passB_adj_w_kernel<R, M, NBW, NTW>), dim3((M / 2) / NBW), dim3(NTW),
                         ldw, s, g, (const cpx<R>*)p->H, image, (const cpx<R>*)p->twiddle,
                         (const R*)p->corr, scale, *wp);
      PC_LAUNCH_CHECK("passB_adj_w");
      return;
    }
    fail(PC_ERR_UNSUPPORTED, "w-planes of an FP64 plan");
  }
  ProfScope ps(p, s, rows ? "passB_adj_rows" : "passB_adj",
               nvr + nr * g.n * sizeof(R), nr * M);
  if constexpr (sizeof(R) == 4 && reg_size(M)) {
    if (reg_passB(g)) {
      constexpr int S = M / kRegN;
      if (rows)
        hipLaunchKernelGGL((passB_adj_reg_kernel<S, true>), dim3(g.n / 2), dim3(kRegT), 0, s, g,
                           (const c32*)p->H, image, (const c32*)p->twiddle, (const float*)p->corr,
                           scale, nullptr, p->max_positive, bits);
      else
        hipLaunchKernelGGL((passB_adj_reg_kernel<S, false>), dim3(g.n / 2), dim3(kRegT), 0, s, g,
                           (const c32*)p->H, image, (const c32*)p->twiddle, (const float*)p->corr,
                           scale, p->maxkey, p->max_positive, nullptr);
      PC_LAUNCH_CHECK("passB_adj");
      return;
    }
  }
#define PC_PASS_B(MASKED)                                                                       \
  set_lds((const void*)passB_adj_kernel<R, M, NBB, NTB, MASKED>, ldb);                          \
  hipLaunchKernelGGL((passB_adj_kernel<R, M, NBB, NTB, MASKED>), dim3((M / 4) / NBB), dim3(NTB), \
                     ldb, s, g, (const cpx<R>*)p->H, image, (const cpx<R>*)p->twiddle,          \
                     (const R*)p->corr, scale, rows ? nullptr : p->maxkey, p->max_positive, bits)
  if constexpr (!reg_always<R, M>) {
    if (rows) {
      PC_PASS_B(true);
    } else {
      PC_PASS_B(false);
    }
    PC_LAUNCH_CHECK("passB_adj");
  }
#undef PC_PASS_B
}

template <typename R, int M>
static void run_passes_fwd(pc_plan* p, const R* image, hipStream_t s,
                           const RowMask* rows = nullptr, bool pass_b = true) {
  constexpr int CB = sizeof(cpx<R>);
  constexpr int NBA = (M * CB >= Shapes<R>::lds_a) ? 1 : Shapes<R>::lds_a / (M * CB);
  constexpr int NTA = nt_for<NBA * M / 16>();
  constexpr int NBB = nb_passB<R, M>();
  constexpr int NTB = nt_for<NBB * M / 16>();
  const GridGeom& g = p->g;
  const size_t lda = (size_t)padded(NBA * M) * CB, ldb = (size_t)padded(NBB * M) * CB;
  const uint32_t* bits = rows ? rows->bits : nullptr;
  const uint32_t* cols = rows ? rows->pair_bits : nullptr;
  const double nr = rows ? (double)rows->count : (double)g.n;
  const double nvr = (double)g.nv * nr * CB;
  if (pass_b) {  // (else the caller has written the pass-A buffer's columns)
    ProfScope ps(p, s, rows ? "passB_fwd_rows" : "passB_fwd", nvr + nr * g.n * sizeof(R), nr * M);
    bool done = false;
    if constexpr (sizeof(R) == 4 && reg_size(M)) {
      if (reg_passB(g)) {
        constexpr int S = M / kRegN;
        if (rows)
          hipLaunchKernelGGL((passB_fwd_reg_kernel<S, true>), dim3(g.n / 2), dim3(kRegT), 0, s, g,
                             image, (c32*)p->H, (const c32*)p->twiddle, (const float*)p->corr,
                             bits);
        else
          hipLaunchKernelGGL((passB_fwd_reg_kernel<S, false>), dim3(g.n / 2), dim3(kRegT), 0, s, g,
                             image, (c32*)p->H, (const c32*)p->twiddle, (const float*)p->corr,
                             nullptr);
        done = true;
      }
    }
    if constexpr (!reg_always<R, M>) {
#define PC_PASS_BF(MASKED)                                                                      \
  set_lds((const void*)passB_fwd_kernel<R, M, NBB, NTB, MASKED>, ldb);                          \
  hipLaunchKernelGGL((passB_fwd_kernel<R, M, NBB, NTB, MASKED>), dim3((M / 4) / NBB), dim3(NTB), \
                     ldb, s, g, image, (cpx<R>*)p->H, (const cpx<R>*)p->twiddle,                \
                     (const R*)p->corr, bits)
      if (done) {
      } else if (rows) {
        PC_PASS_BF(true);
      } else {
        PC_PASS_BF(false);
      }
#undef PC_PASS_BF
    }
    PC_LAUNCH_CHECK("passB_fwd");
  }
  ProfScope ps(p, s, rows ? "passA_fwd_rows" : "passA_fwd", (double)g.nv * g.nu * CB + nvr,
               (double)g.nv * M);
  bool done = false;
  if constexpr (sizeof(R) == 4 && reg_size(M)) {
    if (reg_passA(g)) {
      constexpr int S = M / kRegN;
      if (rows)
        hipLaunchKernelGGL((passA_fwd_reg_kernel<S, true>), dim3(g.nv), dim3(kRegT), 0, s, g,
                           (const c32*)p->H, (c32*)p->grid, (const c32*)p->twiddle, cols);
      else
        hipLaunchKernelGGL((passA_fwd_reg_kernel<S, false>), dim3(g.nv), dim3(kRegT), 0, s, g,
                           (const c32*)p->H, (c32*)p->grid, (const c32*)p->twiddle, nullptr);
      done = true;
    }
  }
  if constexpr (!reg_always<R, M>) {
#define PC_PASS_AF(MASKED)                                                                      \
  set_lds((const void*)passA_fwd_kernel<R, M, NBA, NTA, MASKED>, lda);                          \
  hipLaunchKernelGGL((passA_fwd_kernel<R, M, NBA, NTA, MASKED>), dim3((g.nv + NBA - 1) / NBA),  \
                     dim3(NTA), lda, s, g, (const cpx<R>*)p->H, (cpx<R>*)p->grid,               \
                     (const cpx<R>*)p->twiddle, cols)
    if (done) {
    } else if (rows) {
      PC_PASS_AF(true);
    } else {
      PC_PASS_AF(false);
    }
#undef PC_PASS_AF
  }
  PC_LAUNCH_CHECK("passA_fwd");
}

template <typename R>
static void dispatch_M(pc_plan* p, bool adjoint, R* img_out, const R* img_in, R scale,
                       hipStream_t s, const WPlane* wp = nullptr, const RowMask* rows = nullptr,
                       bool pass_b = true) {
  switch (p->g.M) {
#define PC_M(m)                                                     \
  case m:                                                           \
    if (adjoint)                                                    \
      run_passes_adj<R, m>(p, img_out, scale, s, wp, rows, pass_b); \
    else                                                            \
      run_passes_fwd<R, m>(p, img_in, s, rows, pass_b);             \
    return;
    PC_M(32) PC_M(64) PC_M(128) PC_M(256) PC_M(512) PC_M(1024) PC_M(2048) PC_M(4096) PC_M(8192)
#undef PC_M
    case 16384:
      if constexpr (sizeof(R) == 4) {
        if (adjoint)
          run_passes_adj<R, 16384>(p, img_out, scale, s, wp, rows, pass_b);
        else
          run_passes_fwd<R, 16384>(p, img_in, s, rows, pass_b);
        return;
      }
      [[fallthrough]];
    default:
      fail(PC_ERR_UNSUPPORTED, "fine grid size " + std::to_string(p->g.M) +
                                   (sizeof(R) == 8 ? " in FP64" : "") + " is not a supported power of two");
  }
}


void forward_grid_set(pc_plan* p, const AtomSet& as, const double* w, const c32* base,
                      bool base_sorted, double* stats, c32* out, hipStream_t s) {
  if (p->Cw || p->precision != PC_PREC_FP32)
    fail(PC_ERR_UNSUPPORTED, "gridded set operators need a coplanar FP32 plan");
  const GridGeom& g = p->g;
  {
    ProfScope ps(p, s, "passB_fwd_set", 8.0 * g.nv * as.rows.count + 12.0 * as.nS,
                 (double)g.nv * as.nS);
    const dim3 grid((unsigned)((g.nv + 255) / 256), (unsigned)as.nrows);
    if (g.M == kSplitGrid)  // (the other sizes share one layout)
      hipLaunchKernelGGL((rows_fwd_direct_kernel<kSplitGrid>), grid, dim3(256), 0, s, g,
                         as.rowlist, as.pix, w, (const float*)p->corr, (c32*)p->H);
    else
      hipLaunchKernelGGL((rows_fwd_direct_kernel<kSplitGrid / 2>), grid, dim3(256), 0, s, g,
                         as.rowlist, as.pix, w, (const float*)p->corr, (c32*)p->H);
    PC_LAUNCH_CHECK("rows_fwd_direct");
  }
  dispatch_M<float>(p, false, nullptr, nullptr, 1.0f, s, nullptr, &as.rows, false);
  launch_interp<float>(p, nullptr, out, s, base, base && !base_sorted ? p->perm : nullptr, stats);
}

void adjoint_grid_set(pc_plan* p, const c32* vis, const AtomSet& as, double* gout,
                      hipStream_t s) {
  if (p->Cw || p->precision != PC_PREC_FP32)
    fail(PC_ERR_UNSUPPORTED, "gridded set operators need a coplanar FP32 plan");
  const GridGeom& g = p->g;
  launch_spread<float>(p, vis, nullptr, s);
  dispatch_M<float>(p, true, nullptr, nullptr, 1.0f, s, nullptr, &as.rows, false);
  ProfScope ps(p, s, "passB_adj_set", 8.0 * g.nv * as.rows.count + 12.0 * as.nS,
               (double)g.nv * as.nS);
  if (g.M == kSplitGrid)  // (the other sizes share one layout)
    hipLaunchKernelGGL((atoms_adj_direct_kernel<kSplitGrid>), dim3((unsigned)as.nS),
                       dim3(256), 0, s, g, as.pix, (const c32*)p->H, (const float*)p->corr, gout);
  else
    hipLaunchKernelGGL((atoms_adj_direct_kernel<kSplitGrid / 2>), dim3((unsigned)as.nS),
                       dim3(256), 0, s, g, as.pix, (const c32*)p->H, (const float*)p->corr, gout);
  PC_LAUNCH_CHECK("atoms_adj_direct");
}

// Small moves of the gridded restricted gradient: caller-order atoms into
// pixel order (weights widened to FP64), the gradient back, and visibilities
// from plan to caller order.
__global__ void atoms_to_set_kernel(int64_t nS, const int32_t* __restrict__ order,
                                    const float* __restrict__ weight, double* __restrict__ w) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nS) w[q] = (double)weight[order[q]];
}
__global__ void set_to_atoms_kernel(int64_t nS, const int32_t* __restrict__ order,
                                    const double* __restrict__ g, double* __restrict__ grad) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < nS) grad[order[q]] = g[q];
}
__global__ void vis_to_caller_kernel(int64_t L, const int32_t* __restrict__ perm,
                                     const c32* __restrict__ in, c32* __restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < L) out[perm[k]] = in[k];
}

void restricted_gradient_grid(pc_plan* p, const c32* vis, int64_t natoms, const int32_t* pix,
                              const float* weight, double* grad, c32* resid, hipStream_t s) {
  if (p->Cw || p->precision != PC_PREC_FP32)
    fail(PC_ERR_UNSUPPORTED, "the gridded restricted gradient needs a coplanar FP32 plan");
  const int64_t L = p->L;
  const unsigned lb = (unsigned)((L + 255) / 256);
  if (natoms == 0) {  // r = V
    if (resid)
      PC_HIP(hipMemcpyAsync(resid, vis, L * sizeof(c32), hipMemcpyDeviceToDevice, s));
    return;
  }
  // the set in pixel order, its occupied rows and their mask, on the host
  const int n = p->g.n;
  std::vector<int32_t> hp((size_t)natoms);
  PC_HIP(hipMemcpyAsync(hp.data(), pix, natoms * 4, hipMemcpyDeviceToHost, s));
  PC_HIP(hipStreamSynchronize(s));
  for (int64_t q = 0; q < natoms; ++q)
    PC_REQUIRE(hp[q] >= 0 && (int64_t)hp[q] < (int64_t)n * n, "pix out of [0, npix^2)");
  std::vector<int32_t> order((size_t)natoms);
  for (int64_t q = 0; q < natoms; ++q) order[q] = (int32_t)q;
  std::stable_sort(order.begin(), order.end(),
                   [&](int32_t a, int32_t b) { return hp[a] < hp[b]; });
  const int64_t words = (n + 31) / 32;
  std::vector<int32_t> rl;
  std::vector<uint32_t> mask((size_t)words, 0u);
  for (int64_t q = 0; q < natoms; ++q) {
    const int i = hp[order[q]] / n;
    if (q == 0 || i != hp[order[q - 1]] / n) rl.insert(rl.end(), {i, (int32_t)q, 0});
    rl.back() = (int32_t)(q + 1);
    mask[i >> 5] |= 1u << (i & 31);
  }
  const int64_t nrows = (int64_t)rl.size() / 3;
  // device scratch: [pixel-order pix | order | rows | mask | w | g]
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t o_ord = al(natoms * 4), o_rows = o_ord + al(natoms * 4);
  const size_t o_mask = o_rows + al(nrows * 12), o_w = o_mask + al(words * 4);
  const size_t o_g = o_w + al(natoms * 8);
  const size_t total = o_g + al(natoms * 8);
  unsigned char* d = (unsigned char*)ensure_atom_scratch(p, total);
  std::vector<unsigned char> up(o_w);
  for (int64_t q = 0; q < natoms; ++q) ((int32_t*)up.data())[q] = hp[order[q]];
  std::memcpy(up.data() + o_ord, order.data(), natoms * 4);
  std::memcpy(up.data() + o_rows, rl.data(), nrows * 12);
  std::memcpy(up.data() + o_mask, mask.data(), words * 4);
  PC_HIP(hipMemcpyAsync(d, up.data(), o_w, hipMemcpyHostToDevice, s));
  const int32_t* dord = (const int32_t*)(d + o_ord);
  double* w = (double*)(d + o_w);
  double* g = (double*)(d + o_g);
  const unsigned ab = (unsigned)((natoms + 255) / 256);
  hipLaunchKernelGGL(atoms_to_set_kernel, dim3(ab), dim3(256), 0, s, natoms, dord, weight, w);
  PC_LAUNCH_CHECK("atoms_to_set");
  const AtomSet as{natoms, (const int32_t*)d, (const int3*)(d + o_rows), nrows,
                   RowMask{(const uint32_t*)(d + o_mask), nrows, (const uint32_t*)(d + o_mask)}};
  // r = V - Phi_S x in plan order, then Phi_S* r
  c32* r = (c32*)p->vis_scratch;
  forward_grid_set(p, as, w, vis, false, nullptr, r, s);
  adjoint_grid_set(p, r, as, g, s);
  hipLaunchKernelGGL(set_to_atoms_kernel, dim3(ab), dim3(256), 0, s, natoms, dord, g, grad);
  PC_LAUNCH_CHECK("set_to_atoms");
  if (resid) {
    hipLaunchKernelGGL(vis_to_caller_kernel, dim3(lb), dim3(256), 0, s, L, p->perm, r, resid);
    PC_LAUNCH_CHECK("vis_to_caller");
  }
  PC_HIP(hipStreamSynchronize(s));  // the host staging above goes out of scope
}

struct ReadbackArgs {
  static constexpr int kMax = 32;
  Readback r[kMax];
};
__global__ __launch_bounds__(256) void readback_kernel(ReadbackArgs a) {
  const Readback r = a.r[blockIdx.x];
  const uint32_t* src = (const uint32_t*)r.src;
  uint32_t* dst = (uint32_t*)r.dst;
  for (uint32_t i = threadIdx.x; i < r.bytes / 4; i += 256) dst[i] = src[i];
}

void readback(const Readback* r, int n, hipStream_t s) {
  for (int i = 0; i < n; i += ReadbackArgs::kMax) {
    ReadbackArgs a{};
    const int m = std::min(n - i, ReadbackArgs::kMax);
    std::copy(r + i, r + i + m, a.r);
    hipLaunchKernelGGL(readback_kernel, dim3((unsigned)m), dim3(256), 0, s, a);
    PC_LAUNCH_CHECK("readback");
  }
}

void maxkey_read(pc_plan* const* plans, int n, hipStream_t s, double* max_abs, int64_t* argmax) {
  std::vector<Readback> r((size_t)n);
  for (int j = 0; j < n; ++j) {
    if (!plans[j]->key_host) plans[j]->key_host = pinned_slot();
    r[j] = Readback{plans[j]->maxkey, plans[j]->key_host, sizeof(unsigned long long)};
  }
  readback(r.data(), n, s);
  PC_HIP(hipStreamSynchronize(s));
  for (int j = 0; j < n; ++j)
    maxkey_decode(*plans[j]->key_host, max_abs ? max_abs + j : nullptr,
                  argmax ? argmax + j : nullptr);
}

void maxkey_read(pc_plan* p, hipStream_t s, double* max_abs, int64_t* argmax) {
  maxkey_read(&p, 1, s, max_abs, argmax);
}

void maxkey_decode(unsigned long long key, double* max_abs, int64_t* argmax) {
  const uint32_t hi = (uint32_t)(key >> 32), lo = (uint32_t)(key & 0xffffffffu);
  float f;
  std::memcpy(&f, &hi, 4);
  if (max_abs) *max_abs = (double)f;
  if (argmax) *argmax = (int64_t)(0xffffffffu - lo);
}

// The w-stacked adjoint: per plane, weights, spread, pass A and the rotating
// pass B; then the w correction and the maximum.
static void adjoint_grid_w(pc_plan* p, const c32* vis, bool vis_sorted, float* image, float scale,
                           hipStream_t s) {
  const WStack& ws = p->ws;
  const float R = 0.5f * (float)p->g.W;
  const unsigned nb = (unsigned)((p->L + 255) / 256);
  std::unique_ptr<WPlanes> own;  // (unless the caller holds the buffers)
  if (!p->w_group) own.reset(new WPlanes(p, s));
  const int together = p->w_group->planes;
  for (int j = 0; j < ws.nplanes; j += together) {
    const int count = std::min(together, ws.nplanes - j);
    const WPlane wp{ws.w0 + j * ws.dw, ws.dw, ws.cmid, j == 0 ? 1 : 0, count, plane_stride(p).H};
    {
      ProfScope ps(p, s, "wplane", p->L * (16.0 + 8.0 * count), (double)p->L * count);
      hipLaunchKernelGGL(wplane_kernel, dim3(nb), dim3(256), 0, s, p->L, p->Cw, vis,
                         vis_sorted ? nullptr : p->perm, wp, 1.0 / ws.dw, R * R, 1.0f / R, es_c(p->g.W),
                         (c32*)p->wvals);
      PC_LAUNCH_CHECK("wplane");
    }
    launch_spread<float>(p, (const c32*)p->wvals, nullptr, s, count);  // also clears the max key
    dispatch_M<float>(p, true, image, nullptr, scale, s, &wp);
  }
  const int64_t N = (int64_t)p->g.n * p->g.n;
  ProfScope ps(p, s, "wfinal", 8.0 * N, (double)N);
  const unsigned nbf = (unsigned)std::min<int64_t>((N + 255) / 256, 1024);
  hipLaunchKernelGGL(wfinal_kernel, dim3(nbf), dim3(256), 0, s, p->g, ws,
                     p->wquad, image, p->maxkey, p->max_positive);
  PC_LAUNCH_CHECK("wfinal");
}

template <typename R>
void adjoint_grid(pc_plan* p, const cpx<R>* vis, bool vis_sorted, R* image, R scale,
                  hipStream_t s, const RowMask* rows) {
  if (p->Cw) {
    if (rows) fail(PC_ERR_UNSUPPORTED, "a row mask with the w-stacked adjoint");
    if constexpr (sizeof(R) == 4) {
      adjoint_grid_w(p, vis, vis_sorted, image, scale, s);
      return;
    }
    fail(PC_ERR_UNSUPPORTED, "w-stacked adjoint of an FP64 plan");
  }
  launch_spread<R>(p, vis, vis_sorted ? nullptr : p->perm, s);  // also clears the max key
  dispatch_M<R>(p, true, image, nullptr, scale, s, nullptr, rows);
}

template <typename R>
void forward_grid(pc_plan* p, const R* image, cpx<R>* vis_out, bool out_sorted, hipStream_t s,
                  const RowMask* rows, const cpx<R>* base, double* stats) {
  if (p->Cw)
    fail(PC_ERR_UNSUPPORTED,
         "the gridded forward operator needs a coplanar plan (w = 0); the direct sums take w");
  if (base && !out_sorted) fail(PC_ERR_INVALID_ARG, "forward_grid: a base needs plan order");
  dispatch_M<R>(p, false, nullptr, image, R(1), s, nullptr, rows);
  launch_interp<R>(p, out_sorted ? nullptr : p->perm, vis_out, s, base, nullptr, stats);
}

// ----------------------------------------------------------------------------
// Batched adjoint across plans
// ----------------------------------------------------------------------------
namespace {
template <int M>
struct PassShape {
  static constexpr int CB = sizeof(c32);
  static constexpr int NBA = (M * CB >= Shapes<float>::lds_a) ? 1 : Shapes<float>::lds_a / (M * CB);
  static constexpr int NTA = nt_for<NBA * M / 16>();
  static constexpr int NBB = nb_passB<float, M>();
  static constexpr int NTB = nt_for<NBB * M / 16>();
};

int passA_blocks(int M, int nv) {
  switch (M) {
#define PC_M(m) case m: return (nv + PassShape<m>::NBA - 1) / PassShape<m>::NBA;
    PC_M(32) PC_M(64) PC_M(128) PC_M(256) PC_M(512) PC_M(1024) PC_M(2048) PC_M(8192) PC_M(16384)
#undef PC_M
  }
  return 0;
}

int passB_blocks(int M) {
  switch (M) {
#define PC_M(m) case m: return (m / 4) / PassShape<m>::NBB;
    PC_M(32) PC_M(64) PC_M(128) PC_M(256) PC_M(512) PC_M(1024) PC_M(2048) PC_M(8192) PC_M(16384)
#undef PC_M
  }
  return 0;
}

template <int M>
void launch_pass_batch(bool passA, const AdjJob* jobs, const int2* items, int nitems,
                       hipStream_t s) {
  using P = PassShape<M>;
  if (passA) {
    const size_t lds = (size_t)padded(P::NBA * M) * P::CB;
    set_lds((const void*)passA_batch_kernel<M, P::NBA, P::NTA>, lds);
    hipLaunchKernelGGL((passA_batch_kernel<M, P::NBA, P::NTA>), dim3(nitems), dim3(P::NTA), lds, s,
                       jobs, items);
    PC_LAUNCH_CHECK("passA_batch");
  } else {
    const size_t lds = (size_t)padded(P::NBB * M) * P::CB;
    set_lds((const void*)passB_batch_kernel<M, P::NBB, P::NTB>, lds);
    hipLaunchKernelGGL((passB_batch_kernel<M, P::NBB, P::NTB>), dim3(nitems), dim3(P::NTB), lds, s,
                       jobs, items);
    PC_LAUNCH_CHECK("passB_batch");
  }
}

template <int S>
void launch_pass_reg_batch(bool passA, const AdjJob* jobs, const int2* items, int nitems,
                           hipStream_t s) {
  if (passA)
    hipLaunchKernelGGL((passA_reg_batch_kernel<S>), dim3(nitems), dim3(kRegT), 0, s, jobs, items);
  else
    hipLaunchKernelGGL((passB_reg_batch_kernel<S>), dim3(nitems), dim3(kRegT), 0, s, jobs, items);
  PC_LAUNCH_CHECK("pass_reg_batch");
}

void pass_batch(int M, bool reg, bool passA, const AdjJob* jobs, const int2* items, int nitems,
                hipStream_t s) {
  if (reg) switch (M) {
      case kRegN: launch_pass_reg_batch<1>(passA, jobs, items, nitems, s); return;
      case 2 * kRegN: launch_pass_reg_batch<2>(passA, jobs, items, nitems, s); return;
      case 4 * kRegN: launch_pass_reg_batch<4>(passA, jobs, items, nitems, s); return;
    }
  switch (M) {
#define PC_M(m) case m: launch_pass_batch<m>(passA, jobs, items, nitems, s); return;
    PC_M(32) PC_M(64) PC_M(128) PC_M(256) PC_M(512) PC_M(1024) PC_M(2048) PC_M(8192) PC_M(16384)
#undef PC_M
  }
  fail(PC_ERR_UNSUPPORTED, "fine grid size");
}

template <int W>
void launch_spread_batch(const AdjJob* jobs, const int2* items, int nitems, hipStream_t s) {
  // grouped work lists: items are (job, workgroup)
  hipLaunchKernelGGL((spread_quad_batch_kernel<W>), dim3(nitems), dim3(64 * kSpreadQuad),
                     SpreadM::lds_bytes, s, jobs, items);
  PC_LAUNCH_CHECK("spread_batch");
}

void spread_batch(int W, const AdjJob* jobs, const int2* items, int nitems, hipStream_t s) {
  switch (W) {
#define PC_W(w) case w: launch_spread_batch<w>(jobs, items, nitems, s); return;
    PC_W(2) PC_W(3) PC_W(4) PC_W(5) PC_W(6) PC_W(7) PC_W(8) PC_W(9) PC_W(10) PC_W(11) PC_W(12)
    PC_W(13) PC_W(14) PC_W(15) PC_W(16)
#undef PC_W
  }
  fail(PC_ERR_UNSUPPORTED, "kernel width");
}
}  // namespace

void BatchCtx::release() {
  if (pending && done) (void)hipEventSynchronize(done);
  pending = false;
  if (dev) (void)hipFree(dev);
  if (host) (void)hipHostFree(host);
  if (done) (void)hipEventDestroy(done);
  dev = host = nullptr;
  dev_bytes = host_bytes = 0;
  done = nullptr;
}

void adjoint_grid_batch(BatchCtx& ctx, pc_plan* const* plans, const c32* const* vis,
                        const bool* vis_sorted, float* const* images, const float* scales, int n,
                        hipStream_t s) {
  if (n <= 0) return;
  // w-stacked plans run on their own, ahead of the shared launches
  {
    std::vector<int> flat;
    for (int j = 0; j < n; ++j) {
      PC_REQUIRE(plans[j] && plans[j]->precision == PC_PREC_FP32, "batched adjoint needs FP32 plans");
      if (plans[j]->Cw)
        adjoint_grid<float>(plans[j], vis[j], vis_sorted[j], images[j],
                            scales ? scales[j] : 1.0f, s);
      else
        flat.push_back(j);
    }
    if ((int)flat.size() < n) {
      if (flat.empty()) return;
      std::vector<pc_plan*> fp;
      std::vector<const c32*> fv;
      std::unique_ptr<bool[]> fs(new bool[flat.size()]);
      std::vector<float*> fi;
      std::vector<float> fsc;
      for (size_t q = 0; q < flat.size(); ++q) {
        const int j = flat[q];
        fp.push_back(plans[j]);
        fv.push_back(vis[j]);
        fs[q] = vis_sorted[j];
        fi.push_back(images[j]);
        fsc.push_back(scales ? scales[j] : 1.0f);
      }
      adjoint_grid_batch(ctx, fp.data(), fv.data(), fs.get(), fi.data(), fsc.data(),
                         (int)flat.size(), s);
      return;
    }
  }
  if (!ctx.done) PC_HIP(hipEventCreateWithFlags(&ctx.done, hipEventDisableTiming));
  if (ctx.pending) PC_HIP(hipEventSynchronize(ctx.done));
  // job descriptors and work lists
  std::vector<AdjJob> jobs(n);
  std::vector<int> Ms, Ws;
  for (int j = 0; j < n; ++j) {
    pc_plan* p = plans[j];
    PC_REQUIRE(p && p->precision == PC_PREC_FP32, "batched adjoint needs FP32 plans");
    AdjJob& J = jobs[j];
    J.g = p->g;
    J.chunks = p->chunks;
    J.fold = p->fold;
    J.flags = p->tile_flags;
    J.cell = p->cell;
    J.off = (const float*)p->off;
    J.vals = vis[j];
    J.perm = vis_sorted[j] ? nullptr : p->perm;
    J.grid = (c32*)p->grid;
    J.partials = (c32*)p->partials;
    J.H = (c32*)p->H;
    J.image = images[j];
    J.tw = (const c32*)p->twiddle;
    J.corr = (const float*)p->corr;
    J.scale = scales ? scales[j] : 1.0f;
    J.maxkey = p->maxkey;
    J.positive = p->max_positive;
    J.rows = nullptr;
    if (std::find(Ms.begin(), Ms.end(), p->g.M) == Ms.end()) Ms.push_back(p->g.M);
    if (std::find(Ws.begin(), Ws.end(), p->g.W) == Ws.end()) Ws.push_back(p->g.W);
  }
  // Table sizes, then the tables themselves, written straight into the pinned
  // staging: the jobs, the spreading workgroups per kernel width, the folded
  // tiles, and the pass items per fine grid (those of the register-held passes
  // apart, every first pass ahead of every second).
  struct PassItems {
    int M;
    bool reg, first;
    size_t off, count;
  };
  size_t bytes = 0;
  auto reserve = [&](size_t count, size_t size) {
    const size_t off = (bytes + 255) & ~size_t(255);
    bytes = off + count * size;
    return off;
  };
  auto blocks_of = [&](int j, int M, bool reg, bool first) -> int {
    const GridGeom& g = plans[j]->g;
    if (g.M != M || (first ? reg_passA(g) : reg_passB(g)) != reg) return 0;
    return reg ? (first ? g.nv : g.n / 2) : (first ? passA_blocks(M, g.nv) : passB_blocks(M));
  };
  const size_t o_jobs = reserve(n, sizeof(AdjJob));
  std::vector<size_t> o_spread(Ws.size()), n_spread(Ws.size(), 0);
  for (size_t w = 0; w < Ws.size(); ++w) {
    for (int j = 0; j < n; ++j)
      if (plans[j]->g.W == Ws[w]) n_spread[w] += plans[j]->chunk_work.size();
    o_spread[w] = reserve(n_spread[w], sizeof(int2));
  }
  size_t n_fold = 0;
  for (int j = 0; j < n; ++j) n_fold += (size_t)plans[j]->n_fold;
  const size_t o_fold = reserve(n_fold, sizeof(int2));
  std::vector<PassItems> passes;
  for (const bool first : {true, false})
    for (const int M : Ms)
      for (const bool reg : {false, true}) {
        size_t count = 0;
        for (int j = 0; j < n; ++j) count += (size_t)blocks_of(j, M, reg, first);
        if (count) passes.push_back({M, reg, first, reserve(count, sizeof(int2)), count});
      }
  if (ctx.host_bytes < bytes) {
    if (ctx.host) (void)hipHostFree(ctx.host);
    ctx.host = nullptr;
    ctx.host_bytes = 0;
    PC_HIP(hipHostMalloc((void**)&ctx.host, bytes * 2));
    ctx.host_bytes = bytes * 2;
  }
  if (ctx.dev_bytes < bytes) {
    if (ctx.dev) (void)hipFree(ctx.dev);
    ctx.dev = nullptr;
    ctx.dev_bytes = 0;
    PC_HIP(hipMalloc((void**)&ctx.dev, bytes * 2));
    ctx.dev_bytes = bytes * 2;
  }
  std::memcpy(ctx.host + o_jobs, jobs.data(), n * sizeof(AdjJob));
  for (size_t w = 0; w < Ws.size(); ++w) {
    // Longest spreading workgroups first across all plans, to a factor of two:
    // each plan lists its own longest first, so the classes of work above 512,
    // 256, ... are taken from the plans in turn.
    int2* it = (int2*)(ctx.host + o_spread[w]);
    std::vector<size_t> at(n, 0);
    for (int32_t above = 512;; above = above > 16 ? above / 2 : -1) {
      for (int j = 0; j < n; ++j) {
        const pc_plan* p = plans[j];
        if (p->g.W != Ws[w]) continue;
        while (at[j] < p->chunk_work.size() && p->chunk_work[at[j]] > above)
          *it++ = make_int2(j, (int)at[j]++);
      }
      if (above < 0) break;
    }
  }
  {
    int2* it = (int2*)(ctx.host + o_fold);
    for (int j = 0; j < n; ++j)
      for (int64_t f = 0; f < plans[j]->n_fold; ++f) *it++ = make_int2(j, (int)f);
  }
  for (const PassItems& ps : passes) {
    int2* it = (int2*)(ctx.host + ps.off);
    for (int j = 0; j < n; ++j) {
      const int blocks = blocks_of(j, ps.M, ps.reg, ps.first);
      for (int r = 0; r < blocks; ++r) *it++ = make_int2(j, r);
    }
  }
  PC_HIP(hipMemcpyAsync(ctx.dev, ctx.host, bytes, hipMemcpyHostToDevice, s));
  const AdjJob* djobs = (const AdjJob*)(ctx.dev + o_jobs);
  for (size_t w = 0; w < Ws.size(); ++w)
    if (n_spread[w])
      spread_batch(Ws[w], djobs, (const int2*)(ctx.dev + o_spread[w]), (int)n_spread[w], s);
  if (n_fold) {
    hipLaunchKernelGGL(fold_batch_kernel, dim3((unsigned)n_fold, kTile * kTile / 64),
                       dim3(64 * kFoldSub), 0, s, djobs, (const int2*)(ctx.dev + o_fold));
    PC_LAUNCH_CHECK("fold_batch");
  }
  for (const PassItems& ps : passes)  // every first pass, then every second
    pass_batch(ps.M, ps.reg, ps.first, djobs, (const int2*)(ctx.dev + ps.off), (int)ps.count, s);
  PC_HIP(hipEventRecord(ctx.done, s));
  ctx.pending = true;
}

template void adjoint_grid<float>(pc_plan*, const c32*, bool, float*, float, hipStream_t,
                                  const RowMask*);
template void adjoint_grid<double>(pc_plan*, const c64*, bool, double*, double, hipStream_t,
                                   const RowMask*);
template void forward_grid<float>(pc_plan*, const float*, c32*, bool, hipStream_t,
                                  const RowMask*, const c32*, double*);
template void forward_grid<double>(pc_plan*, const double*, c64*, bool, hipStream_t,
                                   const RowMask*, const c64*, double*);

}  // namespace pc
