// Loss derivatives with fused column norms, and the prediction update
// (Section 2: eq. 2 gives the first and second derivatives of the loss at the
// current predictions; the model is updated by a_t = a_{t-1} + eps * f_t).
//
// k_grad: one thread per row, the rows of a block in one 256-row tile, tiles
//   grid-strided.  The lanes of a wave take consecutive rows, so every load
//   and store is one 256-byte run of a column of the column-major matrices.
//   Softmax cross-entropy (rows of more than 1024 scores, or leading dimensions
//   of 2^24 and more; others stay in registers, k_grad_softmax_regs and
//   k_grad_softmax_wide): a first pass over the row's scores keeps a running
//   maximum and the sum of exp(a - max), rescaled chunk by chunk; the second
//   pass re-reads the scores and writes g = p - onehot(y), h = p (1 - p).
//   Sigmoid cross-entropy needs one pass: g = s - Y, h = s (1 - s).
//   The squared column norms of the stored G (what Top Outputs and Random
//   Sampling rank and draw by, Sections 3.1, 3.2) are summed in the same pass:
//   each 16-column chunk of g goes through LDS, 16 threads per column add 16
//   rows each in fp64, a fixed shift-and-add over their 16 lanes (DPP, in
//   registers) joins them, and one thread adds the
//   tile's sum to its slot's partial (slot = tile mod GRAD_PARTS, always the
//   same thread of the same block, in tile order).  k_grad_norm_final adds the
//   slots in a fixed order, so the norms are deterministic and the same for
//   every grid that divides the slot count (the fused update below launches
//   fewer blocks than the derivatives alone).  k_grad_softmax_wide has a partial
//   per block instead, and a grid that follows from the shape (sb_grad_plan.h).
// k_update: F[i, j] += lr * V[leaf of i, j] in fp64, rounded once to fp32.
//   lr * V of a chunk of columns is staged in LDS; the leaf ids come from the
//   leaf segments (k_leaf_ids, shared with the leaf values).
// The update of one tree followed by the derivatives of the next (the two
// consecutive steps of the boosting loop) can run as one pass, so that F is read
// once instead of twice: for softmax with d <= 104 k_grad_softmax_regs with UPD
// loads a row's scores, adds lr * V of the row's leaf (all of lr * V staged in
// LDS), stores the new scores and goes on from them; for sigmoid
// k_update_sigmoid does so by chunks of 16 columns.  The arithmetic is k_update's,
// so the result is bit-identical to the two calls.
#include <cmath>

#include "sb_common.h"
#include "sb_grad_plan.h"
#include "sb_leaf_ids.h"

namespace sb {
namespace {

// A double moved across lanes by a DPP control; lanes it does not write get 0.
template <int CTRL>
__device__ inline double dpp_f64(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// Sum over each row of 16 lanes, in registers (no LDS traffic): shifts by 1,
// 2, 4 and 8 lanes (lanes a shift does not write add 0), so the last lane of
// each row ends with the row's sum, always added in the same order.
__device__ inline double row16_sum(double x) {
  x += dpp_f64<0x111>(x);
  x += dpp_f64<0x112>(x);
  x += dpp_f64<0x114>(x);
  x += dpp_f64<0x118>(x);
  return x;
}

constexpr int GRAD_THREADS = 256;
constexpr int GRAD_JA = 8;          // columns per load batch of the softmax first pass
constexpr int GRAD_JC = 16;         // columns per chunk of the second pass (norm staging)
// Column-norm partial slots: tile t adds into slot t % GRAD_PARTS, and the
// grid divides the slot count (or is one block per tile), so every slot
// belongs to one block and sums its tiles in tile order: the norms do not
// depend on the grid.  1536 = 2^9 * 3 has the divisors 512 and 768 (two and
// three blocks per CU of MI355X).
constexpr int GRAD_PARTS = 1536;
constexpr int UPD_THREADS = 256;
constexpr int UPD_LDS_DOUBLES = 8192;  // lr * V of one column chunk: at most 64 KB
constexpr int UPD_JC = 16;             // columns per chunk at most
constexpr int UPD_MAX_BLOCKS = 2048;
constexpr int UPD_SIG_BLOCKS = 768;  // three blocks per CU; a divisor of GRAD_PARTS

struct GradArgs {
  int loss;
  const float* F;
  int64_t n;
  int32_t d;
  int64_t ld_f;
  const int32_t* labels;
  const uint8_t* Y;
  int64_t ld_y;
  float* G;
  int64_t ld_g;
  float* hess;
  int64_t ld_h;
  float* h_row;
  double* npart;  // [d][n_parts] or NULL: sums of g^2 per column and slot
  int32_t n_tiles;
  int32_t n_parts;  // min(n_tiles, GRAD_PARTS)
  // update before the derivatives (k_grad_softmax_regs with UPD): F_upd is F
  // (updated in place), ids the leaf of every row, lv_stride the doubles per
  // leaf of lr * V in LDS
  float* F_upd;
  const uint8_t* ids;
  int32_t n_leaves;
  int32_t lv_stride;
  const double* V;
  int64_t ld_v;
  double lr;
};

// The squared norms of a tile's chunk of 16 columns from j0, staged in gbuf:
// 16 threads per column add 16 rows each, and the column's sum goes to its
// tile's slot.
__device__ inline void add_norms(const GradArgs& a, float (*gbuf)[GRAD_THREADS], int64_t base, int d, int j0) {
  if (!a.npart) return;
  lds_barrier();
  // lanes c*16 .. c*16+15 share column c
  const int c = threadIdx.x >> 4, seg = threadIdx.x & 15;
  const float4* src = reinterpret_cast<const float4*>(&gbuf[c][seg * 16]);
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = src[q];
    acc += (double)v.x * v.x;
    acc += (double)v.y * v.y;
    acc += (double)v.z * v.z;
    acc += (double)v.w * v.w;
  }
  acc = row16_sum(acc);  // in the row's last lane
  if (seg == 15 && j0 + c < d) {
    const int tile = (int)(base / GRAD_THREADS);
    double* pp = a.npart + (int64_t)(j0 + c) * a.n_parts + tile % a.n_parts;
    *pp = tile < a.n_parts ? acc : *pp + acc;  // the slot's first tile writes it
  }
  lds_barrier();
}

// One tile of k_grad (the loss, whether the tile is full and whether the
// hessians are stored are template parameters, so the column loop has no
// runtime branch).  Columns past d in the last chunk load column d-1 and
// store column d-1's own values there (same address, same value), and d is
// passed in opaque to the compiler, as in grad_softmax_tile below.
template <int LOSS, bool FULL, bool HESS>
__device__ inline void grad_tile(const GradArgs& a, float (*gbuf)[GRAD_THREADS], int64_t base, int d) {
  const int tid = threadIdx.x;
  const int64_t row = base + tid;
  const bool ok = FULL || row < a.n;
  const int64_t rc = ok ? row : a.n - 1;  // rows past the end read row n-1 and store nothing
  float m = -INFINITY, s = 0.0f, inv = 0.0f;
  int y = -1;
  if constexpr (LOSS == SB_LOSS_SOFTMAX_CE) {
    y = a.labels[rc];
    for (int j0 = 0; j0 < d; j0 += GRAD_JA) {
      float x[GRAD_JA];
      // columns past d (last chunk only) repeat column d-1: a repeat of
      // the row's own score leaves the maximum unchanged, and its exp is
      // dropped from the sum below
#pragma unroll
      for (int u = 0; u < GRAD_JA; ++u) x[u] = a.F[(int64_t)(j0 + u < d ? j0 + u : d - 1) * a.ld_f + rc];
      float cm = x[0];
#pragma unroll
      for (int u = 1; u < GRAD_JA; ++u) cm = fmaxf(cm, x[u]);
      const float mn = fmaxf(m, cm);
      float add = 0.0f;
#pragma unroll
      for (int u = 0; u < GRAD_JA; ++u) add += (j0 + u < d) ? expf(x[u] - mn) : 0.0f;
      s = s * expf(m - mn) + add;
      m = mn;
    }
    inv = 1.0f / s;
  }
  float hsum = 0.0f;
  for (int j0 = 0; j0 < d; j0 += GRAD_JC) {
    float x[GRAD_JC];
#pragma unroll
    for (int u = 0; u < GRAD_JC; ++u) x[u] = a.F[(int64_t)(j0 + u < d ? j0 + u : d - 1) * a.ld_f + rc];
    uint8_t yb[GRAD_JC];
    if constexpr (LOSS == SB_LOSS_SIGMOID_BCE) {
#pragma unroll
      for (int u = 0; u < GRAD_JC; ++u) yb[u] = a.Y[(int64_t)(j0 + u < d ? j0 + u : d - 1) * a.ld_y + rc];
    }
#pragma unroll
    for (int u = 0; u < GRAD_JC; ++u) {
      const int j = j0 + u;
      const int jj = j < d ? j : d - 1;
      float g, hh;
      if constexpr (LOSS == SB_LOSS_SOFTMAX_CE) {
        const float p = expf(x[u] - m) * inv;
        g = (jj == y) ? p - 1.0f : p;
        hh = p * (1.0f - p);
      } else {
        // e = exp(-|a|) never overflows, so s keeps its relative accuracy
        // for scores far below zero (down to fp32's subnormals)
        const float e = expf(-fabsf(x[u]));
        const float sg = (x[u] >= 0.0f ? 1.0f : e) / (1.0f + e);
        g = sg - (float)yb[u];
        hh = sg * (1.0f - sg);
      }
      if (ok) {
        a.G[(int64_t)jj * a.ld_g + row] = g;
        if (HESS) a.hess[(int64_t)jj * a.ld_h + row] = hh;
      }
      hsum += (j < d) ? hh : 0.0f;
      gbuf[u][tid] = ok ? g : 0.0f;
    }
    add_norms(a, gbuf, base, d, j0);
  }
  if (a.h_row && ok) a.h_row[row] = hsum * (1.0f / (float)d);
}

template <int LOSS>
__global__ void __launch_bounds__(GRAD_THREADS) k_grad(GradArgs a) {
  __shared__ __align__(16) float gbuf[GRAD_JC][GRAD_THREADS];
  for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
    int d = a.d;
    asm volatile("" : "+s"(d));
    const int64_t base = (int64_t)tile * GRAD_THREADS;
    const bool full = base + GRAD_THREADS <= a.n;
    if (a.hess) {
      if (full) grad_tile<LOSS, true, true>(a, gbuf, base, d);
      else grad_tile<LOSS, false, true>(a, gbuf, base, d);
    } else {
      if (full) grad_tile<LOSS, true, false>(a, gbuf, base, d);
      else grad_tile<LOSS, false, false>(a, gbuf, base, d);
    }
  }
}

// The sigmoid loss at the updated scores, one pass: the update of the previous
// tree (as k_update) and the derivatives (as k_grad) of a chunk of 16 columns
// for every tile of the block, then the next chunk, so that lr * V of the
// chunk is staged in LDS once per block (leaf-major with an odd stride).  F is
// read once: 300,001 rows x 203 outputs, 128 leaves, 273 us for k_update and
// k_grad, 228 us here.  The row sums of the hessians wait in h_row between the
// chunks (fp32, as in k_grad's register).
template <bool FULL, bool HESS>
__device__ inline void update_sigmoid_tile(const GradArgs& a, float (*gbuf)[GRAD_THREADS], const double* lv,
                                           int64_t base, int d, int j0) {
  const int tid = threadIdx.x;
  const int64_t row = base + tid;
  const bool ok = FULL || row < a.n;
  const int loc = ok ? tid : (int)(a.n - 1 - base);  // rows past the end read row n-1 and store nothing
  // column u's offset is u leading dimensions, capped at column d-1 (columns
  // past d, in the last chunk only, repeat it and store its own values there);
  // the addresses are a uniform base and the lane's 32-bit offset
  const int last = d - 1 - j0;
  const float* Fb = a.F + (int64_t)j0 * a.ld_f + base;
  const uint8_t* Yb = a.Y + (int64_t)j0 * a.ld_y + base;
  float x[GRAD_JC];
  uint8_t yb[GRAD_JC];
#pragma unroll
  for (int u = 0; u < GRAD_JC; ++u) {
    x[u] = Fb[loc];
    if (u < last) Fb += a.ld_f;
  }
#pragma unroll
  for (int u = 0; u < GRAD_JC; ++u) {
    yb[u] = Yb[loc];
    if (u < last) Yb += a.ld_y;
  }
  int L = a.ids[base + loc];
  L = L < a.n_leaves ? L : a.n_leaves - 1;
  const double* lvL = lv + L * (GRAD_JC + 1);
  float hsum = a.h_row && j0 > 0 ? a.h_row[base + loc] : 0.0f;
  float* Fw = a.F_upd + (int64_t)j0 * a.ld_f + base;
  float* Gw = a.G + (int64_t)j0 * a.ld_g + base;
  float* Hw = HESS ? a.hess + (int64_t)j0 * a.ld_h + base : nullptr;
#pragma unroll
  for (int u = 0; u < GRAD_JC; ++u) {
    const float f = (float)((double)x[u] + lvL[u]);
    const float e = expf(-fabsf(f));
    const float sg = (f >= 0.0f ? 1.0f : e) / (1.0f + e);
    const float g = sg - (float)yb[u];
    const float hh = sg * (1.0f - sg);
    if (ok) {
      Fw[tid] = f;
      Gw[tid] = g;
      if (HESS) Hw[tid] = hh;
    }
    if (u < last) {
      Fw += a.ld_f;
      Gw += a.ld_g;
      if (HESS) Hw += a.ld_h;
    }
    hsum += (u <= last) ? hh : 0.0f;
    gbuf[u][tid] = ok ? g : 0.0f;
  }
  add_norms(a, gbuf, base, d, j0);
  if (a.h_row && ok) a.h_row[row] = j0 + GRAD_JC < d ? hsum : hsum * (1.0f / (float)d);
}

// The block's tiles are t0, t0 + grid, ...: blocks go to the 8 XCDs in turn,
// and each XCD takes a run of neighbouring t0, because neighbouring tiles share
// cache lines where columns do not start on a line (n = 300,001: 243 us
// without, 227 us with, before; the other passes over F and G gain at some sizes and
// lose at others).  The launch has a multiple of 8 blocks.
__global__ void __launch_bounds__(GRAD_THREADS) k_update_sigmoid(GradArgs a, int grid) {
  __shared__ __align__(16) float gbuf[GRAD_JC][GRAD_THREADS];
  extern __shared__ double lv[];  // lr * V of the chunk, [leaf][GRAD_JC + 1]
  const int t0 = (int)(blockIdx.x & 7) * ((grid + 7) >> 3) + (int)(blockIdx.x >> 3);
  if (t0 >= grid) return;
  for (int j0 = 0; j0 < a.d; j0 += GRAD_JC) {
    __syncthreads();  // the previous chunk's readers are done
    for (int e = threadIdx.x; e < a.n_leaves * GRAD_JC; e += GRAD_THREADS) {
      const int L = e / GRAD_JC, u = e % GRAD_JC;
      lv[L * (GRAD_JC + 1) + u] = a.lr * a.V[(int64_t)L * a.ld_v + (j0 + u < a.d ? j0 + u : a.d - 1)];
    }
    __syncthreads();
    for (int tile = t0; tile < a.n_tiles; tile += grid) {
      int d = a.d;
      asm volatile("" : "+s"(d));
      const int64_t base = (int64_t)tile * GRAD_THREADS;
      const bool full = base + GRAD_THREADS <= a.n;
      if (a.hess) {
        if (full) update_sigmoid_tile<true, true>(a, gbuf, lv, base, d, j0);
        else update_sigmoid_tile<false, true>(a, gbuf, lv, base, d, j0);
      } else {
        if (full) update_sigmoid_tile<true, false>(a, gbuf, lv, base, d, j0);
        else update_sigmoid_tile<false, false>(a, gbuf, lv, base, d, j0);
      }
    }
  }
}

// Softmax cross-entropy with the row's d <= DMAX scores held in registers:
// F is read once.  Columns past d load column d-1 (the maximum is unchanged
// and the sum skips them), so every load is unconditional and all of them
// are in flight together.  The maximum is exact, the sum of exp(a - max) is
// taken in column order and its terms are kept for p = exp(a - max) / sum,
// then the second half as in k_grad (stores, the hessians and the
// column-norm staging).  The grid holds as many blocks as fit on the GPU at
// once, each looping over tiles, so no last round of blocks runs part-empty.
//
// The column count d reaches this function opaque to the compiler, and is
// made opaque again between the loads and the stores, so that the
// per-column tests j < d (uniform lane masks) and column offsets are formed
// where they are used instead of all at once and held, spilled, across a
// phase or the tile loop.  Columns past d stay on column d-1 and store
// column d-1's own values there (same address, same value), so the stores
// need no branch; a full tile stores without a row guard.
template <int DMAX, bool FULL, bool HESS, bool UPD>
__device__ inline void grad_softmax_tile(const GradArgs& a, float (*gbuf)[GRAD_THREADS], const double* lv,
                                         int64_t base, int64_t ld_f, int64_t ld_g, int64_t ld_h, int d) {
  const int tid = threadIdx.x;
  const int64_t row = base + tid;
  const bool ok = FULL || row < a.n;
  const int loc = ok ? tid : (int)(a.n - 1 - base);  // rows past the end read row n-1 and store nothing
  const int y = a.labels[base + loc];
  const float* Fb = a.F + base;
  float x[DMAX];
#pragma unroll
  for (int j = 0; j < DMAX; ++j) x[j] = Fb[(int64_t)(j < d ? j : d - 1) * ld_f + loc];
  if constexpr (UPD) {
    // the update of the previous tree, as k_update: fp64 sum, rounded once;
    // columns past d repeat column d-1 and store its own value there
    int L = a.ids[base + loc];
    L = L < a.n_leaves ? L : a.n_leaves - 1;
    const double* lvL = lv + L * a.lv_stride;
    asm volatile("" : "+s"(d));
#pragma unroll
    for (int j = 0; j < DMAX; ++j) x[j] = (float)((double)x[j] + lvL[j < d ? j : d - 1]);
    asm volatile("" : "+s"(d));
    float* Fw = a.F_upd + base;
#pragma unroll
    for (int j = 0; j < DMAX; ++j)
      if (ok) Fw[(int64_t)(j < d ? j : d - 1) * ld_f + tid] = x[j];
    asm volatile("" : "+s"(d));
  }
  float m = x[0];
#pragma unroll
  for (int j = 1; j < DMAX; ++j) m = fmaxf(m, x[j]);
  // x[j] becomes exp(x[j] - max), reused for p below
  float s = 0.0f;
#pragma unroll
  for (int j = 0; j < DMAX; ++j) {
    x[j] = expf(x[j] - m);
    s += (j < d) ? x[j] : 0.0f;
  }
  const float inv = 1.0f / s;
  float hsum = 0.0f;
  asm volatile("" : "+s"(d));
  float* Gb = a.G + base;
  float* Hb = HESS ? a.hess + base : nullptr;
#pragma unroll
  for (int j0 = 0; j0 < DMAX; j0 += GRAD_JC) {
    if (j0 >= d) break;
#pragma unroll
    for (int u = 0; u < GRAD_JC; ++u) {
      const int j = j0 + u;
      const int jj = j < d ? j : d - 1;
      const float p = x[j] * inv;
      const float hh = p * (1.0f - p);
      const float g = (jj == y) ? p - 1.0f : p;
      if (ok) {
        Gb[(int64_t)jj * ld_g + tid] = g;
        if (HESS) Hb[(int64_t)jj * ld_h + tid] = hh;
      }
      hsum += (j < d) ? hh : 0.0f;
      gbuf[u][tid] = ok ? g : 0.0f;
    }
    add_norms(a, gbuf, base, d, j0);
  }
  if (a.h_row && ok) a.h_row[row] = hsum * (1.0f / (float)d);
}

template <int DMAX, bool UPD>
__global__ void __launch_bounds__(GRAD_THREADS) k_grad_softmax_regs(GradArgs a) {
  __shared__ __align__(16) float gbuf[GRAD_JC][GRAD_THREADS];
  extern __shared__ double lv[];  // UPD: lr * V, [leaf][lv_stride]
  if constexpr (UPD) {
    for (int e = threadIdx.x; e < a.n_leaves * a.d; e += GRAD_THREADS) {
      const int L = e / a.d, j = e - L * a.d;
      lv[L * a.lv_stride + j] = a.lr * a.V[(int64_t)L * a.ld_v + j];
    }
    __syncthreads();
  }
  for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
    const int64_t ld_f = a.ld_f, ld_g = a.ld_g, ld_h = a.ld_h;
    // d as seen by the compiler changes at every tile: the per-column tests
    // j < d are made where they are used, not hoisted out of the tile loop
    // as DMAX lane masks held (spilled) across it
    int d = a.d;
    asm volatile("" : "+s"(d));
    const int64_t base = (int64_t)tile * GRAD_THREADS;
    const bool full = base + GRAD_THREADS <= a.n;
    if (a.hess) {
      if (full) grad_softmax_tile<DMAX, true, true, UPD>(a, gbuf, lv, base, ld_f, ld_g, ld_h, d);
      else grad_softmax_tile<DMAX, false, true, UPD>(a, gbuf, lv, base, ld_f, ld_g, ld_h, d);
    } else {
      if (full) grad_softmax_tile<DMAX, true, false, UPD>(a, gbuf, lv, base, ld_f, ld_g, ld_h, d);
      else grad_softmax_tile<DMAX, false, false, UPD>(a, gbuf, lv, base, ld_f, ld_g, ld_h, d);
    }
  }
}

// Softmax cross-entropy of wide rows (104 < d <= 1024): the scores of ROWS rows
// stay in the registers of one block, WIDE_C = 32 columns per lane, so F is
// read once (the two-pass kernel above reads it twice: 700,001 x 200 399 us, 290 us
// here; 300,007 x 1000 854 us, 703 us here).  Up to 512 columns a wave takes 64
// rows x 32 columns; past that 32 rows x 64 columns, its upper 32 lanes the
// second 32 columns, so that 16 waves reach 1024 (64 columns per lane need more
// than the 128 registers that 16 waves have: spilled, 1722 us).  The waves'
// maxima and sums of exp(a - max) meet in LDS (two barriers per tile that wait
// for LDS operations only).  While a tile's gradients go out, column by column,
// the same register takes the column's score of the block's next tile, so the
// loads are in flight across the barriers and the stores.
//
// Column norms: the squares of columns c and c + 16 meet by exchanging rows of
// 16 lanes (v_permlane16_swap: a lane ends with two rows' squares of one of the
// two columns), and the 16 fp64 sums of a tile by exchanging half of the
// remaining columns with the partner lane (DPP mirrors and quad permutations),
// so lane l ends with column l mod 32's sum over its rows, in a fixed order, and
// adds it to its own fp64 total over the block's tiles.  Block b's totals are
// partial b.
// v[0..N): the lane keeps the half of the columns that its bit names, adds the
// partner's values of them and passes the other half on.
template <int CTRL, int N>
__device__ inline void exchange_half(double (&v)[16], bool upper) {
#pragma unroll
  for (int c = 0; c < N / 2; ++c) {
    const double keep = upper ? v[c + N / 2] : v[c];
    const double send = upper ? v[c] : v[c + N / 2];
    v[c] = keep + dpp_f64<CTRL>(send);
  }
}
__device__ inline void swap_rows(float& x, float& y) {  // x's odd rows of 16 lanes <-> y's even rows
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}

// lane offsets within a wave's columns are 32-bit byte offsets
constexpr int64_t WIDE_MAX_LD = int64_t(1) << 24;

__device__ inline float load_at(const float* base, uint32_t bytes) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + bytes);
}
__device__ inline void store_at(float* base, uint32_t bytes, float v) {
  *reinterpret_cast<float*>(reinterpret_cast<char*>(base) + bytes) = v;
}

// FULLC: all columns of the wave exist; else those past d - 1 load column d - 1
// and are dropped.
template <int ROWS, bool FULLC, bool HESS>
__device__ __forceinline__ void softmax_wide_wave(const GradArgs& a, float (*sred)[WIDE_MAX_WAVES][64], int nw, int w,
                                                  int bx, int grid, int tiles) {
  constexpr int PARTS = 64 / ROWS;  // lanes of a row
  const uint32_t lane = threadIdx.x & 63, rl = lane & (ROWS - 1);
  const int hb = PARTS == 1 ? 0 : (int)(lane >> 5);
  const int j0 = w * WIDE_C * PARTS, c0 = hb * WIDE_C;  // the wave's first column, the lane's first from there
  const int last = a.d - 1 - j0;                        // the wave's last column, from j0
  // A column's address is a uniform base that steps by the leading dimension
  // and the lane's byte offset: its row and, for the upper half, 32 columns.
  // Where those columns do not all exist the offset of slot i is capped at the
  // wave's last column (uniform bases alone serve one column set per wave).
  constexpr bool STEP = FULLC || PARTS == 1;
  auto at = [&](int i, int cl, uint32_t row, int64_t ld) -> uint32_t {
    if (PARTS == 1) return 4 * row;
    if (FULLC) return 4 * (row + (uint32_t)cl * (uint32_t)ld);
    const int c = cl + i < last ? cl + i : last;
    return 4 * (row + (uint32_t)c * (uint32_t)ld);
  };
  auto rows_of = [&](int tile, int64_t& base, uint32_t& loc) {
    base = (int64_t)tile * ROWS;
    const int64_t left = a.n - 1 - base;  // rows past the end read row n-1
    loc = rl < left ? rl : (uint32_t)left;
  };
  int64_t base;
  uint32_t loc;
  rows_of(bx, base, loc);
  int y = a.labels[base + loc] - j0 - c0;
  float x[WIDE_C];
  {
    const float* p = a.F + (int64_t)j0 * a.ld_f + base;
#pragma unroll
    for (int i = 0; i < WIDE_C; ++i) {
      x[i] = load_at(p, at(i, c0, loc, a.ld_f));
      if (STEP && (FULLC || i < last)) p += a.ld_f;
    }
  }
  double total = 0.0;
  for (int tile = bx; tile < tiles; tile += grid) {
    const bool ok = base + rl < a.n;
    float m4[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
    for (int i = 4; i < WIDE_C; ++i) m4[i & 3] = fmaxf(m4[i & 3], x[i]);
    float m = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
    sred[0][w][lane] = m;
    lds_barrier();
    for (int u = 0; u < nw; ++u)
#pragma unroll
      for (int h = 0; h < PARTS; ++h) m = fmaxf(m, sred[0][u][ROWS * h + rl]);
    // x[i] becomes exp(x[i] - max), reused for p below
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < WIDE_C; ++i) {
      x[i] = expf(x[i] - m);
      s += (FULLC || c0 + i <= last) ? x[i] : 0.0f;
    }
    sred[1][w][lane] = s;
    lds_barrier();
    s = 0.0f;
    for (int u = 0; u < nw; ++u)
#pragma unroll
      for (int h = 0; h < PARTS; ++h) s += sred[1][u][ROWS * h + rl];
    const float inv = 1.0f / s;
    float hsum = 0.0f;
    // the next tile (past the last: this one again, not used)
    int64_t nbase;
    uint32_t nloc;
    rows_of(tile + grid < tiles ? tile + grid : tile, nbase, nloc);
    const int ny = a.labels[nbase + nloc] - j0 - c0;
    // the columns' addresses step by the leading dimensions, which the compiler
    // sees anew at every step: it would otherwise form all column offsets
    // before the tile loop and hold them, spilled, across it
    int64_t ld_f = a.ld_f, ld_g = a.ld_g, ld_h = a.ld_h;
    const float* Fc[2];
    float *Gc[2], *Hc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int jq = j0 + (!STEP ? 0 : FULLC || 16 * q < last ? 16 * q : last);
      Fc[q] = a.F + (int64_t)jq * ld_f + nbase;
      Gc[q] = a.G + (int64_t)jq * ld_g + base;
      Hc[q] = HESS ? a.hess + (int64_t)jq * ld_h + base : nullptr;
    }
    double v[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      float g2[2];
      asm volatile("" : "+s"(ld_f), "+s"(ld_g));
      if (HESS) asm volatile("" : "+s"(ld_h));
      int cl = c0;  // as the leading dimensions
      if (!STEP) asm volatile("" : "+v"(cl));
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int i = c + 16 * q;
        const bool live = ok && (FULLC || cl + i <= last);
        const float p = x[i] * inv;
        const float g = i == y ? p - 1.0f : p;
        const float hh = p * (1.0f - p);
        if (live) {
          store_at(Gc[q], at(i, cl, rl, ld_g), g);
          if (HESS) store_at(Hc[q], at(i, cl, rl, ld_h), hh);
          hsum += hh;
        }
        g2[q] = live ? g : 0.0f;
        x[i] = load_at(Fc[q], at(i, cl, nloc, ld_f));
        if (STEP && (FULLC || i < last)) {
          Fc[q] += ld_f;
          Gc[q] += ld_g;
          if (HESS) Hc[q] += ld_h;
        }
      }
      swap_rows(g2[0], g2[1]);
      v[c] = (double)g2[0] * g2[0] + (double)g2[1] * g2[1];
    }
    exchange_half<0x140, 16>(v, lane & 8);  // row_mirror: the partner differs in bit 3 (and below)
    exchange_half<0x141, 8>(v, lane & 4);   // row_half_mirror: in bit 2 (and below)
    exchange_half<0x4e, 4>(v, lane & 2);    // quad_perm [2, 3, 0, 1]
    exchange_half<0xb1, 2>(v, lane & 1);    // quad_perm [1, 0, 3, 2]
    total += v[0];
    if (a.h_row) {
      sred[2][w][lane] = hsum;
      lds_barrier();
      if (w == 0 && hb == 0 && ok) {
        float hs = 0.0f;
        for (int u = 0; u < nw; ++u)
#pragma unroll
          for (int h = 0; h < PARTS; ++h) hs += sred[2][u][ROWS * h + rl];
        a.h_row[base + rl] = hs * (1.0f / (float)a.d);
      }
    }
    base = nbase;
    loc = nloc;
    y = ny;
  }
  if constexpr (PARTS == 1) total += __shfl_xor(total, 32, 64);  // the rows of the other half
  const int col = j0 + (int)(PARTS == 1 ? (lane & 31) : lane);
  if (a.npart && lane < 32 * PARTS && col < a.d) a.npart[(int64_t)col * a.n_parts + bx] = total;
}

// Five waves per SIMD: with hessians and 32 rows the compiler otherwise takes 97
// registers, one too many, and a CU holds one block of 9 or 10 waves instead of two.
template <int ROWS, bool HESS>
__global__ void __launch_bounds__(64 * WIDE_MAX_WAVES)
k_grad_softmax_wide(GradArgs a, int grid, int tiles) {
  __shared__ float sred[3][WIDE_MAX_WAVES][64];
  // each XCD takes a run of neighbouring tiles (see k_update_sigmoid)
  const int bx = (int)(blockIdx.x & 7) * ((grid + 7) >> 3) + (int)(blockIdx.x >> 3);
  if (bx >= grid) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  constexpr int WC = WIDE_C * (64 / ROWS);
  if ((w + 1) * WC <= a.d) softmax_wide_wave<ROWS, true, HESS>(a, sred, nw, w, bx, grid, tiles);
  else softmax_wide_wave<ROWS, false, HESS>(a, sred, nw, w, bx, grid, tiles);
}

// One wave per column: lane l adds partials l, l+64, ... in order, then a fixed butterfly.
__global__ void __launch_bounds__(256) k_grad_norm_final(const double* __restrict__ npart, int32_t d, int32_t parts,
                                                         double* __restrict__ norm2) {
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (j >= d) return;
  double s = lane_strided_sum(npart + (int64_t)j * parts, parts, lane);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) norm2[j] = s;
}

struct UpdArgs {
  float* F;
  int64_t n;
  int32_t d;
  int64_t ld_f;
  const void* ids;
  int32_t n_leaves;
  const double* V;
  int64_t ld_v;
  double lr;
  int32_t jc;  // columns per chunk
  int32_t n_tiles;
};

template <typename LT>
__global__ void __launch_bounds__(UPD_THREADS) k_update(UpdArgs a) {
  // lr * V of the chunk's columns, leaf-major with an odd stride (jc + 1
  // doubles) so that lanes of different leaves fall on different banks
  extern __shared__ double lv[];
  const LT* ids = static_cast<const LT*>(a.ids);
  const int top = a.n_leaves - 1;
  const int stride = a.jc + 1;
  for (int j0 = 0; j0 < a.d; j0 += a.jc) {
    const int w = (a.d - j0 < a.jc) ? a.d - j0 : a.jc;
    __syncthreads();  // the previous chunk's readers are done
    for (int e = threadIdx.x; e < a.n_leaves * a.jc; e += UPD_THREADS) {
      const int L = e / a.jc, u = e - L * a.jc;
      lv[L * stride + u] = u < w ? a.lr * a.V[(int64_t)L * a.ld_v + j0 + u] : 0.0;
    }
    __syncthreads();
    for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
      const int64_t row = (int64_t)tile * UPD_THREADS + threadIdx.x;
      const bool ok = row < a.n;
      const int64_t rc = ok ? row : a.n - 1;
      int L = (int)ids[rc];
      L = L > top ? top : L;
      const double* lvL = lv + L * stride;
      // every load of the chunk first (columns past w repeat the last one),
      // then the sums and the stores
      float f[UPD_JC];
#pragma unroll
      // streamed once (non-temporal): 301 us instead of 328 us at 2M x 100
      for (int u = 0; u < UPD_JC; ++u) f[u] = ld_stream(a.F + (int64_t)(j0 + (u < w ? u : w - 1)) * a.ld_f + rc);
#pragma unroll
      for (int u = 0; u < UPD_JC; ++u)
        if (u < w && ok) a.F[(int64_t)(j0 + u) * a.ld_f + row] = (float)((double)f[u] + lvL[u]);
    }
  }
}

// Blocks of a kernel that fit on the current device at once (at least 1),
// with lds bytes of dynamic LDS per block.
template <typename K>
int resident_blocks(K kernel, int threads, size_t lds = 0) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, lds) != hipSuccess)
    return GRAD_PARTS;
  const int r = cus * per;
  return r > 0 ? r : 1;
}

// Largest lr * V table (n_leaves x lv_stride doubles) the fused update takes.
constexpr int64_t UPDGRAD_LDS_BYTES = 64 * 1024;

// Grid of a gradient launch over `tiles` tiles, at most `cap` blocks: one
// block per tile up to GRAD_PARTS tiles, else the largest divisor of
// GRAD_PARTS within the cap, so that block b owns the slots b mod grid.
int grad_grid(int64_t tiles, int cap) {
  if (tiles <= GRAD_PARTS) return (int)tiles;
  int g = cap < GRAD_PARTS ? (cap > 1 ? cap : 1) : GRAD_PARTS;
  while (GRAD_PARTS % g) --g;
  return g;
}

// The register softmax kernel for d <= 104, with or without the update (lds:
// the update's table).  Where the rows are wide (DMAX = 104) or the update's
// table takes LDS, the grid is capped at the blocks that fit at once, each
// looping over tiles.
template <bool UPD>
void launch_softmax_regs(const GradArgs& a, size_t lds, hipStream_t st) {
  auto grid = [&](auto kernel, bool wide) {
    if (!wide && !UPD) return grad_grid(a.n_tiles, GRAD_PARTS);
    static thread_local size_t fit_lds = ~size_t(0);  // per-thread cache of the occupancy query
    static thread_local int fit = 0;
    if (fit_lds != lds) {
      fit = resident_blocks(kernel, GRAD_THREADS, lds);
      fit_lds = lds;
    }
    return grad_grid(a.n_tiles, fit);
  };
  if (a.d <= 16) {
    const int b = grid(k_grad_softmax_regs<16, UPD>, false);
    hipLaunchKernelGGL((k_grad_softmax_regs<16, UPD>), dim3(b), dim3(GRAD_THREADS), lds, st, a);
  } else if (a.d <= 32) {
    const int b = grid(k_grad_softmax_regs<32, UPD>, false);
    hipLaunchKernelGGL((k_grad_softmax_regs<32, UPD>), dim3(b), dim3(GRAD_THREADS), lds, st, a);
  } else if (a.d <= 64) {
    const int b = grid(k_grad_softmax_regs<64, UPD>, false);
    hipLaunchKernelGGL((k_grad_softmax_regs<64, UPD>), dim3(b), dim3(GRAD_THREADS), lds, st, a);
  } else {
    const int b = grid(k_grad_softmax_regs<104, UPD>, true);
    hipLaunchKernelGGL((k_grad_softmax_regs<104, UPD>), dim3(b), dim3(GRAD_THREADS), lds, st, a);
  }
}

// The register softmax kernel for 104 < d <= 1024, split by wide_plan(); returns
// the blocks, the partials' stride.
int launch_softmax_wide(GradArgs a, hipStream_t st) {
  const WidePlan p = wide_plan(a.n, a.d, a.n_parts);
  const int threads = 64 * p.waves, grid = p.grid, tiles = p.tiles;
  a.n_parts = grid;
  const dim3 blocks((grid + 7) / 8 * 8);
#define SB_WIDE(R, H) hipLaunchKernelGGL((k_grad_softmax_wide<R, H>), blocks, dim3(threads), 0, st, a, grid, tiles)
  if (p.rows == 64) { if (a.hess) SB_WIDE(64, true); else SB_WIDE(64, false); }
  else if (a.hess) SB_WIDE(32, true);
  else SB_WIDE(32, false);
#undef SB_WIDE
  return grid;
}

}  // namespace

int64_t grad_ws_bytes(int64_t n, int32_t d) {
  const int64_t tiles = (n + GRAD_THREADS - 1) / GRAD_THREADS;
  return align256((int64_t)d * (tiles < GRAD_PARTS ? tiles : GRAD_PARTS) * 8);
}

int32_t launch_gradients(int32_t loss, const float* F, int64_t n, int32_t d, int64_t ld_f, const int32_t* labels,
                         const uint8_t* Y, int64_t ld_y, float* G, int64_t ld_g, float* hess, int64_t ld_hess,
                         float* h_row, double* norm2, void* ws, hipStream_t st) {
  const int64_t tiles = (n + GRAD_THREADS - 1) / GRAD_THREADS;
  const int parts = (int)(tiles < GRAD_PARTS ? tiles : GRAD_PARTS);
  double* npart = norm2 ? static_cast<double*>(ws) : nullptr;
  GradArgs a{loss, F, n, d, ld_f, labels, Y, ld_y, G, ld_g, hess, ld_hess, h_row, npart, (int32_t)tiles, parts};
  const int blocks = grad_grid(tiles, GRAD_PARTS);
  if (loss == SB_LOSS_SOFTMAX_CE && d <= 104)
    launch_softmax_regs<false>(a, 0, st);
  else if (loss == SB_LOSS_SOFTMAX_CE && d <= WIDE_MAX_D && ld_f < WIDE_MAX_LD && ld_g < WIDE_MAX_LD &&
           (!hess || ld_hess < WIDE_MAX_LD))
    a.n_parts = launch_softmax_wide(a, st);
  else if (loss == SB_LOSS_SOFTMAX_CE)
    hipLaunchKernelGGL(k_grad<SB_LOSS_SOFTMAX_CE>, dim3(blocks), dim3(GRAD_THREADS), 0, st, a);
  else
    hipLaunchKernelGGL(k_grad<SB_LOSS_SIGMOID_BCE>, dim3(blocks), dim3(GRAD_THREADS), 0, st, a);
  if (norm2) hipLaunchKernelGGL(k_grad_norm_final, dim3((d + 3) / 4), dim3(256), 0, st, npart, d, a.n_parts, norm2);
  return check_launch("sb_gradients");
}

int64_t update_ws_bytes(int64_t n) { return leaf_ids_bytes(n); }

int32_t launch_update(float* F, int64_t n, int32_t d, int64_t ld_f, const int32_t* row_idx, const int32_t* leaf_off,
                      int32_t n_leaves, const double* V, int64_t ld_v, double lr, void* ws, hipStream_t st) {
  const int64_t tiles = (n + UPD_THREADS - 1) / UPD_THREADS;
  const int blocks = (int)(tiles < UPD_MAX_BLOCKS ? tiles : UPD_MAX_BLOCKS);
  int jc = UPD_LDS_DOUBLES / n_leaves - 1;  // (jc + 1) doubles per leaf
  if (jc > UPD_JC) jc = UPD_JC;
  if (jc > d) jc = d;
  launch_leaf_ids(row_idx, leaf_off, n_leaves, n, ws, st);
  const UpdArgs a{F, n, d, ld_f, ws, n_leaves, V, ld_v, lr, jc, (int32_t)tiles};
  const size_t lds = (size_t)n_leaves * (jc + 1) * 8;
  if (n_leaves <= 256)
    hipLaunchKernelGGL(k_update<uint8_t>, dim3(blocks), dim3(UPD_THREADS), lds, st, a);
  else
    hipLaunchKernelGGL(k_update<uint16_t>, dim3(blocks), dim3(UPD_THREADS), lds, st, a);
  return check_launch("sb_update_predictions");
}

// Workspace: [norm partials (grad_ws_bytes)][leaf ids (update_ws_bytes)]
int64_t update_gradients_ws_bytes(int64_t n, int32_t d) { return grad_ws_bytes(n, d) + update_ws_bytes(n); }

int32_t launch_update_gradients(int32_t loss, float* F, int64_t n, int32_t d, int64_t ld_f, const int32_t* row_idx,
                                const int32_t* leaf_off, int32_t n_leaves, const double* V, int64_t ld_v, double lr,
                                const int32_t* labels, const uint8_t* Y, int64_t ld_y, float* G, int64_t ld_g,
                                float* hess, int64_t ld_hess, float* h_row, double* norm2, void* ws,
                                hipStream_t st) {
  char* w = static_cast<char*>(ws);
  void* ws_ids = w + grad_ws_bytes(n, d);
  const int stride = d | 1;  // odd: lanes of different leaves fall on different banks
  const int64_t table = (int64_t)n_leaves * stride * 8;
  const bool softmax_fused = loss == SB_LOSS_SOFTMAX_CE && d <= 104 && table <= UPDGRAD_LDS_BYTES;
  const size_t chunk_table = (size_t)n_leaves * (GRAD_JC + 1) * 8;  // at most 34 KB
  if (n_leaves > 256 || !(softmax_fused || loss == SB_LOSS_SIGMOID_BCE)) {
    const int32_t rc = launch_update(F, n, d, ld_f, row_idx, leaf_off, n_leaves, V, ld_v, lr, ws_ids, st);
    if (rc) return rc;
    return launch_gradients(loss, F, n, d, ld_f, labels, Y, ld_y, G, ld_g, hess, ld_hess, h_row, norm2, ws, st);
  }
  launch_leaf_ids(row_idx, leaf_off, n_leaves, n, ws_ids, st);
  const int64_t tiles = (n + GRAD_THREADS - 1) / GRAD_THREADS;
  const int parts = (int)(tiles < GRAD_PARTS ? tiles : GRAD_PARTS);
  double* npart = norm2 ? reinterpret_cast<double*>(w) : nullptr;
  GradArgs a{loss, F, n, d, ld_f, labels, Y, ld_y, G, ld_g, hess, ld_hess, h_row, npart, (int32_t)tiles, parts};
  a.F_upd = F;
  a.ids = static_cast<const uint8_t*>(ws_ids);
  a.n_leaves = n_leaves;
  a.lv_stride = stride;
  a.V = V;
  a.ld_v = ld_v;
  a.lr = lr;
  if (loss == SB_LOSS_SIGMOID_BCE) {
    // the chunk's table is staged by every block: up to two tiles per block
    // where one each would give more blocks than run at once
    const int per = (int)((tiles + UPD_SIG_BLOCKS - 1) / UPD_SIG_BLOCKS);
    const int grid = tiles <= GRAD_PARTS ? (int)((tiles + per - 1) / per) : grad_grid(tiles, UPD_SIG_BLOCKS);
    hipLaunchKernelGGL(k_update_sigmoid, dim3((grid + 7) / 8 * 8), dim3(GRAD_THREADS), chunk_table, st, a, grid);
  } else {
    launch_softmax_regs<true>(a, (size_t)table, st);
  }
  if (norm2) hipLaunchKernelGGL(k_grad_norm_final, dim3((d + 3) / 4), dim3(256), 0, st, npart, d, parts, norm2);
  return check_launch("sb_update_and_gradients");
}

}  // namespace sb
