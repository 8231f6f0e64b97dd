// Multislice passes over batches of parent columns (step a).
//
// A slice step psi <- F^-1[P F[T_j psi]] (eq. propagator, eq.
// smatrix-advance) is split into two HBM passes over the column stack:
//   row pass:    [row inverse FFT] -> [window gather] -> x T_j -> [gather]
//                -> [row FFT]
//   column pass: column FFT -> x P(q)/G -> column inverse FFT
// Between passes the state is kept row-transformed (F_row psi), so a row pass
// fuses the inverse row transform of one step with the forward row transform
// of the next, and the real-space wave is only ever materialized in
// registers -- which is where the ionized atoms' windows are cropped.  The S2
// sweep (transpose multislice, eq. s2) runs the same passes in the other
// order (column pass, then row pass with T after the propagation).
#include "fft_core.h"

#include <algorithm>

namespace bip {

namespace {

template <int NX>
struct RowShape {
  static constexpr int T = NX / 16;            // threads per row transform
  static constexpr int ROWS = 256 / T;         // rows per block
  static constexpr int LDS_ROW = NX + NX / 16; // padded complex elements per row
};

constexpr int GREC_LDS = 64;  // gather records of a plane staged in LDS

// Crop the real-space row segment that falls into the windows of the atoms
// of this plane; de-tilt by exp(-sign 2 pi i h_p.r/N) on the way.  Records
// q < GREC_LDS come from LDS, the rest from memory.
template <int NX>
__device__ inline void gather_row(const float2 (&v)[16], int t, int y, int col, int ny,
                                  const GatherArgs& ga, const GatherRec* srec, int gb, int ge,
                                  int2 hp, const float2* __restrict__ tw, int L, int sign) {
  constexpr int T = RowShape<NX>::T;
  const int my = hp.x * y * (L / ny);
  for (int q = 0; q < ge - gb; ++q) {
    const GatherRec g = q < GREC_LDS ? srec[q] : ga.rec[gb + q];
    int ry = y - g.oy;
    if (ry < 0) ry += ny;
    if (ry >= g.W) continue;
    float2* dst = ga.win + g.off + ((int64_t)col * g.W + ry) * g.W;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int x = t + T * e;
      int rx = x - g.ox;
      if (rx < 0) rx += NX;
      if (rx < g.W) {
        const int m = (my + hp.y * x * (L / NX)) & (L - 1);
        const float2 w = tw[m];  // exp(-2 pi i h_p.r/N)
        dst[rx] = sign > 0 ? cmul(v[e], w) : cmulc(v[e], w);
      }
    }
  }
}

// A batch may hold the last columns of S1 and the first of S2, each workgroup on a
// column of either (ROW_BOTH): the two sides advance side by side, so that a few
// columns share their launches, where that saves a batch.  256 x 256, 30 slices, hex
// parents: 57 + 58 passes of 15 us, 28 + 29 of 26 so; a map at f = 4, 50 slices: 4.95
// ms of passes, 4.42 so; two configurations of 20 slices: 16.3 and 15.9.
// A sweep of a plan without checkpoints starts with ROW_START, in registers: the
// S1 wave is a plane wave, and so is the S2 wave after its first propagation, so
// the state is neither written first nor read by this pass, and S2 needs no
// column pass before it.  (Plans with checkpoints start from a state written by
// launch_init_planewaves: a saved sum keeps its rounding.)  The last pass of a
// sweep stores no state and only transforms the rows that a window covers.
//   The sweeps' kernels took 53.9 ms with the stored start for 6 slices of 1024 x
// 1024 and 42.7 so, 169 and 159 for 16 of 512 x 512, 16.9 and 16.3 for 20 of 256 x 256.
template <int NX, int FLAGS>
__global__ __launch_bounds__(256, 4) void k_row_pass(float2* __restrict__ state, int ny,
                                                  const float2* __restrict__ T,
                                                  const float2* __restrict__ twg, int L,
                                                  const int2* __restrict__ parents, int sign,
                                                  GatherArgs ga, int gb, int ge, int col0,
                                                  float2* __restrict__ save, RowStart start, RowBoth both) {
  using S = RowShape<NX>;
  __shared__ float2 lds[S::ROWS * S::LDS_ROW];
  extern __shared__ float2 tw[];  // [L] twiddle table
  constexpr int GATHER = FLAGS & (ROW_GATHER_BEFORE_T | ROW_GATHER_AFTER_T | ROW_BOTH);
  __shared__ GatherRec srec[GATHER ? GREC_LDS : 1];
  if constexpr ((FLAGS & ROW_BOTH) != 0) {
    if ((int)blockIdx.y >= both.n1) {
      T = both.T;
      parents = both.parents;
      ga = both.ga;
      gb = both.gb;
      ge = both.ge;
      col0 = -both.n1;
      sign = -1;
    }
  }
  for (int i = threadIdx.x; i < L; i += 256) tw[i] = twg[i];
  if constexpr (GATHER != 0) {
    if ((int)threadIdx.x < ge - gb && threadIdx.x < GREC_LDS) srec[threadIdx.x] = ga.rec[gb + threadIdx.x];
  }
  // the only workgroup barrier: a row and its LDS row belong to one wave, so
  // the transforms order their exchanges per wave
  __syncthreads();
  const int t = threadIdx.x % S::T;
  const int f = threadIdx.x / S::T;
  const int y = blockIdx.x * S::ROWS + f;
  const int col = blockIdx.y;   // column of this launch's batch
  const int pcol = col0 + col;  // parent index
  if constexpr ((FLAGS & (ROW_FWD | ROW_SAVE)) == 0) {  // only the windows' rows are wanted
    bool any = false;
    for (int q = gb; q < ge; ++q) any |= ((y - ga.rec[q].oy) & (ny - 1)) < ga.rec[q].W;
    if (!any) return;
  }
  float2* row = state + ((int64_t)col * ny + y) * NX;
  float2* my_lds = lds + f * S::LDS_ROW;
  float2 v[16];
  if constexpr ((FLAGS & ROW_START) != 0) {
    const int2 hp = parents[pcol];
    float2 c = make_float2(1.f, 0.f);
    if (start.prop && sign < 0) c = cscale(start.prop[(-hp.x & (ny - 1)) * NX + (-hp.y & (NX - 1))], start.scale);
    const int my = hp.x * y * (L / ny);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float2 w = tw[(my + hp.y * (t + S::T * e) * (L / NX)) & (L - 1)];  // exp(-2 pi i h.r/N)
      v[e] = sign > 0 ? make_float2(w.x, -w.y) : cmul(c, w);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = row[t + S::T * e];
  }
  if (FLAGS & ROW_INV) fft::transform<NX, true, 1, true, true>(v, my_lds, t, tw, L);
  auto gather = [&] {
    if (ge > gb) gather_row<NX>(v, t, y, pcol, ny, ga, srec, gb, ge, parents[pcol], tw, L, sign);
  };
  auto times_T = [&] {
    const float2* Trow = T + (int64_t)y * NX;
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = cmul(v[e], Trow[t + S::T * e]);
  };
  if constexpr ((FLAGS & ROW_BOTH) != 0) {
    if (sign < 0) times_T();
    gather();
    if (sign > 0) times_T();
  } else {
    if constexpr ((FLAGS & ROW_GATHER_BEFORE_T) != 0) gather();
    if constexpr ((FLAGS & ROW_T) != 0) times_T();
  }
  if constexpr ((FLAGS & ROW_SAVE) != 0) {  // slice checkpoint: the state after T_j
    float2* srow = save + ((int64_t)col * ny + y) * NX;
#pragma unroll
    for (int e = 0; e < 16; ++e) srow[t + S::T * e] = v[e];
  }
  if constexpr ((FLAGS & ROW_GATHER_AFTER_T) != 0) gather();
  if (FLAGS & ROW_FWD) {
    // Above 256 the twiddles are read again: kept from the inverse transform they
    // took 142 to 180 registers, two or three waves a SIMD (in 235 MB batches, 16
    // slices of 512: 83.3 us, 78.0 so; 6 of 1024: 103.3 and 86.7.  With 100 slices of
    // 512 and 20 windows a plane the tables and the windows share the cache with the
    // state: 114 us).
    int tf = t;
    if constexpr (NX > 256) asm volatile("" : "+v"(tf));
    fft::transform<NX, false, 1, true, true>(v, my_lds, tf, tw, L);
#pragma unroll
    for (int e = 0; e < 16; ++e) row[t + S::T * e] = v[e];
  }
}

// Scatter-add of window cotangents into a real-space row (adjoint of the
// gather; the cotangents are already multiplied by the conjugate de-tilt).
template <int NX>
__device__ inline void inject_row(float2 (&v)[16], int t, int y, int col, int ny,
                                  const GatherArgs& ga, const GatherRec* srec, int gb, int ge) {
  constexpr int T = RowShape<NX>::T;
  for (int q = 0; q < ge - gb; ++q) {
    const GatherRec g = q < GREC_LDS ? srec[q] : ga.rec[gb + q];
    int ry = y - g.oy;
    if (ry < 0) ry += ny;
    if (ry >= g.W) continue;
    const float2* src = ga.win + g.off + ((int64_t)col * g.W + ry) * g.W;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int x = t + T * e;
      int rx = x - g.ox;
      if (rx < 0) rx += NX;
      if (rx < g.W) v[e] = cadd(v[e], src[rx]);
    }
  }
}

// Adjoint row pass over the columns of one batch (reverse sweeps).  The state
// holds the cotangent of the parent columns, row-transformed between passes
// like the forward state.  Per column, in order: [load or start from zero]
// -> [row inverse FFT] -> [inject window cotangents] -> [slice-potential
// gradient against the checkpointed forward state after T_j] -> [x conj(T_j)]
// -> [inject] -> [row FFT, store].  A workgroup owns ROWS rows and the
// columns cg, cg + CG, ...: it sums the gradient over its columns in
// registers and writes one partial row block, reduced later in a fixed order.
// dL/dV_j(r) = 2 Re[conj(c(r)) i sigma f(r)] = 2 sigma (c_im f_re - c_re f_im)
// with c the cotangent and f the forward state after T_j.
//
// The groups fix the order of the sum over columns, and with it the number of
// waves (two a SIMD at 256^2), so the next column's state and checkpoint are
// loaded into registers before the current one is transformed: three streams
// of 235 MB a batch (slice steps of the 256^2 specimen, 447 columns) took 148
// us without it, 83 us so (8.5 TB/s: part of it stays in the last-level cache).
template <int NX, int FLAGS>
__global__ __launch_bounds__(256, 2) void k_row_adjoint(float2* __restrict__ state, int ny, int ncols,
                                                        const float2* __restrict__ T,
                                                        const float2* __restrict__ twg, int L,
                                                        GatherArgs inj, int gb, int ge, int col0,
                                                        const float2* __restrict__ ckpt,
                                                        float two_sigma, float* __restrict__ dv_partial) {
  using S = RowShape<NX>;
  constexpr bool READ = (FLAGS & ADJ_ZERO) == 0, DV = (FLAGS & ADJ_DV) != 0;
  __shared__ float2 lds[S::ROWS * S::LDS_ROW];
  __shared__ GatherRec srec[GREC_LDS];
  extern __shared__ float2 tw[];  // [L]
  if ((int)threadIdx.x < ge - gb && threadIdx.x < GREC_LDS) srec[threadIdx.x] = inj.rec[gb + threadIdx.x];
  for (int i = threadIdx.x; i < L; i += 256) tw[i] = twg[i];
  __syncthreads();
  const int t = threadIdx.x % S::T;
  const int f = threadIdx.x / S::T;
  const int y = blockIdx.x * S::ROWS + f;
  const int64_t off = (int64_t)y * NX + t, G = (int64_t)ny * NX;
  float2* my_lds = lds + f * S::LDS_ROW;
  float dv[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) dv[e] = 0.f;
  float2 v[16], fw[DV ? 16 : 1], nv[READ ? 16 : 1], nf[DV ? 16 : 1];
  auto fetch = [&](int col) {
    if constexpr (READ) {
#pragma unroll
      for (int e = 0; e < 16; ++e) nv[e] = state[col * G + off + S::T * e];
    }
    if constexpr (DV) {
#pragma unroll
      for (int e = 0; e < 16; ++e) nf[e] = ckpt[col * G + off + S::T * e];
    }
  };
  if ((int)blockIdx.y < ncols) fetch(blockIdx.y);
  for (int col = blockIdx.y; col < ncols; col += gridDim.y) {
    const int pcol = col0 + col;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      v[e] = READ ? nv[READ ? e : 0] : make_float2(0.f, 0.f);
      if constexpr (DV) fw[e] = nf[e];
    }
    if (col + (int)gridDim.y < ncols) fetch(col + gridDim.y);
    if constexpr ((FLAGS & ADJ_INV) != 0) fft::transform<NX, true, 1, true, true>(v, my_lds, t, tw, L);
    if constexpr ((FLAGS & ADJ_INJ_BEFORE) != 0)
      if (ge > gb) inject_row<NX>(v, t, y, pcol, ny, inj, srec, gb, ge);
    if constexpr (DV) {
#pragma unroll
      for (int e = 0; e < 16; ++e) dv[e] += two_sigma * (v[e].y * fw[e].x - v[e].x * fw[e].y);
    }
    if constexpr ((FLAGS & ADJ_CONJT) != 0) {
      const float2* Tj = T;
      if constexpr (NX > 256) asm volatile("" : "+s"(Tj));  // read again: no registers to keep it in
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = cmulc(v[e], Tj[off + S::T * e]);
    }
    if constexpr ((FLAGS & ADJ_INJ_AFTER) != 0)
      if (ge > gb) inject_row<NX>(v, t, y, pcol, ny, inj, srec, gb, ge);
    if constexpr ((FLAGS & ADJ_FWD) != 0) {
      fft::transform<NX, false, 1, true, true>(v, my_lds, t, tw, L);
#pragma unroll
      for (int e = 0; e < 16; ++e) state[col * G + off + S::T * e] = v[e];
    }
  }
  if constexpr (DV) {
    float* pr = dv_partial + ((int64_t)blockIdx.y * ny + y) * NX;
#pragma unroll
    for (int e = 0; e < 16; ++e) pr[t + S::T * e] = dv[e];
  }
}

// dV[i] += sum_{g < n_groups} partial[g][i], groups in order.
__global__ void k_dv_reduce(const float* __restrict__ partial, int n_groups, int64_t n, float* dv) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s = 0.f;
#pragma unroll 16  // loads in flight, the sum in order: 4.8 us for 32 groups of 256^2, 10.9 one by one
  for (int g = 0; g < n_groups; ++g) s += partial[(int64_t)g * n + i];
  dv[i] += s;
}

template <int NY>
struct ColShape {
  static constexpr int T = NY / 16;                       // threads per column transform
  // adjacent columns per block: 256 threads, and at 1024 rows 512
  static constexpr int CB = NY >= 512 ? 8 : 4096 / NY;
  static constexpr int THREADS = CB * T;
  static constexpr bool TAB16 = NY >= 512;                // second-stage twiddles in their own table
};

// Column pass.  A workgroup owns a block of CB adjacent x and the columns c, c
// + cstep, ... (a few: the launch has about kColWaves waves a CU, so that the
// dispatch still evens out the load): the next column's block is loaded into
// registers before the current one is transformed, and the block's part of
// the propagator is read once and kept.
//   Bound by the state's way in and out at 256 rows: 68.6 us for the 469 MB of
// a 447-column batch, 6.8 TB/s, where an in-place copy of random data with the
// same arithmetic beside it takes 67 to 73 us.
//   Workgroup i runs on XCD i mod 8: each XCD takes an eighth of x, so that it
// reads only its part of the propagator, and neighbouring blocks, which share
// 128-byte lines when CB < 16, meet in its L2.  For the same bytes, blocks
// dealt over the XCDs took 117 us at 512 rows (CB = 8) and 177 us at 1024 (CB =
// 16, one workgroup a CU); so 83 us and 109 us (16 and 6 slices; in the midst of 100
// slices with 20 windows a plane, 512 rows: 122 and 95 us).
constexpr int kColWaves = 60;
template <int NY>
__global__ __launch_bounds__(ColShape<NY>::THREADS, ColShape<NY>::THREADS > 256 ? 2 : 3) void k_col_pass(
    float2* __restrict__ state, int nx, int ncols, const float2* __restrict__ prop,
    const float2* __restrict__ twg, int L) {
  using S = ColShape<NY>;
  __shared__ float2 lds[S::CB * NY];
  __shared__ float2 tab[S::TAB16 ? fft::TW16 : 1];
  extern __shared__ float2 tw[];  // [L] twiddle table: the transforms' barriers order the fills
  for (int i = threadIdx.x; i < L; i += S::THREADS) tw[i] = twg[i];
  if constexpr (S::TAB16) fft::fill_tw16(tab, twg, L, threadIdx.x, S::THREADS);
  const int c = threadIdx.x % S::CB;
  const int t = threadIdx.x / S::CB;
  const int nbx = nx / S::CB, cstep = (int)gridDim.x / nbx;
  int col, xb;
  if (nbx % 8 == 0) {
    const int s = (int)(blockIdx.x >> 3), nb8 = nbx >> 3;
    col = s / nb8;
    xb = (int)(blockIdx.x & 7) * nb8 + (s - col * nb8);
  } else {
    col = (int)blockIdx.x / nbx;
    xb = (int)blockIdx.x - col * nbx;
  }
  const int off = t * nx + xb * S::CB + c, pitch = S::T * nx;
  const int64_t G = (int64_t)NY * nx;
  float2 v[16], nv[16], pr[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) pr[e] = prop[off + e * pitch];
#pragma unroll
  for (int e = 0; e < 16; ++e) nv[e] = state[col * G + off + e * pitch];
  for (; col < ncols; col += cstep) {
    const int next = col + cstep;
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = nv[e];
    if (next < ncols) {
#pragma unroll
      for (int e = 0; e < 16; ++e) nv[e] = state[next * G + off + e * pitch];
    }
    fft::transform<NY, false, S::CB, false, false, S::TAB16>(v, lds + c, t, tw, L, tab);
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = cmul(v[e], pr[e]);
    fft::transform<NY, true, S::CB, false, false, S::TAB16>(v, lds + c, t, tw, L, tab);
#pragma unroll
    for (int e = 0; e < 16; ++e) state[col * G + off + e * pitch] = v[e];
  }
}

// Whole sweeps of small grids (sides of 64 or 128): one workgroup advances one
// parent column of either side through all its slices, 16 elements of the state
// per thread, the exchanges and transposes through LDS (one padded row or column
// of the buffer per row or column of the grid), the windows cropped on the way.
//   Only T_j, P and the windows are read or written, from L2, so a slice of a column
// is bound by the instructions of its four transforms: at 128 x 128 some 1700 a
// wave, 16 waves a CU, 10 us (14 with every CU busy).  The passes keep the state in
// memory and are two launches a slice: over 10 slices, the sweeps' kernels took 231
// us for the parents of a map (every fourth beam either way) and 1600 us with every
// detector beam in passes, 98 and 1140 us here.
//   Lane pairs four rows apart would share banks where a transpose reads 128 x
// 128; swz moves every other group of four rows by four elements.
template <int NY, int NX>
struct SweepShape {
  static constexpr int THREADS = NY * NX / 16, TX = NX / 16, TY = NY / 16;
  static constexpr int PR = NX + TX, PC = NY + TY;  // LDS elements of a row, of a column
  static constexpr int BUF = NY * PR > NX * PC ? NY * PR : NX * PC;
  static constexpr int RX = NX / 16, RY = NY / 16;  // radix of the second stage
  static __device__ int swz(int y, int x) { return NY == 128 && NX == 128 ? x ^ (y & 4) : x; }
};

template <int NY, int NX>
__global__ __launch_bounds__(NY * NX / 16) void k_sweep(const SweepArgs a) {
  using S = SweepShape<NY, NX>;
  extern __shared__ float2 buf[];
  float2* tw = buf + S::BUF;  // [L]
  float2* tabx = tw + a.L;
  float2* taby = tabx + (S::RX - 1) * 16;
  for (int i = threadIdx.x; i < a.L; i += S::THREADS) tw[i] = a.tw[i];
  fft::fill_tw16(tabx, a.tw, a.L, threadIdx.x, S::THREADS, S::RX);
  fft::fill_tw16(taby, a.tw, a.L, threadIdx.x, S::THREADS, S::RY);
  __syncthreads();
  const bool s2 = (int)blockIdx.x < a.side[1].n;
  const SweepSide& sd = a.side[s2 ? 1 : 0];
  const int col = s2 ? blockIdx.x : blockIdx.x - a.side[1].n;
  const int2 hp = sd.parents[col];
  // row layout: elements (y, t + TX e); column layout: (tc + TY e, x)
  const int t = threadIdx.x % S::TX, y = threadIdx.x / S::TX;
  const int tc = threadIdx.x % S::TY, x = threadIdx.x / S::TY;
  float2* rbuf = buf + y * S::PR;
  float2* cbuf = buf + x * S::PC;
  float2 v[16];
  float2 c = make_float2(1.f, 0.f);  // the first row pass starts as in k_row_pass (ROW_START)
  if (s2) c = cscale(a.prop[(-hp.x & (NY - 1)) * NX + (-hp.y & (NX - 1))], a.scale2);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const float2 w = tw[(hp.x * y * (a.L / NY) + hp.y * (t + S::TX * e) * (a.L / NX)) & (a.L - 1)];
    v[e] = s2 ? cmul(c, w) : make_float2(w.x, -w.y);
  }
  for (int j = sd.j0;; j += s2 ? -1 : 1) {
    const bool last = j == sd.j1;
    const float2* Tj = a.T + (int64_t)j * (NY * NX) + y * NX + t;
    float2 w[16];
    if (j != sd.j0) {
      fft::transform<NY, false, 1, true, true, true>(v, cbuf, tc, tw, a.L, taby);
      int po = tc * NX + x;
      asm volatile("" : "+v"(po));  // not 16 addresses kept over the slices: no registers for them
#pragma unroll
      for (int e = 0; e < 16; ++e) w[e] = a.prop[po + S::TY * NX * e];
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = cmul(v[e], w[e]);
      fft::transform<NY, true, 1, true, true, true>(v, cbuf, tc, tw, a.L, taby);
      __syncthreads();  // every column's exchange is done
#pragma unroll
      for (int e = 0; e < 16; ++e) buf[(tc + S::TY * e) * S::PR + S::swz(tc + S::TY * e, x)] = v[e];
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = rbuf[S::swz(y, t + S::TX * e)];
      fft::exchange_sync<true>();
    }
    if (j != sd.j0) fft::transform<NX, true, 1, true, true, true>(v, rbuf, t, tw, a.L, tabx);
    const int gb = a.planes[j], ge = a.planes[j + 1];
    auto times_T = [&] {
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = cmul(v[e], Tj[S::TX * e]);
    };
    if (s2) times_T();
    if (ge > gb) gather_row<NX>(v, t, y, col, NY, sd.ga, sd.ga.rec + gb, gb, ge, hp, tw, a.L, s2 ? -1 : +1);
    if (last) break;
    if (!s2) times_T();
    fft::transform<NX, false, 1, true, true, true>(v, rbuf, t, tw, a.L, tabx);
#pragma unroll
    for (int e = 0; e < 16; ++e) rbuf[S::swz(y, t + S::TX * e)] = v[e];  // this wave's rows
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = buf[(tc + S::TY * e) * S::PR + S::swz(tc + S::TY * e, x)];
    __syncthreads();
  }
}

template <int NY, int NX>
hipError_t sweep_launch(const SweepArgs& a, hipStream_t s) {
  using S = SweepShape<NY, NX>;
  const size_t lds = (size_t)(S::BUF + a.L + 16 * (S::RX + S::RY - 2)) * sizeof(float2);
  hipError_t e = hipFuncSetAttribute((const void*)k_sweep<NY, NX>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_sweep<NY, NX>), dim3(a.side[0].n + a.side[1].n), dim3(S::THREADS), lds, s, a);
  return hipGetLastError();
}

// Columns advanced at a time by a launch of `parts` workgroups per column: as
// many as give it `slots` workgroups, the columns shared evenly over the rounds.
inline int columns_at_once(int ncols, int parts, int slots) {
  const int most = std::max(1, slots / parts);
  const int rounds = (ncols + most - 1) / most;
  return (ncols + rounds - 1) / rounds;
}

template <int NX, int FLAGS>
hipError_t row_launch(float2* state, int ncols, int ny, const float2* T, const float2* tw, int L,
                      const int2* parents, int sign, const GatherArgs& ga, int gb, int ge,
                      int col0, float2* save, const RowStart& start, const RowBoth& both, hipStream_t s) {
  using S = RowShape<NX>;
  dim3 grid(ny / S::ROWS, ncols);
  hipLaunchKernelGGL((k_row_pass<NX, FLAGS>), grid, dim3(256), L * sizeof(float2), s, state, ny, T, tw, L, parents,
                     sign, ga, gb, ge, col0, save, start, both);
  return hipGetLastError();
}

template <int NX>
hipError_t row_dispatch(int flags, float2* state, int ncols, int ny, const float2* T,
                        const float2* tw, int L, const int2* parents, int sign,
                        const GatherArgs& ga, int gb, int ge, int col0, float2* save,
                        const RowStart& start, const RowBoth& both, hipStream_t s) {
#define ROW_CASE(F) \
  case F:           \
    return row_launch<NX, F>(state, ncols, ny, T, tw, L, parents, sign, ga, gb, ge, col0, save, start, both, s);
  switch (flags) {
    ROW_CASE(ROW_BOTH | ROW_START | ROW_T | ROW_FWD)
    ROW_CASE(ROW_BOTH | ROW_INV | ROW_T | ROW_FWD)
    ROW_CASE(ROW_START | ROW_GATHER_BEFORE_T | ROW_T | ROW_FWD)
    ROW_CASE(ROW_START | ROW_GATHER_BEFORE_T)
    ROW_CASE(ROW_START | ROW_T | ROW_GATHER_AFTER_T | ROW_FWD)
    ROW_CASE(ROW_START | ROW_T | ROW_GATHER_AFTER_T)
    ROW_CASE(ROW_GATHER_BEFORE_T | ROW_T | ROW_FWD | ROW_SAVE)
    ROW_CASE(ROW_INV | ROW_GATHER_BEFORE_T | ROW_T | ROW_FWD | ROW_SAVE)
    ROW_CASE(ROW_INV | ROW_T | ROW_GATHER_AFTER_T | ROW_FWD | ROW_SAVE)
    ROW_CASE(ROW_INV | ROW_T | ROW_GATHER_AFTER_T | ROW_SAVE)
    ROW_CASE(ROW_INV | ROW_GATHER_BEFORE_T | ROW_T | ROW_FWD)
    ROW_CASE(ROW_INV | ROW_GATHER_BEFORE_T)
    ROW_CASE(ROW_GATHER_BEFORE_T)
    ROW_CASE(ROW_FWD)
    ROW_CASE(ROW_INV | ROW_T | ROW_FWD | ROW_SAVE)  // recomputing a checkpoint segment
    ROW_CASE(ROW_INV | ROW_T | ROW_GATHER_AFTER_T | ROW_FWD)
    ROW_CASE(ROW_INV | ROW_T | ROW_GATHER_AFTER_T)
    default:
      return hipErrorInvalidValue;
  }
#undef ROW_CASE
}

template <int NX, int FLAGS>
hipError_t adj_launch(float2* state, int ncols, int ny, const float2* T, const float2* tw, int L,
                      const GatherArgs& inj, int gb, int ge, int col0, const float2* ckpt,
                      float two_sigma, float* dv_partial, int groups, hipStream_t s) {
  using S = RowShape<NX>;
  hipLaunchKernelGGL((k_row_adjoint<NX, FLAGS>), dim3(ny / S::ROWS, groups), dim3(256), L * sizeof(float2), s,
                     state, ny, ncols, T, tw, L, inj, gb, ge, col0, ckpt, two_sigma, dv_partial);
  return hipGetLastError();
}

template <int NX>
hipError_t adj_dispatch(int flags, float2* state, int ncols, int ny, const float2* T,
                        const float2* tw, int L, const GatherArgs& inj, int gb, int ge, int col0,
                        const float2* ckpt, float two_sigma, float* dv_partial, int groups,
                        hipStream_t s) {
#define ADJ_CASE(F) \
  case F:           \
    return adj_launch<NX, F>(state, ncols, ny, T, tw, L, inj, gb, ge, col0, ckpt, two_sigma, dv_partial, groups, s);
  switch (flags) {
    ADJ_CASE(ADJ_ZERO | ADJ_INJ_AFTER | ADJ_FWD)                              // S1, deepest plane
    ADJ_CASE(ADJ_INV | ADJ_DV | ADJ_CONJT | ADJ_INJ_AFTER | ADJ_FWD)          // S1, slice j > 0
    ADJ_CASE(ADJ_INV | ADJ_DV)                                                // S1 slice 0, S2 last
    ADJ_CASE(ADJ_ZERO | ADJ_INJ_BEFORE | ADJ_DV | ADJ_CONJT | ADJ_FWD)         // S2, shallowest plane
    ADJ_CASE(ADJ_ZERO | ADJ_INJ_BEFORE | ADJ_DV)                              // S2, single slice
    ADJ_CASE(ADJ_INV | ADJ_INJ_BEFORE | ADJ_DV | ADJ_CONJT | ADJ_FWD)          // S2, slice j
    ADJ_CASE(ADJ_INV | ADJ_INJ_BEFORE | ADJ_DV)                               // S2, exit slice
    default:
      return hipErrorInvalidValue;
  }
#undef ADJ_CASE
}

}  // namespace

hipError_t launch_row_adjoint(int flags, float2* state, int ncols, int ny, int nx, const float2* T,
                              const float2* tw, int L, const GatherArgs& inj, int gb, int ge,
                              int col0, const float2* ckpt, float two_sigma, float* dv_partial,
                              int groups, hipStream_t s) {
  if (ncols == 0) return hipSuccess;
  if (groups < 1 || ((flags & ADJ_DV) && (!ckpt || !dv_partial))) return hipErrorInvalidValue;
  switch (nx) {
    case 64: return adj_dispatch<64>(flags, state, ncols, ny, T, tw, L, inj, gb, ge, col0, ckpt, two_sigma, dv_partial, groups, s);
    case 128: return adj_dispatch<128>(flags, state, ncols, ny, T, tw, L, inj, gb, ge, col0, ckpt, two_sigma, dv_partial, groups, s);
    case 256: return adj_dispatch<256>(flags, state, ncols, ny, T, tw, L, inj, gb, ge, col0, ckpt, two_sigma, dv_partial, groups, s);
    case 512: return adj_dispatch<512>(flags, state, ncols, ny, T, tw, L, inj, gb, ge, col0, ckpt, two_sigma, dv_partial, groups, s);
    case 1024: return adj_dispatch<1024>(flags, state, ncols, ny, T, tw, L, inj, gb, ge, col0, ckpt, two_sigma, dv_partial, groups, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_dv_reduce(const float* partial, int n_groups, int64_t n, float* dv, hipStream_t s) {
  hipLaunchKernelGGL(k_dv_reduce, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, partial,
                     n_groups, n, dv);
  return hipGetLastError();
}

hipError_t launch_row_pass(int flags, float2* state, int ncols, int ny, int nx, const float2* T,
                           const float2* tw, int L, const int2* parents, int detilt_sign,
                           const GatherArgs& ga, int gather_begin, int gather_end, int col0,
                           float2* save, const RowStart& start, hipStream_t s, const RowBoth& both) {
  if (ncols == 0) return hipSuccess;
  if ((flags & ROW_SAVE) && !save) return hipErrorInvalidValue;
  switch (nx) {
    case 64: return row_dispatch<64>(flags, state, ncols, ny, T, tw, L, parents, detilt_sign, ga, gather_begin, gather_end, col0, save, start, both, s);
    case 128: return row_dispatch<128>(flags, state, ncols, ny, T, tw, L, parents, detilt_sign, ga, gather_begin, gather_end, col0, save, start, both, s);
    case 256: return row_dispatch<256>(flags, state, ncols, ny, T, tw, L, parents, detilt_sign, ga, gather_begin, gather_end, col0, save, start, both, s);
    case 512: return row_dispatch<512>(flags, state, ncols, ny, T, tw, L, parents, detilt_sign, ga, gather_begin, gather_end, col0, save, start, both, s);
    case 1024: return row_dispatch<1024>(flags, state, ncols, ny, T, tw, L, parents, detilt_sign, ga, gather_begin, gather_end, col0, save, start, both, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_col_pass(float2* state, int ncols, int ny, int nx, const float2* prop,
                           const float2* tw, int L, int n_cu, hipStream_t s) {
  if (ncols == 0) return hipSuccess;
#define COL_CASE(N)                                                                  \
  case N: {                                                                          \
    using S = ColShape<N>;                                                           \
    if (nx % S::CB) return hipErrorInvalidValue;                                     \
    const int nbx = nx / S::CB;                                                      \
    const int at_once = columns_at_once(ncols, nbx, n_cu * kColWaves * 64 / S::THREADS); \
    hipLaunchKernelGGL(k_col_pass<N>, dim3(nbx * at_once), dim3(S::THREADS), L * sizeof(float2), s, \
                       state, nx, ncols, prop, tw, L);                               \
    return hipGetLastError();                                                        \
  }
  switch (ny) {
    COL_CASE(64)
    COL_CASE(128)
    COL_CASE(256)
    COL_CASE(512)
    COL_CASE(1024)
    default:
      return hipErrorInvalidValue;
  }
#undef COL_CASE
}

hipError_t launch_sweep(const SweepArgs& a, int ny, int nx, hipStream_t s) {
  if (a.side[0].n < 0 || a.side[1].n < 0 || a.L != std::max(ny, nx)) return hipErrorInvalidValue;
  if (a.side[0].n + a.side[1].n == 0) return hipSuccess;
  if (ny == 64 && nx == 64) return sweep_launch<64, 64>(a, s);
  if (ny == 64 && nx == 128) return sweep_launch<64, 128>(a, s);
  if (ny == 128 && nx == 64) return sweep_launch<128, 64>(a, s);
  if (ny == 128 && nx == 128) return sweep_launch<128, 128>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace bip
