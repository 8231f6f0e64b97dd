// Probe synthesis on the atom's window (step c, the sum over aperture beams).
//
// psi(r, rho) = sum_b c_b(rho) S1~^b(r) with the raster coefficients
// c_b(rho) = c exp(-2 pi i (h_y u / S_y + h_x v / S_x)), rho = (u, v) (eq.
// probe, illumination coefficients of eq. coupling).  The phase depends on the
// beam only through the residues (h_y mod S_y, h_x mod S_x), so the beams are
// first summed into an S_y x S_x grid of residues (the fold) and psi is the
// unnormalised forward 2-D DFT of that grid, evaluated as two 1-D DFTs.  This
// is the same sum, reordered: 8 W^2 P (S_y + S_x) flops per atom instead of
// 8 W^2 P B for the dense product with the coefficient matrix.  At an
// interpolation factor f > 1 only every f-th beam is kept and an atom only
// contributes on its crop mask: the residues are multiples of g = gcd(f, S)
// (S / g of them are summed) and only the mask's scans are evaluated.
//
// The windowed reconstruction of S1~ (eq. window-recon, eq. magpreserve) is
// fused into the fold, so S1~ never reaches memory.
//
// Pass 1, k_probe_fold_x: a workgroup owns 64 window pixels (one per lane) and
//   one residue row a.  F[c][r] = sum over beams in cell (a, c) of S1~^b(r) is
//   built in LDS, then X[a][v][r] = sum_c exp(-2 pi i c v / S_x) F[c][r] goes
//   to the workspace (complex64, r fastest).  The S_y workgroups of one pixel
//   tile run on one XCD, so the tile's parent windows are read from its L2.
// Pass 2, k_probe_y: a workgroup owns 64 window pixels and one scan column v;
//   psi[u][v][r] = c sum_a exp(-2 pi i a u / S_y) X[a][v][r] is stored as the
//   contraction operand psi^T[rho][r] (map) or as U_n = H_n psi (detector
//   contraction), in the planes of the requested precision.
// Both DFTs run on the FP32 matrix cores with twiddles rounded from FP64.
#include <type_traits>

#include "bip_internal.h"
#include "planes.h"
#include "recon_core.h"

namespace bip {

namespace {

constexpr int RT = 64;     // window pixels per workgroup (16 per wave)
constexpr int kBufferWord3 = 0x00020000;  // raw (untyped) buffer descriptor, 32-bit data
constexpr int NT = 256;    // threads per workgroup (4 wave64)

typedef float v4f __attribute__((ext_vector_type(4)));

// Four 16 x 16 output blocks of a DFT along the LDS rows, on the FP32 matrix
// cores: X[o][r] = sum_{j < S / g} T[(o g j) mod S] F[j][r] for the 64 outputs
// o = (o0 + obase + i) mod S, i < 64 (of n in all), and this wave's pixels r in
// [16 wave, 16 wave + 16).  F rows beyond S / g, up to a multiple of 4, must be zero.  A complex block is
// four real v_mfma_f32_16x16x4f32 products (the A operand is the twiddle,
// lane l holding row l mod 16 and K index l / 16; the B operand is F, lane l
// holding K index l / 16 and column l mod 16).  Output: lane l holds rows
// obase + 16 ob + 4 (l / 16) + q, column 16 wave + l mod 16, in xr / xi[ob][q].
// The same product restricted to K rows [jb, je) (je - jb a multiple of 4),
// sF holding row j at j - jb, added to xr / xi.
__device__ inline void dft_mfma_part(const float2* sF, const float2* sT, int S, int g, int o0, int n, int obase,
                                     int jb, int je, int wave, int lane, v4f (&xr)[4], v4f (&xi)[4]) {
  const int li = lane & 15, lk = lane >> 4;
  int idx[4], step[4];
#pragma unroll
  for (int ob = 0; ob < 4; ++ob) {
    const int i = obase + 16 * ob + li;
    const int o = i < n ? (o0 + i) % S : 0;
    idx[ob] = (o * g * (jb + lk)) % S;
    step[ob] = (4 * o * g) % S;
  }
  for (int j0 = jb; j0 < je; j0 += 4) {
    const float2 f = sF[(j0 - jb + lk) * RT + 16 * wave + li];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
      if (obase + 16 * ob < n) {  // wave-uniform
        const float2 e = sT[idx[ob]];
        xr[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(e.x, f.x, xr[ob], 0, 0, 0);
        xr[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(-e.y, f.y, xr[ob], 0, 0, 0);
        xi[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(e.x, f.y, xi[ob], 0, 0, 0);
        xi[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(e.y, f.x, xi[ob], 0, 0, 0);
      }
      idx[ob] += step[ob];
      if (idx[ob] >= S) idx[ob] -= S;
    }
  }
}

// The same DFT with g = 1 and every output, in half the products: with F = a + i b,
// X[o] and X[S - o] are sums and differences of C = sum cos(o j) F[j] and D = sum
// sin(o j) F[j], so only the rows o < ceil(S / 2) are multiplied, cos and sin each
// against re and im.  Row 0 of sin, zero otherwise, takes the alternating signs of
// X[S / 2] when S is even.  Blocks 2 k and 2 k + 1 of a group hold C and D of rows 32
// vi + 16 k + ..; dft_half_out hands out the outputs.  (Every map but those of plans
// with checkpoints, which keep the order of their sums, and f > 1, whose masks need
// few outputs.  Fold and DFT over y, 64 x 64 raster, 112 windows of 24 x 24: 2.57 and
// 1.68 ms with all rows, 2.21 and 1.43 so; 128 x 128, 12 windows of 24 to 64: 7.1 and
// 6.6, 5.2 and 4.2.)
__device__ inline void dft_half_part(const float2* sF, const float2* sT, int S, int vi, int jb, int je, int wave,
                                     int lane, v4f (&xr)[4], v4f (&xi)[4]) {
  const int li = lane & 15, lk = lane >> 4, R = (S + 1) / 2;
  int idx[2], step[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = 32 * vi + 16 * k + li, o = i < R ? i : 0;
    idx[k] = (o * (jb + lk)) % S;
    step[k] = (4 * o) % S;
  }
  const bool alt = vi == 0 && li == 0 && S % 2 == 0;
  const float sign = lk & 1 ? -1.f : 1.f;  // (-1)^j: jb and the steps of j are even
  for (int j0 = jb; j0 < je; j0 += 4) {
    const float2 f = sF[(j0 - jb + lk) * RT + 16 * wave + li];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (32 * vi + 16 * k < R) {  // wave-uniform
        const float2 e = sT[idx[k]];
        const float sn = k == 0 && alt ? sign : -e.y;
        xr[2 * k] = __builtin_amdgcn_mfma_f32_16x16x4f32(e.x, f.x, xr[2 * k], 0, 0, 0);
        xi[2 * k] = __builtin_amdgcn_mfma_f32_16x16x4f32(e.x, f.y, xi[2 * k], 0, 0, 0);
        xr[2 * k + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(sn, f.x, xr[2 * k + 1], 0, 0, 0);
        xi[2 * k + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(sn, f.y, xi[2 * k + 1], 0, 0, 0);
      }
      idx[k] += step[k];
      if (idx[k] >= S) idx[k] -= S;
    }
  }
}
template <typename Out>
__device__ inline void dft_half_out(int S, int vi, int lane, const v4f (&xr)[4], const v4f (&xi)[4], Out out) {
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 32 * vi + 16 * k + 4 * (lane >> 4) + q;
      const float cr = xr[2 * k][q], ci = xi[2 * k][q], dr = xr[2 * k + 1][q], di = xi[2 * k + 1][q];
      if (i >= (S + 1) / 2) continue;
      if (i == 0) {
        out(0, cr, ci);
        if (S % 2 == 0) out(S / 2, dr, di);
      } else {
        out(i, cr + di, ci - dr);
        out(S - i, cr - di, ci + dr);
      }
    }
}

__device__ inline void dft_mfma(const float2* sF, const float2* sT, int S, int obase, int wave,
                                int lane, v4f (&xr)[4], v4f (&xi)[4]) {
#pragma unroll
  for (int ob = 0; ob < 4; ++ob) {
    xr[ob] = v4f{0.f, 0.f, 0.f, 0.f};
    xi[ob] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  dft_mfma_part(sF, sT, S, 1, 0, S, obase, 0, (S + 3) & ~3, wave, lane, xr, xi);
}

constexpr int FOLD_CH = 64;  // residue cells of the fold held in LDS at a time

// The table rows of a beam of the fold (wave-uniform).
struct FoldBeam {
  int2 h;
  int ec[ELL_W];
  float ew[ELL_K];
};
__device__ inline void fold_beam(FoldBeam& q, const ProbeArgs& pa, int b) {
  q.h = pa.beams[b];
#pragma unroll
  for (int j = 0; j < ELL_W; ++j) q.ec[j] = pa.ellc[(int64_t)b * ELL_W + j];
#pragma unroll
  for (int j = 0; j < ELL_K; ++j) q.ew[j] = pa.ellw[(int64_t)b * ELL_W + j];
}

// 1-D grid.  Workgroups are dispatched to the 8 XCDs in turn, so blocks x,
// x + 8, x + 16, ... share XCD x: its slot s takes residue row s mod n_y of
// pixel tile unit0 + 8 (s / n_y) + x, and the n_y rows of a tile run together
// in one L2.  A tile is 64 pixels of one job (the job with the last t0 <= the
// tile).  The dispatch order only affects speed.
// The residue cells are folded FOLD_CH at a time into LDS, and each chunk's
// share of the DFT over x is added to the NV = ceil(columns / 64) output blocks
// held in registers (the products run in the same K order as one pass).
// A wave's beam needs its table rows before its parent values, and these before
// the sum: with each loaded when needed, three trips to L2 a beam, a map of 112
// windows of 24 x 24 with 8.1k beams and a 64 x 64 raster took 3.3 ms, 12 windows
// of 24 to 64 with a 128 x 128 raster 8.0, 24 of 64 x 64 with hex parents 4.9;
// with both loaded ahead 2.6, 7.2 and 4.1, and 2.2, 5.2 and 3.3 with the DFT by
// halves (whose matrix products alone are 0.45, and the 50 vector instructions a
// beam and 64 pixels 0.7, of the first).
// Residue row i of the workspace is row i g_y of the grid.  (256 x 256, 112
// atoms, 64 x 64 scans, f = 4: the fold takes 0.21 ms and the DFT over y 0.09,
// against 2.48 and 1.67 with every residue and every scan, of which 15 of 16 are
// zero or outside the masks.)
template <int NV, bool HALF>
__global__ __launch_bounds__(NT, NV <= 2 ? 4 : NV == 3 ? 3 : 2) void k_probe_fold_x(const ProbeArgs pa) {
  extern __shared__ float2 sm[];
  const int Sx = pa.Sx, nc = Sx / pa.gx, nr = pa.Sy / pa.gy;  // residue columns and rows in use
  const int CH = min((nc + 3) & ~3, FOLD_CH);
  float2* sF = sm;           // [CH][RT]
  float2* sT = sm + CH * RT; // [Sx]
  float2* sW = sT + Sx;      // [L] exp(-2 pi i m / L), gathered per lane
  const int slot = blockIdx.x >> 3;
  const int k8 = slot / nr;
  const int ai = slot - k8 * nr, a = ai * pa.gy;
  const int u = pa.unit0 + 8 * k8 + (blockIdx.x & 7);
  if (u >= pa.unit0 + pa.n_units) return;  // the grid's last row of 8 tiles
  int lo = 0, hi = pa.n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pa.jobs[mid].t0 <= u) lo = mid;
    else hi = mid - 1;
  }
  const ProbeJob job = pa.jobs[lo];
  const int W = job.W, W2 = W * W;
  const int r0 = (u - job.t0) * RT;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = threadIdx.x; i < Sx; i += NT) sT[i] = pa.twx[i];
  for (int i = threadIdx.x; i < pa.L; i += NT) sW[i] = pa.tw[i];
  __syncthreads();
  const int r = r0 + lane;
  const bool live = r < W2;
  const int rr = live ? r : 0;
  const int ry = rr / W, rx = rr - ry * W;
  const int py = ((job.oy + ry) & (pa.ny - 1)) * (pa.L / pa.ny);
  const int px = ((job.ox + rx) & (pa.nx - 1)) * (pa.L / pa.nx);
  const float2* win = pa.win + job.win_off;
  // The parent values are read through a buffer descriptor of the atom's
  // window stack: the parent's offset in a scalar register, the pixel's in a
  // vector one, so a load needs no per-lane address arithmetic.  A stack
  // block beyond the descriptor's 32-bit offsets (2 GiB) is read through
  // 64-bit pointers instead (a choice uniform over the workgroup).
  const bool rsrc_ok = (int64_t)pa.n_par * W2 * (int64_t)sizeof(float2) <= 0x7fffffff;
  const __amdgpu_buffer_rsrc_t rwin = __builtin_amdgcn_make_buffer_rsrc(
      (void*)win, (short)0, rsrc_ok ? pa.n_par * W2 * (int)sizeof(float2) : 0, kBufferWord3);
  const int voff = rr * (int)sizeof(float2);
  v4f xr[NV][4], xi[NV][4];
#pragma unroll
  for (int vi = 0; vi < NV; ++vi)
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
      xr[vi][ob] = v4f{0.f, 0.f, 0.f, 0.f};
      xi[vi][ob] = v4f{0.f, 0.f, 0.f, 0.f};
    }
  for (int cc = 0; cc < nc; cc += CH) {
    const int ce = min(nc, cc + CH);
    const int cp = cc + ((ce - cc + 3) & ~3);  // the chunk's K rows, zero beyond ce
    // The chunk's beams are consecutive in cell_beams (cells between two
    // multiples of g_x hold none).  Lane i keeps the end of cell cc + i; each
    // wave takes the cells that end within its quarter of the beams.
    const int nce = ce - cc, cell0 = a * Sx + cc * pa.gx;
    const int ends = lane < nce ? pa.cell_start[cell0 + lane * pa.gx + 1] : INT32_MAX;
    const int kb = pa.cell_start[cell0], nk = __builtin_amdgcn_readlane(ends, nce - 1) - kb;
    auto cells_to = [&](int w) { return w >= 4 ? nce : w <= 0 ? 0 : (int)__popcll(__ballot(ends <= kb + nk * w / 4)); };
    auto end_of = [&](int c) { return c < 0 ? kb : __builtin_amdgcn_readlane(ends, c); };
    int c = cells_to(wave);
    const int c1 = cells_to(wave + 1);
    int k = end_of(c - 1);
    const int kl = end_of(c1 - 1);
    float2 F = make_float2(0.f, 0.f);
    auto store = [&] {  // cell c is complete
      sF[c * RT + lane] = live ? F : make_float2(0.f, 0.f);
      F = make_float2(0.f, 0.f);
      ++c;
    };
    // The table rows are loaded two beams ahead of their use and the parent
    // values one ahead (past the last beam, the last one's again), into D0 and
    // D1 in turn.
    auto beams = [&](auto buffered) {
      if (k >= kl) return;
      auto fetch = [&](const FoldBeam& q, float2 (&D)[ELL_K]) {
        if constexpr (decltype(buffered)::value) {
#pragma unroll
          for (int j = 0; j < ELL_K; ++j)
            D[j] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(
                                                  rwin, voff, q.ec[j] * W2 * (int)sizeof(float2), 0));
        } else {
          recon_load(win, W2, rr, q.ec, D);
        }
      };
      FoldBeam n1, n2;
      float2 D0[ELL_K], D1[ELL_K];
      fold_beam(n1, pa, pa.cell_beams[k]);
      fold_beam(n2, pa, pa.cell_beams[min(k + 1, kl - 1)]);
      int b3 = pa.cell_beams[min(k + 2, kl - 1)];  // the beam after n2
      fetch(n1, D0);
      auto step = [&](const float2 (&D)[ELL_K], float2 (&nD)[ELL_K]) {
        while (k == end_of(c)) store();
        const FoldBeam q = n1;
        n1 = n2;
        fetch(n1, nD);
        fold_beam(n2, pa, b3);
        b3 = pa.cell_beams[min(k + 3, kl - 1)];
        const float2 t = sW[(q.h.x * py + q.h.y * px) & (pa.L - 1)];  // exp(-2 pi i h.r/N)
        const float2 sv = recon_finish(D, win, W2, rr, q.ec, q.ew, pa.col, pa.w, pa.mode);
        F = cadd(F, cmulc(sv, t));  // re-tilt by exp(+2 pi i h.r/N)
        ++k;
      };
      while (k + 1 < kl) {
        step(D0, D1);
        step(D1, D0);
      }
      if (k < kl) step(D0, D1);
    };
    if (rsrc_ok) beams(std::true_type{});
    else beams(std::false_type{});
    while (c < c1) store();
    for (int c = ce + wave; c < cp; c += 4) sF[(c - cc) * RT + lane] = make_float2(0.f, 0.f);
    __syncthreads();
#pragma unroll
    for (int vi = 0; vi < NV; ++vi) {
      if constexpr (HALF) dft_half_part(sF, sT, Sx, vi, cc, cp, wave, lane, xr[vi], xi[vi]);
      else dft_mfma_part(sF, sT, Sx, pa.gx, job.cv0, job.cnv, 64 * vi, cc, cp, wave, lane, xr[vi], xi[vi]);
    }
    __syncthreads();  // the chunk is consumed before the next one is folded
  }
  const int li = lane & 15, lk = lane >> 4;
  float2* X = pa.fx + job.fx_off + (int64_t)ai * Sx * job.ldf + r0 + 16 * wave + li;
  if constexpr (HALF) {
#pragma unroll
    for (int vi = 0; vi < NV; ++vi)
      dft_half_out(Sx, vi, lane, xr[vi], xi[vi],
                   [&](int v, float re, float im) { X[(int64_t)v * job.ldf] = make_float2(re, im); });
    return;
  }
#pragma unroll
  for (int vi = 0; vi < NV; ++vi)
#pragma unroll
    for (int ob = 0; ob < 4; ++ob)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int iv = 64 * vi + 16 * ob + 4 * lk + q;
        if (iv < job.cnv) X[(int64_t)((job.cv0 + iv) % Sx) * job.ldf] = make_float2(xr[vi][ob][q], xi[vi][ob][q]);
      }
}

// The residue rows are staged FOLD_CH at a time, each chunk's share of the DFT
// over y added to the NV = ceil(rows / 64) output blocks in registers.  The map
// operand's rows are the scans of the atom's mask, (i_u, i_v) row by row (all
// scans at f = 1); U_n's are all scans, those off the mask not written (the
// products mask them).
// The channels of U_n are dealt over zc workgroups, each with a DFT of its own, while
// that leaves two workgroups a CU: 17 of them that wrote 34 channels of 65 x 17 scans of
// an 8 x 8 window one after the other took 194 us (FP16; 43 at the probe's own kernel of
// focal maps, one workgroup a scan, which this one replaced), 39 us in 30 groups.  With
// four a CU the DFT repeated for 768 workgroups of 3 channels cost more than it gave (170
// and 240 us).
template <int PREC, bool U, int NV, bool HALF>
__global__ __launch_bounds__(NT) void k_probe_y(const ProbeArgs pa) {
  extern __shared__ float2 sm[];
  const int Sy = pa.Sy, Sx = pa.Sx, nr = Sy / pa.gy;
  const int CH = min((nr + 3) & ~3, FOLD_CH);
  float2* sG = sm;            // [CH][RT]
  float2* sT = sm + CH * RT;  // [Sy]
  const int zc = U ? pa.zc : 1, cg = U ? (int)blockIdx.z % zc : 0;  // channel group
  const ProbeJob job = pa.jobs[blockIdx.z / zc];
  const int W2 = job.W * job.W;
  const int kd = job.kd;
  const int r0 = blockIdx.x * RT;
  const int iv = blockIdx.y;
  if (r0 >= kd || iv >= job.cnv) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int v = (job.cv0 + iv) % Sx;
  for (int i = threadIdx.x; i < Sy; i += NT) sT[i] = pa.twy[i];
  const int r = r0 + lane;
  const bool live = r < W2;
  const float2* X = pa.fx + job.fx_off + (int64_t)v * job.ldf + r;
  v4f xr[NV][4], xi[NV][4];
#pragma unroll
  for (int vi = 0; vi < NV; ++vi)
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
      xr[vi][ob] = v4f{0.f, 0.f, 0.f, 0.f};
      xi[vi][ob] = v4f{0.f, 0.f, 0.f, 0.f};
    }
  for (int ac = 0; ac < nr; ac += CH) {
    const int ap = ac + ((min(nr, ac + CH) - ac + 3) & ~3);  // the chunk's K rows, zero beyond the last
    // this wave's rows of the chunk: all loads in flight before the LDS stores
    float2 xg[FOLD_CH / 4];
#pragma unroll
    for (int q = 0; q < FOLD_CH / 4; ++q) {
      const int a = ac + wave + 4 * q;
      xg[q] = (a < ap && live && a < nr) ? X[(int64_t)a * Sx * job.ldf] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int q = 0; q < FOLD_CH / 4; ++q) {
      const int a = ac + wave + 4 * q;
      if (a < ap) sG[(a - ac) * RT + lane] = xg[q];
    }
    __syncthreads();
#pragma unroll
    for (int vi = 0; vi < NV; ++vi) {
      if constexpr (HALF) dft_half_part(sG, sT, Sy, vi, ac, ap, wave, lane, xr[vi], xi[vi]);
      else dft_mfma_part(sG, sT, Sy, pa.gy, job.cu0, job.cnu, 64 * vi, ac, ap, wave, lane, xr[vi], xi[vi]);
    }
    __syncthreads();  // the chunk is consumed before the next one is staged
  }
  // this lane's output pixel
  const int li = lane & 15, lk = lane >> 4;
  const int ro = r0 + 16 * wave + li;
  const bool in = ro < kd, live_o = ro < W2;
  auto put = [&](int rho, float re, float im) {
    if constexpr (U) {
      for (int n = pa.n_ch * cg / zc; n < pa.n_ch * (cg + 1) / zc; ++n) {
        const float2 hn = live_o ? pa.H[job.h_off + (int64_t)n * W2 + ro] : make_float2(0.f, 0.f);
        store_planes<PREC>(pa.out, job.out_off + ((int64_t)n * pa.Ppad + rho) * kd + ro,
                           pa.out_plane, hn.x * re - hn.y * im, hn.x * im + hn.y * re);
      }
    } else {
      store_planes<PREC>(pa.out, job.out_off + (int64_t)rho * kd + ro, pa.out_plane, re, im);
    }
  };
  if constexpr (HALF) {
    if (in) {
#pragma unroll
      for (int vi = 0; vi < NV; ++vi)
        dft_half_out(Sy, vi, lane, xr[vi], xi[vi],
                     [&](int u, float re, float im) { put(u * Sx + v, pa.cb * re, pa.cb * im); });
    }
  } else if (in) {
#pragma unroll
    for (int vi = 0; vi < NV; ++vi)
#pragma unroll
      for (int ob = 0; ob < 4; ++ob)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int iu = 64 * vi + 16 * ob + 4 * lk + q;
          if (iu < job.cnu) put(U ? (job.cu0 + iu) % Sy * Sx + v : iu * job.cnv + iv, pa.cb * xr[vi][ob][q], pa.cb * xi[vi][ob][q]);
        }
  }
  // at f = 1 rows P .. Ppad-1 of the operand are zero (otherwise unused)
  if (blockIdx.y == 0 && in && job.cnu * job.cnv == pa.P)
    for (int rho = pa.P + lk; rho < pa.Ppad; rho += 4) put(rho, 0.f, 0.f);
}

// One DFT pass of the probe-sum adjoint: for every outer index o and window
// pixel r < W2 of an atom (grid z),
//   out[k][o][r] = sum_j T[(j k) mod S] in[j][o][r],
// with T = exp(+2 pi i k/S) (the conjugate of the synthesis twiddles).  Along
// x (j = v, o = u) the rows of g_psi [u][v][kd] become X [u][k][ldf]; along y
// (j = u, o = k_x) X becomes Z [k][k_x][ldf].
__global__ __launch_bounds__(NT) void k_dft_adjoint(int along_y, const AdjAtom* __restrict__ atoms,
                                                    const float2* __restrict__ in_all, int64_t in_stride,
                                                    float2* out_all, int64_t out_stride, int Sy, int Sx,
                                                    const float2* __restrict__ tws) {
  extern __shared__ float2 sm[];
  const AdjAtom at = atoms[blockIdx.z];
  const int W2 = at.W * at.W, r0 = blockIdx.x * RT;
  if (r0 >= W2) return;
  const int S = along_y ? Sy : Sx;
  const int64_t kd = (W2 + 31) & ~31, ldf = (W2 + 63) & ~63;
  const float2* in = in_all + (int64_t)at.slot * in_stride;
  float2* out = out_all + (int64_t)(along_y ? at.sub : at.slot) * out_stride;
  const int64_t js = along_y ? Sx * ldf : kd, os = along_y ? ldf : Sx * kd;
  const int64_t ks = along_y ? Sx * ldf : ldf, os2 = along_y ? ldf : Sx * ldf;
  float2* sF = sm;
  float2* sT = sm + ((S + 3) & ~3) * RT;
  const int o = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = threadIdx.x; i < S; i += NT) sT[i] = tws[i];
  const int r = r0 + lane;
  // this wave's rows, 16 loads in flight before their LDS stores
  const int Sc = (S + 3) & ~3;
  for (int j0 = wave; j0 < Sc; j0 += 64) {
    float2 v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int j = j0 + 4 * q;
      v[q] = (r < W2 && j < S) ? in[(int64_t)j * js + (int64_t)o * os + r] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int j = j0 + 4 * q;
      if (j < Sc) sF[j * RT + lane] = v[q];
    }
  }
  __syncthreads();
  const int li = lane & 15, lk = lane >> 4;
  const int ro = r0 + 16 * wave + li;
  for (int k0 = 0; k0 < S; k0 += 64) {
    v4f xr[4], xi[4];
    dft_mfma(sF, sT, S, k0, wave, lane, xr, xi);
    if (ro < W2) {
#pragma unroll
      for (int ob = 0; ob < 4; ++ob)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int k = k0 + 16 * ob + 4 * lk + q;
          if (k < S) out[(int64_t)k * ks + (int64_t)o * os2 + ro] = make_float2(xr[ob][q], xi[ob][q]);
        }
    }
  }
}

template <typename K>
hipError_t launch_lds(K kernel, dim3 grid, size_t lds, const ProbeArgs& pa, hipStream_t s) {
  hipError_t e = hipFuncSetAttribute((const void*)kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, grid, dim3(NT), lds, s, pa);
  return hipGetLastError();
}

}  // namespace

size_t probe_lds_bytes(int S) { return (size_t)(((S + 3) & ~3) * RT + S) * sizeof(float2); }

hipError_t launch_dft_adjoint(bool along_y, const AdjAtom* atoms, int n, int max_w2, const float2* in, int64_t in_stride,
                              float2* out, int64_t out_stride, int Sy, int Sx, const float2* tws, hipStream_t s) {
  if (n <= 0 || max_w2 <= 0) return hipSuccess;
  const size_t lds = probe_lds_bytes(along_y ? Sy : Sx);
  hipError_t e = hipFuncSetAttribute((const void*)k_dft_adjoint,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_dft_adjoint, dim3((max_w2 + RT - 1) / RT, along_y ? Sx : Sy, n), dim3(NT), lds, s, along_y ? 1 : 0,
                     atoms, in, in_stride, out, out_stride, Sy, Sx, tws);
  return hipGetLastError();
}

hipError_t launch_probe_fold_x(const ProbeArgs& pa, int unit0, int n_units, int n_jobs, int max_cnv, hipStream_t s) {
  if (n_jobs <= 0 || n_units <= 0 || max_cnv <= 0) return hipSuccess;
  if (unit0 < 0 || pa.Sy < 1 || pa.gy < 1 || pa.gx < 1 || pa.Sy % pa.gy || pa.Sx % pa.gx) return hipErrorInvalidValue;
  const int64_t blocks = (int64_t)((n_units + 7) / 8) * 8 * (pa.Sy / pa.gy);
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  ProbeArgs q = pa;
  q.unit0 = unit0;
  q.n_units = n_units;
  q.n_jobs = n_jobs;
  const size_t lds = ((size_t)std::min((pa.Sx / pa.gx + 3) & ~3, FOLD_CH) * RT + pa.Sx + pa.L) * sizeof(float2);
  if (pa.half && (pa.gx != 1 || pa.gy != 1 || max_cnv != pa.Sx)) return hipErrorInvalidValue;
  const int nv = (max_cnv + 63) / 64;
#define PF(NV)                                                                                     \
  if (nv == NV)                                                                                    \
    return pa.half ? launch_lds(k_probe_fold_x<NV, true>, dim3((unsigned)blocks), lds, q, s)       \
                   : launch_lds(k_probe_fold_x<NV, false>, dim3((unsigned)blocks), lds, q, s);
  PF(1) PF(2) PF(3) PF(4)
#undef PF
  return hipErrorInvalidValue;
}

hipError_t launch_probe_y(const ProbeArgs& pa, int prec, bool u, int max_kd, int max_cnu, int max_cnv, int n_jobs,
                          hipStream_t s) {
  if (n_jobs <= 0 || max_cnu <= 0 || max_cnv <= 0) return hipSuccess;
  ProbeArgs q = pa;
  q.zc = 1;
  if (u) {  // up to two workgroups a CU
    const int64_t wgs = (int64_t)((max_kd + RT - 1) / RT) * max_cnv * n_jobs;
    q.zc = (int)std::max<int64_t>(1, std::min<int64_t>(pa.n_ch, 2 * pa.n_cu / wgs));
  }
  const dim3 grid((unsigned)((max_kd + RT - 1) / RT), (unsigned)max_cnv, (unsigned)(n_jobs * q.zc));
  const size_t lds = ((size_t)std::min((pa.Sy / pa.gy + 3) & ~3, FOLD_CH) * RT + pa.Sy) * sizeof(float2);
  const int nv = (max_cnu + 63) / 64;
  if (pa.half && (pa.gx != 1 || pa.gy != 1 || max_cnu != pa.Sy || max_cnv != pa.Sx)) return hipErrorInvalidValue;
#define PYV(P, UU, NV)                                                          \
  if (nv == NV)                                                                 \
    return pa.half ? launch_lds(k_probe_y<P, UU, NV, true>, grid, lds, q, s)    \
                   : launch_lds(k_probe_y<P, UU, NV, false>, grid, lds, q, s);
#define PY(P)                                                                                  \
  if (prec == P) {                                                                             \
    if (u) {                                                                                   \
      PYV(P, true, 1) PYV(P, true, 2) PYV(P, true, 3) PYV(P, true, 4)                          \
    } else {                                                                                   \
      PYV(P, false, 1) PYV(P, false, 2) PYV(P, false, 3) PYV(P, false, 4)                      \
    }                                                                                          \
    return hipErrorInvalidValue;                                                               \
  }
  PY(BIP_PREC_FP32)
  PY(BIP_PREC_SPLIT_BF16)
  PY(BIP_PREC_BF16)
  PY(BIP_PREC_FP16)
#undef PY
#undef PYV
  return hipErrorInvalidValue;
}

}  // namespace bip
