// Focal back-propagation of S1 (section "Magnitude-preserving reconstruction
// and focal back-propagation"): the S1 parent columns, cropped to an enlarged
// M x M window around the atom's W x W window, are Fresnel-stepped back from
// the ionization plane to the scattering centroid of the entrance-to-ionization
// path, interpolated there, and the synthesized probe is stepped forward again
// and cropped to the atom's window.
//
// The Fresnel step of a window takes it as periodic: the window's 2-D DFT is
// multiplied by exp(s i pi lambda dist |q|^2) with q the frequencies of the
// window grid (k / (M delta) per axis, signed k), s = +1 back, -1 forward.
//
// The forward step is linear in the probe, so it commutes with the sum over
// beams: k_focal_step applies it, with the crop, between the two raster DFTs
// of the probe synthesis, and the second one then runs on the W x W window.
// The back-step of the parents runs in LDS: the window is placed at bit-reversed positions, transformed
// by a radix-2 decimation-in-time pass (natural-order spectrum), multiplied,
// and inverted by a decimation-in-frequency pass, whose bit-reversed output
// is read back at bit-reversed positions.  M is a power of two from 8 to 128.
#include "bip_internal.h"
#include "planes.h"

namespace bip {

namespace {

constexpr int NT = 256;

__device__ inline int bitrev(int v, int logm) { return (int)(__brev((unsigned)v) >> (32 - logm)); }

// One radix-2 pass over the rows (dim 0) or the columns (dim 1) of the M x M
// LDS array a: decimation in time (dit, len = 2 .. M) or in frequency (len =
// M .. 2); tw[k] = exp(-2 pi i k / M), conjugated for the inverse.
__device__ inline void fft_dim(float2* a, int M, int logm, const float2* tw, bool inverse, bool dit,
                               int dim) {
  const int nb = M * M / 2;
  for (int s = 0; s < logm; ++s) {
    const int len = dit ? (2 << s) : (M >> s), half = len >> 1;
    for (int t = threadIdx.x; t < nb; t += NT) {
      const int line = t / (M / 2), k = t - line * (M / 2);
      const int g = k / half, j = k - g * half;
      const int i0 = g * len + j, i1 = i0 + half;
      const int e0 = dim == 0 ? line * M + i0 : i0 * M + line;
      const int e1 = dim == 0 ? line * M + i1 : i1 * M + line;
      float2 w = tw[j * (M / len)];
      if (inverse) w.y = -w.y;
      const float2 u = a[e0], v = a[e1];
      if (dit) {
        const float2 vw = cmul(v, w);
        a[e0] = cadd(u, vw);
        a[e1] = csub(u, vw);
      } else {
        a[e0] = cadd(u, v);
        a[e1] = cmul(csub(u, v), w);
      }
    }
    __syncthreads();
  }
}

// exp(sign i pi lambda dist (qy^2 + qx^2)) at natural-order bin (ky, kx) of
// the M x M window grid, the phase in FP64 and reduced mod 2 pi.
__device__ inline float2 fresnel_factor(int ky, int kx, int M, double dy, double dx, double lambda,
                                        double dist, int sign) {
  const int sy = ky < M / 2 ? ky : ky - M, sx = kx < M / 2 ? kx : kx - M;
  const double qy = sy / (M * dy), qx = sx / (M * dx);
  double ph = 3.14159265358979323846 * lambda * dist * (qy * qy + qx * qx);
  ph -= 6.28318530717958647692 * floor(ph / 6.28318530717958647692);
  double s, c;
  sincos(ph, &s, &c);
  return make_float2((float)c, (float)(sign * s));
}

// The Fresnel step of the window in LDS a (natural order in, bit-reversed out).
__device__ inline void window_fresnel(float2* a, int M, int logm, const float2* tw, double dy, double dx,
                                      double lambda, double dist, int sign) {
  fft_dim(a, M, logm, tw, false, true, 0);
  fft_dim(a, M, logm, tw, false, true, 1);
  const float inv = 1.f / (float)(M * M);
  for (int e = threadIdx.x; e < M * M; e += NT) {
    const int ky = e / M, kx = e - ky * M;
    a[e] = cscale(cmul(a[e], fresnel_factor(ky, kx, M, dy, dx, lambda, dist, sign)), inv);
  }
  __syncthreads();
  fft_dim(a, M, logm, tw, true, false, 0);
  fft_dim(a, M, logm, tw, true, false, 1);
}

__device__ inline int ilog2(int m) { return 31 - __clz(m); }

// Back-step of every S1 parent window of every atom (grid: parents x atoms),
// in place in the window stack; the stored windows are de-tilted, so each is
// re-tilted by its parent's carrier first and de-tilted again after the step.
__global__ __launch_bounds__(NT) void k_focal_parents(float2* win, const FocalAtom* __restrict__ atoms,
                                                      const double* __restrict__ dist,
                                                      const int2* __restrict__ parents, int ny, int nx,
                                                      double dy, double dx, double lambda,
                                                      const float2* __restrict__ gtw, int L) {
  extern __shared__ float2 sm[];
  const FocalAtom fa = atoms[blockIdx.y];
  const int M = fa.M, logm = ilog2(M);
  float2* a = sm;
  float2* tw = sm + M * M;
  for (int k = threadIdx.x; k < M; k += NT) tw[k] = gtw[(int64_t)k * (L / M)];
  const int2 h = parents[blockIdx.x];
  float2* wp = win + fa.win_off + (int64_t)blockIdx.x * M * M;
  for (int e = threadIdx.x; e < M * M; e += NT) {
    const int ry = e / M, rx = e - ry * M;
    const int y = (fa.oy + ry) & (ny - 1), x = (fa.ox + rx) & (nx - 1);
    const float2 c = gtw[(h.x * y * (L / ny) + h.y * x * (L / nx)) & (L - 1)];  // exp(-2 pi i h.r/N)
    a[bitrev(ry, logm) * M + bitrev(rx, logm)] = cmulc(wp[e], c);               // re-tilt
  }
  __syncthreads();
  window_fresnel(a, M, logm, tw, dy, dx, lambda, dist[fa.atom], +1);
  for (int e = threadIdx.x; e < M * M; e += NT) {
    const int ry = e / M, rx = e - ry * M;
    const int y = (fa.oy + ry) & (ny - 1), x = (fa.ox + rx) & (nx - 1);
    const float2 c = gtw[(h.x * y * (L / ny) + h.y * x * (L / nx)) & (L - 1)];
    wp[e] = cmul(a[bitrev(ry, logm) * M + bitrev(rx, logm)], c);                 // de-tilt
  }
}

// Periodic kernel of the forward step along one axis, per atom (grid: atoms x
// axes, M threads): c[d] = 1/M sum_k exp(2 pi i k d / M) exp(-i pi lambda dist
// q_k^2), in FP64, rounded once; ker[atom][axis][FOCAL_M].  The M values of either
// factor are evaluated once, one a thread (a sine and cosine per term, a thread's
// M terms one after the other, made a focal map of one atom 20 us longer).
constexpr int FOCAL_M = 128;
__global__ __launch_bounds__(FOCAL_M) void k_focal_kernel(const FocalAtom* __restrict__ atoms,
                                                          const double* __restrict__ dist, double dy, double dx,
                                                          double lambda, float2* __restrict__ ker) {
  __shared__ double2 step[FOCAL_M], root[FOCAL_M];
  const FocalAtom fa = atoms[blockIdx.x];
  const int M = fa.M, d = threadIdx.x;
  const double delta = blockIdx.y == 0 ? dy : dx;
  const double pi = 3.14159265358979323846;
  if (d < M) {
    const double q = (d < M / 2 ? d : d - M) / (M * delta);
    sincos(-pi * lambda * dist[fa.atom] * q * q, &step[d].y, &step[d].x);
    sincos(2.0 * pi * d / M, &root[d].y, &root[d].x);
  }
  __syncthreads();
  if (d >= M) return;
  double re = 0.0, im = 0.0;
  for (int k = 0; k < M; ++k) {
    const double2 a = step[k], w = root[(k * d) & (M - 1)];
    re += a.x * w.x - a.y * w.y;
    im += a.x * w.y + a.y * w.x;
  }
  ker[((int64_t)fa.atom * 2 + blockIdx.y) * FOCAL_M + d] = make_float2((float)(re / M), (float)(im / M));
}

typedef float v4f __attribute__((ext_vector_type(4)));

// Complex 16 x 16 block product step on the FP32 matrix cores, K = 4: lane l
// holds row l mod 16 and K index l / 16 of a, column l mod 16 and K index
// l / 16 of b.
__device__ inline void cmfma(float2 a, float2 b, v4f& re, v4f& im) {
  re = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, re, 0, 0, 0);
  im = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.y, im, 0, 0, 0);
  re = __builtin_amdgcn_mfma_f32_16x16x4f32(-a.y, b.y, re, 0, 0, 0);
  im = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.x, im, 0, 0, 0);
}

// Forward step and crop of one row of the DFT workspace (grid: rows x atoms of
// the chunk): the M x M window X becomes Z = A_y X A_x^T, A[w][m] =
// c[(w + pad - m) mod M] (W x M), stored at the head of the row.  Two FP32
// matrix products: the step costs 8 W M (M + W) flop a row and one read of X,
// against 40 M^2 log2 M for the two transforms and their FP64 phases, which
// took 18.2 ms of the 34.8 ms of a 24-atom, 64 x 64-raster map (W = 32); this
// kernel takes 1.42 ms there (4.0 GB moved, 2.8 TB/s; 109 TFLOP/s of FP32
// products), and the second DFT, on W^2 instead of M^2 pixels, 0.65 instead of
// 2.36 ms.  A wave owns 16 columns
// of X at a time and all W rows of Y = A_y X, so X is read once, from memory
// straight into the operand registers.  NR: row blocks of 16 that the widest
// window of the launch needs.
template <int NR>
__global__ __launch_bounds__(NT, 4) void k_focal_step(const ProbeJob* __restrict__ jobs_m,
                                                   const ProbeJob* __restrict__ jobs_w,
                                                   const float2* __restrict__ ker, float2* __restrict__ fx,
                                                   int Sx) {
  extern __shared__ float2 sm[];
  const ProbeJob jm = jobs_m[blockIdx.y];
  const int v = (int)blockIdx.x % Sx;
  if ((v - jm.cv0 + Sx) % Sx >= jm.cnv) return;  // a scan column off the atom's mask: uniform per workgroup
  const int M = jm.W, W = jobs_w[blockIdx.y].W, pad = (M - W) / 2;
  const int ly = M + 1;                // LDS pitch of Y
  float2* cy = sm;                     // [M]
  float2* cx = sm + M;                 // [M]
  float2* Y = sm + 2 * M;              // [16 NR][ly]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  float2* row = fx + jm.fx_off + (int64_t)blockIdx.x * jm.ldf;
  for (int i = threadIdx.x; i < 2 * M; i += NT)
    sm[i] = ker[((int64_t)jm.atom * 2 + (i >= M)) * FOCAL_M + (i & (M - 1))];
  __syncthreads();
  constexpr int KB = 8;  // K steps (of 4 rows) loaded at a time, zero beyond M
  for (int cb = wave; cb * 16 < M; cb += NT / 64) {
    const int x = cb * 16 + li;
    v4f re[NR], im[NR];
#pragma unroll
    for (int rb = 0; rb < NR; ++rb) re[rb] = im[rb] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < M; k0 += 4 * KB) {
      float2 b[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int y = k0 + 4 * k + lk;
        b[k] = (y < M && x < M) ? row[y * M + x] : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int y = k0 + 4 * k + lk;
#pragma unroll
        for (int rb = 0; rb < NR; ++rb)
          cmfma(cy[(16 * rb + li + pad - y) & (M - 1)], b[k], re[rb], im[rb]);
      }
    }
    if (x < M) {
#pragma unroll
      for (int rb = 0; rb < NR; ++rb)
#pragma unroll
        for (int q = 0; q < 4; ++q) Y[(16 * rb + 4 * lk + q) * ly + x] = make_float2(re[rb][q], im[rb][q]);
    }
  }
  __syncthreads();  // Y complete; X read
  for (int blk = wave; blk < NR * NR; blk += NT / 64) {
    const int rb = blk / NR, vb = blk - rb * NR;
    if (16 * rb >= W || 16 * vb >= W) continue;  // wave-uniform
    v4f re = v4f{0.f, 0.f, 0.f, 0.f}, im = re;
    for (int x = lk; x < M; x += 4)
      cmfma(Y[(16 * rb + li) * ly + x], cx[(16 * vb + li + pad - x) & (M - 1)], re, im);
    const int v = 16 * vb + li;
    if (v < W) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int w = 16 * rb + 4 * lk + q;
        if (w < W) row[w * W + v] = make_float2(re[q], im[q]);
      }
    }
  }
}

// Depth of the scattering centroid of each atom's entrance-to-ionization path
// and the back-step distance (one workgroup per atom): the mean of the slice
// mid-depths (j + 1/2) dz over the slices above the ionization plane, each
// weighted by its projected potential summed over the atom's W x W window;
// distance 0 at plane 0 or with no potential on the path.  FP64 sums.
__global__ __launch_bounds__(NT) void k_focal_dist(const float* __restrict__ V, const FocalAtom* __restrict__ atoms,
                                                   int n_atoms, int ny, int nx, double dz,
                                                   double* __restrict__ dist) {
  __shared__ double red[NT];
  const FocalAtom fa = atoms[blockIdx.x];
  const int W = fa.W, pad = (fa.M - W) / 2;
  double num = 0.0, den = 0.0;
  for (int j = 0; j < fa.plane; ++j) {
    double s = 0.0;
    for (int e = threadIdx.x; e < W * W; e += NT) {
      const int ry = e / W, rx = e - ry * W;
      const int y = (fa.oy + pad + ry) & (ny - 1), x = (fa.ox + pad + rx) & (nx - 1);
      s += (double)V[((int64_t)j * ny + y) * nx + x];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = NT / 2; k > 0; k >>= 1) {
      if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
      __syncthreads();
    }
    const double m = red[0];
    __syncthreads();
    num += (j + 0.5) * dz * m;
    den += m;
  }
  if (threadIdx.x == 0)
    dist[fa.atom] = (fa.plane > 0 && den > 0.0) ? fa.plane * dz - num / den : 0.0;
}

}  // namespace

hipError_t launch_focal_dist(const float* V, const FocalAtom* atoms, int n_atoms, int ny, int nx,
                             double dz, double* dist, hipStream_t s) {
  if (n_atoms <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_focal_dist, dim3(n_atoms), dim3(NT), 0, s, V, atoms, n_atoms, ny, nx, dz, dist);
  return hipGetLastError();
}

hipError_t launch_focal_parents(float2* win, const FocalAtom* atoms, int n_atoms, const double* dist,
                                const int2* parents, int n_par, int max_m, int ny, int nx, double dy,
                                double dx, double lambda, const float2* tw, int L, hipStream_t s) {
  if (n_atoms <= 0 || n_par <= 0) return hipSuccess;
  const size_t lds = (size_t)(max_m * max_m + max_m) * sizeof(float2);
  hipError_t e = hipFuncSetAttribute((const void*)k_focal_parents,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_focal_parents, dim3(n_par, n_atoms), dim3(NT), lds, s, win, atoms, dist, parents,
                     ny, nx, dy, dx, lambda, tw, L);
  return hipGetLastError();
}

hipError_t launch_focal_kernel(const FocalAtom* atoms, int n_atoms, const double* dist, double dy, double dx,
                               double lambda, float2* ker, hipStream_t s) {
  if (n_atoms <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_focal_kernel, dim3(n_atoms, 2), dim3(FOCAL_M), 0, s, atoms, dist, dy, dx, lambda, ker);
  return hipGetLastError();
}

hipError_t launch_focal_step(const ProbeJob* jobs_m, const ProbeJob* jobs_w, const float2* ker, float2* fx, int rows,
                             int Sx, int n_jobs, int max_m, hipStream_t s) {
  if (n_jobs <= 0 || rows <= 0) return hipSuccess;
  if (max_m > FOCAL_M || n_jobs > 65535) return hipErrorInvalidValue;
  const int nr = std::max(1, max_m / 32);  // W <= M / 2
  const size_t lds = (size_t)(2 * max_m + 16 * nr * (max_m + 1)) * sizeof(float2);
  const dim3 grid((unsigned)rows, (unsigned)n_jobs);
#define FS(N)                                                                                              \
  if (nr == N) {                                                                                           \
    hipError_t e =                                                                                         \
        hipFuncSetAttribute((const void*)k_focal_step<N>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
    if (e != hipSuccess) return e;                                                                         \
    hipLaunchKernelGGL(k_focal_step<N>, grid, dim3(NT), lds, s, jobs_m, jobs_w, ker, fx, Sx);                  \
    return hipGetLastError();                                                                              \
  }
  FS(1)
  FS(2)
  FS(4)
#undef FS
  return hipErrorInvalidValue;
}

int focal_kernel_elems() { return 2 * FOCAL_M; }

}  // namespace bip
