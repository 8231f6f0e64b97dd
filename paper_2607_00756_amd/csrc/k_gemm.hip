// Complex contractions on the matrix cores (step c).
//
// Every contraction is an "NT" complex product C[m][n] = sum_k A[m][k] B[n][k]
// (optionally with conj(A)), K running along the rows of both operands, each
// operand stored as separate real planes:
//   FP32        : re, im                          (v_mfma_f32_16x16x4_f32)
//   SPLIT_BF16  : re_hi, re_lo, im_hi, im_lo       (v_mfma_f32_16x16x32_bf16;
//                 hi*hi + hi*lo + lo*hi per real product, FP32 accumulate)
//   BF16        : re, im                          (v_mfma_f32_16x16x32_bf16)
//   FP16        : re, im                          (v_mfma_f32_16x16x32_f16)
// A complex product is four real products; the minus sign of re*re - im*im is
// applied by flipping the sign bit of the A imaginary fragment.
//
// Tiling (Cfg): a workgroup of 4 or 8 wave64s owns a 128 x 128 output tile
// (64 x 64 for FP32 operands).  K advances in 64-byte chunks per plane row (16
// FP32 or 32 BF16 values); consecutive chunks of a row are either adjacent (K
// contiguous) or a fixed stride apart (K-blocked operands, where every 64-byte
// column block of the matrix is stored contiguously).  Operand chunks move
// from global memory straight into LDS with global_load_lds_dwordx4 (no VGPR
// staging), buffered NS deep, one barrier per chunk; the 16-byte slots of each
// LDS row are XOR-permuted (swz) so that the 16 rows read by one MFMA fragment
// load hit distinct banks.
//
// Roles (epilogues):
//   EPI_ABS2_MAP / EPI_ABS2_BEAMS
//              a_d(rho) = sum_r S2~^d(r) U_n(r, rho), U_n = H_n psi from the
//              probe synthesis; |a|^2 accumulated over
//              the (atom, channel) jobs in registers, then summed over d (map)
//              or added into [rho][d] (beams)
//   EPI_GRAMQ  G[r][r'] = sum_d conj(S2~^d(r)) S2~^d(r') and its product with
//              sum_n conj(H_n(r)) H_n(r') -> Q (operand of EPI_QUAD)
//   EPI_QUAD   (Q psi)(r, rho); I(rho) += Re sum_r conj(psi(r, rho)) (Q psi)(r, rho)
//              accumulated over atoms, then summed over the tile's r
//   EPI_STORE  the product itself as complex64 (optionally scaled per row):
//              the contractions of the map-loss gradient
// For the map, sum_n sum_d |a_d|^2 = psi^H Q psi exactly, which replaces the
// n_det x N_ch P detector contraction by a W^2 x W^2 Gram matrix per atom.
#include "bip_internal.h"
#include "planes.h"

#include <type_traits>

namespace bip {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

template <int PREC>
struct PT;
template <>
struct PT<BIP_PREC_FP32> {
  static constexpr int PLANES = 2, ESZ = 4, BK = 16;
};
template <>
struct PT<BIP_PREC_SPLIT_BF16> {
  static constexpr int PLANES = 4, ESZ = 2, BK = 32;
};
template <>
struct PT<BIP_PREC_BF16> {
  static constexpr int PLANES = 2, ESZ = 2, BK = 32;
};
template <>
struct PT<BIP_PREC_FP16> {
  static constexpr int PLANES = 2, ESZ = 2, BK = 32;
};

// Cost model of the Gram's K split, in chunk times (about 2 us): filling and
// epilogue of a unit, and the 256 KB that a partial 128 x 128 tile moves.
constexpr double GRAM_FILL = 6.0, GRAM_PART = 0.03;

// Tile of a workgroup: WM x WN waves, each NBM x NBN blocks of 16 x 16; NS
// chunk buffers; WPE waves per SIMD the kernel is built for.
//   FP32 products run at 1/16 of the 16-bit rate, so a 64 x 64 tile still
//   needs only about a third of the LDS and L2 rate it has, and small tiles
//   waste less of a window's edge and of the last round of workgroups: three
//   workgroups a CU, three stages each.  (28 atoms of 20 x 20 and 28 x 28
//   pixels, 32,417 beams: Gram 36.4 -> 14.4 ms with the equal shares of the
//   XCDs, 98 TFLOP/s of the 154 that a large FP32 product reaches.)
//   Split planes (12 products per block pair) take 8 waves, two per SIMD, so
//   that one wave's fragment reads and waits run under the other's products.
//   The rate of all 16-bit roles is near what a large library product reaches
//   (1.24 PFLOP/s): per-beam products at W = 64, 64,713 beams x 2304 scans,
//   168 -> 115 ms (1.28 PFLOP/s of hardware products); at W = 24, 16,207 beams
//   x 960 scans x 72 channels, 26.8 -> 12.5 ms (with the tile order below).
//   The Gram and store products of two-plane operands run two workgroups of 4
//   waves per CU for the same reason, and their per-beam products 8 waves: with
//   4, one a SIMD, the job stream's addresses had the accumulators copied through
//   AGPRs in every chunk (BF16, 9 tiles of 648 chunks, no job groups: 0.57 ms
//   before the stream, 0.89 with it, 0.57 so; 32,417 beams x 2304 scans, 6 windows
//   of 32 x 32 x 3 channels: 14.4, 14.9 and 10.8 ms).  Their quadratic form keeps
//   one of 4, with four stages and the larger register set of its running sums.
// The quadratic form's waves are always 64 columns (r) wide and its tiles
// 128: the order of its sum over r is the same in every configuration.
template <int PREC, int EPI>
struct Cfg {
  static constexpr bool TWO = EPI == EPI_GRAMQ || EPI == EPI_STORE, BEAM = EPI == EPI_ABS2_MAP || EPI == EPI_ABS2_BEAMS;
  static constexpr int WM = 2, WN = BEAM ? 4 : 2, NBM = 4, NBN = BEAM ? 2 : 4, NS = TWO ? 2 : 4, WPE = TWO || BEAM ? 2 : 1;
};
template <int EPI>
struct Cfg<BIP_PREC_FP32, EPI> {
  static constexpr int WM = 2, WN = 2, NBM = 2, NBN = 2, NS = 3, WPE = 3;
};
// The Gram matrix of a plan that keeps its order of summation, where 64 x 64
// tiles are fewer than the CUs: a tile's K loop cannot be split, so it is cut
// smaller, one block a wave (4 atoms of 20 x 20 pixels, 2053 beams: 124 tiles
// 196 us, 436 of 32 x 32 111 us).
template <>
struct Cfg<BIP_PREC_FP32, EPI_GRAMQ_SMALL> {
  static constexpr int WM = 2, WN = 2, NBM = 1, NBN = 1, NS = 4, WPE = 4;
};
template <>
struct Cfg<BIP_PREC_FP32, EPI_QUAD> {
  static constexpr int WM = 2, WN = 2, NBM = 2, NBN = 4, NS = 3, WPE = 2;
};
template <int EPI>
struct Cfg<BIP_PREC_SPLIT_BF16, EPI> {
  static constexpr int WM = 2, WN = 4, NBM = 4, NBN = 2, NS = 2, WPE = 2;
};
template <>
struct Cfg<BIP_PREC_SPLIT_BF16, EPI_QUAD> {
  static constexpr int WM = 4, WN = 2, NBM = 2, NBN = 4, NS = 2, WPE = 2;
};
template <int PREC, int EPI>
struct Tile : Cfg<PREC, EPI> {
  using C = Cfg<PREC, EPI>;
  static constexpr int NW = C::WM * C::WN, NT = 64 * NW;    // waves, threads
  static constexpr int BM = 16 * C::WM * C::NBM, BN = 16 * C::WN * C::NBN;
  static constexpr int PLA = BM * 64, PLB = BN * 64;        // bytes of one plane of an operand's chunk
  static constexpr int OPA = PT<PREC>::PLANES * PLA;        // A's chunk
  static constexpr int SB = OPA + PT<PREC>::PLANES * PLB;   // one stage
  static constexpr int RA = BM / 16 / NW, RB = BN / 16 / NW;  // 16-row blocks loaded per wave and plane
  static constexpr int UNITS = PT<PREC>::PLANES * (BM + BN) / 16;  // 1 KB pieces of a chunk
  static constexpr int LPC = UNITS / NW;                           // loads per wave and chunk
  static constexpr int LDS = C::NS * SB;
  // accumulator quads per thread (re and im): the layout of a partial tile
  static constexpr int QUADS = 2 * C::NBM * C::NBN;
  static constexpr bool ROWS = RA * 16 * NW == BM && RB * 16 * NW == BN;  // every wave loads rows of each plane
  static_assert(UNITS % NW == 0, "whole pieces per wave");
};

// The FP32 Gram matrix sums its K products (all detector beams) in segments
// of KSEG: each segment in its own accumulators, added to a running total.
// v_mfma_f32_16x16x4f32 rounds the accumulator every 4 products, so an
// unsegmented sum over 10^5 beams rounds ~5*10^4 times per element; the
// segments bound that to KSEG/4 + K/KSEG.  (The 16-bit products accumulate
// 32 products per rounding and are not segmented.)
template <int PREC, int EPI>
constexpr bool k_segmented() {
  return (EPI == EPI_GRAMQ || EPI == EPI_GRAMQ_SMALL) && PREC == BIP_PREC_FP32;
}
constexpr int KSEG = 2048;

// The quadratic form's epilogue stages the job's psi^T tile [rho][r] in LDS
// once the K loop is done, rows padded by 16 bytes against bank conflicts of
// the per-lane reads.
template <int PREC>
constexpr int quad_row() {
  return Tile<PREC, EPI_QUAD>::BN + 16 / PT<PREC>::ESZ;
}
template <int PREC>
constexpr int quad_lds_bytes() {
  return PT<PREC>::PLANES * Tile<PREC, EPI_QUAD>::BM * quad_row<PREC>() * PT<PREC>::ESZ;
}
template <int PREC, int EPI>
constexpr int kernel_lds_bytes() {
  return (EPI == EPI_QUAD && quad_lds_bytes<PREC>() > Tile<PREC, EPI>::LDS) ? quad_lds_bytes<PREC>()
                                                                            : Tile<PREC, EPI>::LDS;
}

// s_waitcnt vmcnt(N) lgkmcnt(0): this wave's loads older than its last N
// have landed and its LDS reads are complete
template <int N>
__device__ inline void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
}

// Workgroup barrier without the memory fence of __syncthreads, which would
// wait for every load in flight; the waits before it are explicit (wait_vm).
// The clobber keeps the compiler from moving memory accesses across it.
__device__ inline void chunk_barrier() { asm volatile("s_barrier" ::: "memory"); }

// 16-byte slot permutation of LDS row `row`.  A 16-byte-per-lane LDS read is
// served in groups of 8 lanes, 128 bytes per cycle: lanes 0-3 with 20-23,
// 4-7 with 16-19, 8-11 with 28-31, 12-15 with 24-27 (and the same 32 lanes
// higher).  With fragment lane l reading row l%16, slot (l/16) ^ swz(row),
// every group then hits eight distinct 16-byte bank quads; the permutation
// also keeps 8 or 16 consecutive lanes conflict-free.
__device__ inline int swz(int row) { return ((row >> 1) & 3) ^ ((row >> 3) & 1); }

template <typename T>
__device__ inline T neg8(T a) {  // sign flip of eight 16-bit floats (bf16 or fp16)
  v4u u = __builtin_bit_cast(v4u, a);
  u ^= 0x80008000u;
  return __builtin_bit_cast(T, u);
}

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// Issue the direct-to-LDS loads of one K chunk of one operand (all planes).
// Wave w, instruction i covers tile rows 16 (RPW w + i) .. +15; lane l writes
// LDS bytes [16 l, 16 l + 16) of that 1 KB block = row 16 (RPW w + i) + l/4,
// slot l%4, which receives global segment (l%4) ^ swz(row).
template <int PREC, int RPW, int PLANE>
__device__ inline void issue_rows(const char* gbase, int64_t plane_bytes, int64_t ld_bytes,
                                  int64_t k0_bytes, char* lds_op, int wave, int lane) {
#pragma unroll
  for (int p = 0; p < PT<PREC>::PLANES; ++p)
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const int blk = RPW * wave + i;
      const int row = 16 * blk + (lane >> 2);
      const int seg = (lane & 3) ^ swz(row);
      const char* src = gbase + p * plane_bytes + row * ld_bytes + k0_bytes + seg * 16;
      char* dst = lds_op + p * PLANE + blk * 1024;
      __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)dst, 16, 0, 0);
    }
}

// One chunk of both operands into stage `buf`.
template <int PREC, int EPI>
__device__ inline void issue_chunk(const char* A, int64_t a_plane_b, int64_t lda_b, const char* B, int64_t b_plane_b,
                                   int64_t ldb_b, int64_t k0_bytes, char* buf, int wave, int lane) {
  using T = Tile<PREC, EPI>;
  if constexpr (T::ROWS) {
    issue_rows<PREC, T::RA, T::PLA>(A, a_plane_b, lda_b, k0_bytes, buf, wave, lane);
    issue_rows<PREC, T::RB, T::PLB>(B, b_plane_b, ldb_b, k0_bytes, buf + T::OPA, wave, lane);
  } else {
    // the chunk's 1 KB pieces in LDS order (A's planes, B's planes, row blocks in each), dealt to the waves
    constexpr int UA = PT<PREC>::PLANES * T::BM / 16;
#pragma unroll
    for (int i = 0; i < T::LPC; ++i) {
      const int u = T::LPC * wave + i, v = u < UA ? u : u - UA, nb = (u < UA ? T::BM : T::BN) / 16;
      const int p = v / nb, row = 16 * (v - p * nb) + (lane >> 2), seg = (lane & 3) ^ swz(row);
      const char* src = (u < UA ? A + p * a_plane_b + row * lda_b : B + p * b_plane_b + row * ldb_b) + k0_bytes + seg * 16;
      __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(buf + u * 1024), 16, 0, 0);
    }
  }
}

template <typename T, int PLANE>
__device__ inline T lds_frag(const char* lds_op, int plane, int row, int kg) {
  return *(const T*)(lds_op + plane * PLANE + row * 64 + ((kg ^ swz(row)) << 4));
}

template <int NBM, int NBN>
struct Acc {
  v4f re[NBM][NBN], im[NBM][NBN];
  __device__ inline void zero() {
#pragma unroll
    for (int i = 0; i < NBM; ++i)
#pragma unroll
      for (int j = 0; j < NBN; ++j) {
        re[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        im[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
      }
  }
};

__device__ inline v4f mfma16(v8bf a, v8bf b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ inline v4f mfma16(v8h a, v8h b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

// Multiply one LDS-resident chunk into the accumulators.  Consecutive
// products go to different accumulators (the blocks of a row, re and im), so
// that none waits for the one before it; each accumulator takes its products
// in a fixed order.
template <int PREC, int EPI, bool CONJA>
__device__ inline void mma_chunk(const char* sA, int wm, int wn, int lane,
                                 Acc<Cfg<PREC, EPI>::NBM, Cfg<PREC, EPI>::NBN>& acc) {
  using C = Tile<PREC, EPI>;
  constexpr int NBM = C::NBM, NBN = C::NBN, PA = C::PLA, PB = C::PLB;
  const char* sB = sA + C::OPA;
  const int lr = lane & 15, kg = lane >> 4;
  const int ra = wm * 16 * NBM + lr, rb = wn * 16 * NBN + lr;
  // scheduling hint: interleave the fragment reads with the products of a
  // chunk as for a single wave per SIMD (3-5% on the Gram matrix and the
  // quadratic form)
  __builtin_amdgcn_iglp_opt(1);
  if constexpr (PREC == BIP_PREC_FP32) {
    float4 bR[NBN], bI[NBN];
#pragma unroll
    for (int bn = 0; bn < NBN; ++bn) {
      bR[bn] = lds_frag<float4, PB>(sB, 0, rb + bn * 16, kg);
      bI[bn] = lds_frag<float4, PB>(sB, 1, rb + bn * 16, kg);
    }
#pragma unroll
    for (int bm = 0; bm < NBM; ++bm) {
      const float4 aR = lds_frag<float4, PA>(sA, 0, ra + bm * 16, kg);
      const float4 aI = lds_frag<float4, PA>(sA, 1, ra + bm * 16, kg);
      const float ar[4] = {aR.x, aR.y, aR.z, aR.w};
      const float ai[4] = {aI.x, aI.y, aI.z, aI.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // (ar + i s ai)(br + i bi), s = -1 for conj(A)
        const float ain = CONJA ? ai[q] : -ai[q];
        const float aip = CONJA ? -ai[q] : ai[q];
#pragma unroll
        for (int bn = 0; bn < NBN; ++bn) {
          const float br = q == 0 ? bR[bn].x : q == 1 ? bR[bn].y : q == 2 ? bR[bn].z : bR[bn].w;
          const float bi = q == 0 ? bI[bn].x : q == 1 ? bI[bn].y : q == 2 ? bI[bn].z : bI[bn].w;
          acc.re[bm][bn] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[q], br, acc.re[bm][bn], 0, 0, 0);
          acc.im[bm][bn] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[q], bi, acc.im[bm][bn], 0, 0, 0);
        }
#pragma unroll
        for (int bn = 0; bn < NBN; ++bn) {
          const float br = q == 0 ? bR[bn].x : q == 1 ? bR[bn].y : q == 2 ? bR[bn].z : bR[bn].w;
          const float bi = q == 0 ? bI[bn].x : q == 1 ? bI[bn].y : q == 2 ? bI[bn].z : bI[bn].w;
          acc.re[bm][bn] = __builtin_amdgcn_mfma_f32_16x16x4f32(ain, bi, acc.re[bm][bn], 0, 0, 0);
          acc.im[bm][bn] = __builtin_amdgcn_mfma_f32_16x16x4f32(aip, br, acc.im[bm][bn], 0, 0, 0);
        }
      }
    }
  } else if constexpr (PREC == BIP_PREC_SPLIT_BF16) {
    v8bf bRh[NBN], bRl[NBN], bIh[NBN], bIl[NBN];
#pragma unroll
    for (int bn = 0; bn < NBN; ++bn) {
      bRh[bn] = lds_frag<v8bf, PB>(sB, 0, rb + bn * 16, kg);
      bRl[bn] = lds_frag<v8bf, PB>(sB, 1, rb + bn * 16, kg);
      bIh[bn] = lds_frag<v8bf, PB>(sB, 2, rb + bn * 16, kg);
      bIl[bn] = lds_frag<v8bf, PB>(sB, 3, rb + bn * 16, kg);
    }
#pragma unroll
    for (int bm = 0; bm < NBM; ++bm) {
      const v8bf aRh = lds_frag<v8bf, PA>(sA, 0, ra + bm * 16, kg);
      const v8bf aRl = lds_frag<v8bf, PA>(sA, 1, ra + bm * 16, kg);
      const v8bf aIh = lds_frag<v8bf, PA>(sA, 2, ra + bm * 16, kg);
      const v8bf aIl = lds_frag<v8bf, PA>(sA, 3, ra + bm * 16, kg);
      const v8bf nIh = neg8(aIh), nIl = neg8(aIl);
      // the re accumulation takes -aI (+aI for conj(A)); the im one +aI (-aI)
      const v8bf rIh = CONJA ? aIh : nIh, rIl = CONJA ? aIl : nIl;
      const v8bf iIh = CONJA ? nIh : aIh, iIl = CONJA ? nIl : aIl;
      // one term of the six of re and of im, every block of the row
      auto term = [&](const v8bf& ar, const v8bf (&br)[NBN], const v8bf& ai, const v8bf (&bi)[NBN]) {
#pragma unroll
        for (int bn = 0; bn < NBN; ++bn) {
          acc.re[bm][bn] = mfma16(ar, br[bn], acc.re[bm][bn]);
          acc.im[bm][bn] = mfma16(ai, bi[bn], acc.im[bm][bn]);
        }
      };
      term(aRl, bRh, aRl, bIh);
      term(aRh, bRl, aRh, bIl);
      term(rIl, bIh, iIl, bRh);
      term(rIh, bIl, iIh, bRl);
      term(aRh, bRh, aRh, bIh);
      term(rIh, bIh, iIh, bRh);
    }
  } else {
    using V = std::conditional_t<PREC == BIP_PREC_FP16, v8h, v8bf>;
    V bR[NBN], bI[NBN];
#pragma unroll
    for (int bn = 0; bn < NBN; ++bn) {
      bR[bn] = lds_frag<V, PB>(sB, 0, rb + bn * 16, kg);
      bI[bn] = lds_frag<V, PB>(sB, 1, rb + bn * 16, kg);
    }
#pragma unroll
    for (int bm = 0; bm < NBM; ++bm) {
      const V aR = lds_frag<V, PA>(sA, 0, ra + bm * 16, kg);
      const V aI = lds_frag<V, PA>(sA, 1, ra + bm * 16, kg);
      const V nI = neg8(aI);
      const V rI = CONJA ? aI : nI, iI = CONJA ? nI : aI;
#pragma unroll
      for (int bn = 0; bn < NBN; ++bn) {
        acc.re[bm][bn] = mfma16(aR, bR[bn], acc.re[bm][bn]);
        acc.im[bm][bn] = mfma16(aR, bI[bn], acc.im[bm][bn]);
      }
#pragma unroll
      for (int bn = 0; bn < NBN; ++bn) {
        acc.re[bm][bn] = mfma16(rI, bI[bn], acc.re[bm][bn]);
        acc.im[bm][bn] = mfma16(iI, bR[bn], acc.im[bm][bn]);
      }
    }
  }
}

// This wave's loads older than those of the last `later` chunks have landed.
template <int LPC, int MOST>
__device__ inline void wait_chunks(int later) {
  if constexpr (MOST >= 2) {
    if (later >= 2) return wait_vm<2 * LPC>();
  }
  if constexpr (MOST >= 1) {
    if (later >= 1) return wait_vm<LPC>();
  }
  wait_vm<0>();
}

// acc = sum over K of A[m0 + .][k] B[n0 + .][k] (A and B point at the tile origins).
// Chunk kc lives in LDS buffer kc mod NS; the loads of chunks kc+1 .. kc+NS-2
// may still be in flight while chunk kc is multiplied.
template <int PREC, int EPI, bool CONJA>
__device__ inline void tile_product(const char* A, int64_t a_plane_b, int64_t lda_b, const char* B,
                                    int64_t b_plane_b, int64_t ldb_b, int K, int64_t CH, char* lds,
                                    int wave, int lane, int wm, int wn,
                                    Acc<Cfg<PREC, EPI>::NBM, Cfg<PREC, EPI>::NBN>& acc) {
  // CH: bytes between consecutive K chunks of a row (64 when K is contiguous)
  using T = Tile<PREC, EPI>;
  constexpr int NS = T::NS;
  const int nk = K / PT<PREC>::BK;
  auto issue = [&](int kc) {
    issue_chunk<PREC, EPI>(A, a_plane_b, lda_b, B, b_plane_b, ldb_b, kc * CH, lds + (kc % NS) * T::SB, wave, lane);
  };
  for (int kc = 0; kc < NS - 1 && kc < nk; ++kc) issue(kc);
  for (int kc = 0; kc < nk; ++kc) {
    // chunk kc has landed for every wave (the later chunks issued so far may
    // still be in flight), and every wave is done with chunk kc - 1
    wait_chunks<T::LPC, NS - 2>(min(NS - 2, nk - 1 - kc));
    chunk_barrier();
    if (kc + NS - 1 < nk) issue(kc + NS - 1);  // into the buffer of chunk kc - 1
    mma_chunk<PREC, EPI, CONJA>(lds + (kc % NS) * T::SB, wm, wn, lane, acc);
  }
  // all reads of the last buffer finish before the caller reuses LDS
  __syncthreads();
}

// ------------------------------------------------------------- the kernel
// Crop mask of a job (PRISM interpolation factor > 1): scan rho = u S_x + v
// is kept when (u - cu0) mod S_y < cnu and (v - cv0) mod S_x < cnv.
__device__ inline bool crop_in(const GemmJob& j, int rho, int Sy, int Sx) {
  const int u = rho / Sx, v = rho - u * Sx;
  return (u - j.cu0 + Sy) % Sy < j.cnu && (v - j.cv0 + Sx) % Sx < j.cnv;
}
// Whether any raster row of the scans rho0 .. rho1 is inside the job's crop
// rows (uniform per workgroup: a tile with none skips the job).
__device__ inline bool crop_rows_any(const GemmJob& j, int rho0, int rho1, int Sy, int Sx) {
  if (j.cnu <= 0 || j.cnv <= 0) return false;
  for (int u = rho0 / Sx; u <= rho1 / Sx && u < Sy; ++u)
    if ((u - j.cu0 + Sy) % Sy < j.cnu) return true;
  return false;
}

// Upper-triangle tile e of an nt x nt tile grid in blocked order: super-blocks
// of GS x GS tiles, row-major over the super-blocks with I <= J, row-major
// inside each (the diagonal ones triangular).  A run of consecutive e then
// touches few distinct row blocks of the operand.
constexpr int GS = 8;
__host__ __device__ inline void blocked_tile(int e, int nt, int& ti, int& tj) {
  const int ns = (nt + GS - 1) / GS;
  for (int I = 0; I < ns; ++I) {
    const int ri = GS < nt - I * GS ? GS : nt - I * GS;
    for (int J = I; J < ns; ++J) {
      const int cj = GS < nt - J * GS ? GS : nt - J * GS;
      const int sz = I == J ? ri * (ri + 1) / 2 : ri * cj;
      if (e >= sz) {
        e -= sz;
        continue;
      }
      int i = 0, j;
      if (I == J) {
        while (e >= ri - i) {
          e -= ri - i;
          ++i;
        }
        j = i + e;
      } else {
        i = e / cj;
        j = e - i * cj;
      }
      ti = I * GS + i;
      tj = J * GS + j;
      return;
    }
  }
  ti = tj = nt;  // not reached for e < nt (nt + 1) / 2
}

// The Gram units of a launch: every (job, K segment, upper-triangle workgroup
// tile), in that order, g.ksplit equal K segments per job.  Job j's units
// start at s0 * ksplit (s0: the tiles of the jobs before it).  Q is stored in
// GRAM_TILE blocks (the quadratic form's columns); of the smaller tiles of a
// block on the diagonal, the one below it is the conjugate transpose of the
// one above, or with g.whole_diag a product of its own (listed after the
// others).
constexpr int GRAM_TILE = 128;
__host__ __device__ inline int gram_tiles(int n_lim, int bm, int whole_diag) {
  const int nt = (n_lim + bm - 1) / bm, R = GRAM_TILE / bm, rest = nt % R;
  return nt * (nt + 1) / 2 + (whole_diag ? nt / R * (R * (R - 1) / 2) + rest * (rest - 1) / 2 : 0);
}
struct GramUnit {
  int jb, seg, m0, n0;
};
template <int BM>
__device__ inline GramUnit gram_unit(const GemmArgs& g, int u, int ksplit) {
  constexpr int R = GRAM_TILE / BM;  // tiles of a block's side
  static_assert(R * BM == GRAM_TILE, "whole tiles a block");
  int lo = 0, hi = g.njobs - 1;  // the job: the last with s0 ksplit <= u
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (g.jobs[mid].s0 * ksplit <= u) lo = mid;
    else hi = mid - 1;
  }
  const int n_lim = g.jobs[lo].n_lim, nt = (n_lim + BM - 1) / BM;
  const int T = gram_tiles(n_lim, BM, g.whole_diag);
  int e = u - g.jobs[lo].s0 * ksplit;
  GramUnit r;
  r.jb = lo;
  r.seg = e / T;
  e -= r.seg * T;
  int ti, tj;
  if (e < nt * (nt + 1) / 2) {
    blocked_tile(e, nt, ti, tj);
  } else {
    // below the diagonal of block b, row by row
    constexpr int C = R > 1 ? R * (R - 1) / 2 : 1;
    e -= nt * (nt + 1) / 2;
    const int b = e / C;
    e -= b * C;
    int i = 1;
    while (e >= i) e -= i++;
    ti = R * b + i;
    tj = R * b + e;
  }
  r.m0 = ti * BM;
  r.n0 = tj * BM;
  return r;
}

// H of a Gram tile's BM rows and BM columns, every channel, staged in LDS so
// that the per-element channel sums do not wait on memory once per channel.
template <int BM>
__device__ inline void gram_stage_h(const GemmArgs& g, const GemmJob& job, int m0, int n0, float2* sHm,
                                    float2* sHn, int tid, int nthreads) {
  for (int i = tid; i < g.n_ch * BM; i += nthreads) {
    const int c = i / BM, j = i - c * BM;
    const int64_t hc = job.h_off + (int64_t)c * job.W2;
    sHm[i] = m0 + j < job.W2 ? g.H[hc + m0 + j] : make_float2(0.f, 0.f);
    sHn[i] = n0 + j < job.W2 ? g.H[hc + n0 + j] : make_float2(0.f, 0.f);
  }
}

// Q = G * sum_c conj(H_c(r)) H_c(r') of one row of a wave's blocks (NBN blocks
// of 16 columns from n, rows m .. m + 3), stored as operand planes.
template <int OPREC, int BM, int NBN>
__device__ inline void gram_store(const GemmArgs& g, const GemmJob& job, int m0, int n0, int mrow, int ncol,
                                  const v4f (&re)[NBN], const v4f (&im)[NBN], bool hlds, const float2* sHm,
                                  const float2* sHn) {
  const bool block_diag = m0 / GRAM_TILE == n0 / GRAM_TILE;
  // the conjugate transpose is stored too, unless it has a unit of its own
  const bool mirror = m0 < n0 && !(block_diag && g.whole_diag);
#pragma unroll
  for (int bn = 0; bn < NBN; ++bn) {
    const int n = n0 + ncol + bn * 16;
    if (n >= job.ldo) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = m0 + mrow + v;
      const float cr = g.gscale * re[bn][v], ci = g.gscale * im[bn][v];
      float qr = 0.f, qi = 0.f;
      if (m < job.W2 && n < job.W2) {
        float hr = 0.f, hi = 0.f;
        if (hlds) {
          for (int c = 0; c < g.n_ch; ++c) {
            const float2 a = sHm[c * BM + (m - m0)];
            const float2 b = sHn[c * BM + (n - n0)];
            hr += a.x * b.x + a.y * b.y;
            hi += a.x * b.y - a.y * b.x;
          }
        } else {
          for (int c = 0; c < g.n_ch; ++c) {
            const float2 a = g.H[job.h_off + (int64_t)c * job.W2 + m];
            const float2 b = g.H[job.h_off + (int64_t)c * job.W2 + n];
            hr += a.x * b.x + a.y * b.y;
            hi += a.x * b.y - a.y * b.x;
          }
        }
        // spelled out: the compiler may contract these either way, and Q is to have the same bits
        // in each kernel that writes it, and those it had before
        qr = fmaf(cr, hr, -(ci * hi));
        qi = fmaf(ci, hr, cr * hi);
      }
      if (g.qtri && !block_diag) {
        // block-triangular Q for the quadratic form: psi^H Q psi sums each
        // block pair r < r' twice (Q Hermitian), so the block above the
        // diagonal is stored doubled and the one below is never read
        store_planes<OPREC>(g.out, job.out_off + (int64_t)m * job.ldo + n, g.out_plane, 2.f * qr, 2.f * qi);
      } else {
        store_planes<OPREC>(g.out, job.out_off + (int64_t)m * job.ldo + n, g.out_plane, qr, qi);
        // Q is Hermitian: below the diagonal it is the conjugate transpose
        if (mirror && m < job.ldo)
          store_planes<OPREC>(g.out, job.out_off + (int64_t)n * job.ldo + m, g.out_plane, qr, -qi);
      }
      if (g.out2) {  // G itself, for the gradient
        const bool in = m < job.W2 && n < job.W2;
        g.out2[job.out_off + (int64_t)m * job.ldo + n] = in ? make_float2(cr, ci) : make_float2(0.f, 0.f);
        if (mirror && m < job.ldo)
          g.out2[job.out_off + (int64_t)n * job.ldo + m] = in ? make_float2(cr, -ci) : make_float2(0.f, 0.f);
      }
    }
  }
}

template <int PREC, int EPI, bool CONJA, int OPREC = PREC>
__global__ __launch_bounds__((Tile<PREC, EPI>::NT), (Cfg<PREC, EPI>::WPE)) void k_zgemm(const GemmArgs g) {
  extern __shared__ char smem[];
  using T = Tile<PREC, EPI>;
  constexpr int BM = T::BM, BN = T::BN, NT = T::NT, NBM = T::NBM, NBN = T::NBN;
  constexpr int ESZ = PT<PREC>::ESZ;
  constexpr bool ACCUM = (EPI == EPI_ABS2_MAP || EPI == EPI_ABS2_BEAMS || EPI == EPI_QUAD);
  constexpr bool ABS2 = EPI == EPI_ABS2_MAP || EPI == EPI_ABS2_BEAMS;
  constexpr bool GRAM = EPI == EPI_GRAMQ || EPI == EPI_GRAMQ_SMALL;
  // wave index in a scalar register: the LDS destinations of the direct loads
  // and the wave's tile offsets are then scalar values
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;
  const int lr = lane & 15, kg = lane >> 4;
  int m0, n0, jb0, jb1, kseg = 0, unit = 0;
  if constexpr (GRAM) {
    // 1-D grid.  Workgroup i runs on XCD i mod 8, and each XCD takes one
    // contiguous eighth of the launch's units: its tiles of one job and K
    // segment share their operand row blocks in its L2, and every XCD has the
    // same number of (equal) units whatever the windows of the launch.
    const int per = (int)(gridDim.x >> 3), slot = (int)(blockIdx.x >> 3);
    unit = (int)(blockIdx.x & 7) * per + slot;
    if (unit >= g.nunits) return;  // uniform per workgroup
    const GramUnit r = gram_unit<BM>(g, unit, g.ksplit);
    jb0 = r.jb;
    jb1 = jb0 + 1;
    kseg = r.seg;
    m0 = r.m0;
    n0 = r.n0;
  } else if constexpr (ABS2) {
    // 1-D grid.  The tiles in panels of 8 along N, row by row down a panel, are
    // cut into eight equal runs, one per XCD (workgroup i runs on XCD i mod 8):
    // the tiles an XCD runs together share a few row blocks of A and the
    // panel's of B in its L2, and every XCD has work however narrow the output
    // is (super-blocks of 16 x 16 tiles had left half of the XCDs idle up to
    // 8 tiles of scans).
    constexpr int PN = 8;
    const int per = (int)(gridDim.x >> 3), u = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (u >= g.mtiles * g.ntiles) return;  // uniform per workgroup
    const int panel = u / (g.mtiles * PN), e = u - panel * g.mtiles * PN;
    const int pw = min(PN, g.ntiles - panel * PN);
    const int mt = e / pw, nt = panel * PN + e - mt * pw;
    m0 = mt * (EPI == EPI_ABS2_MAP ? ABS2_MAP_ROWS : BM);
    n0 = nt * BN;
    jb0 = (int)((int64_t)g.njobs * blockIdx.z / g.zsplit);  // job group z of g.zsplit
    jb1 = (int)((int64_t)g.njobs * (blockIdx.z + 1) / g.zsplit);
  } else {
    // consecutive workgroups take consecutive M tiles of one N tile
    m0 = blockIdx.x * BM;
    n0 = blockIdx.y * BN;
    if constexpr (EPI == EPI_QUAD) {  // job group and K segment
      const int jz = g.zsplit / g.ksplit, zj = (int)blockIdx.z / g.ksplit;
      kseg = (int)blockIdx.z - zj * g.ksplit;
      jb0 = (int)((int64_t)g.njobs * zj / jz);
      jb1 = (int)((int64_t)g.njobs * (zj + 1) / jz);
    } else {  // EPI_STORE: one job per grid z
      jb0 = (int)blockIdx.z;
      jb1 = jb0 + 1;
    }
  }
  v4f sq[NBM][NBN];
  if constexpr (ACCUM) {
#pragma unroll
    for (int i = 0; i < NBM; ++i)
#pragma unroll
      for (int j = 0; j < NBN; ++j) sq[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  Acc<NBM, NBN> acc;
  if constexpr (ABS2) {
    // The jobs' K chunks run as one stream: the loads of the next job's first
    // chunks are issued under the last products of the current one, so a job
    // switch drains nothing (its epilogue is in registers).
    constexpr int NS = T::NS;
    // the map sums over d, so its workgroups take MF tiles of rows, each (job, tile) a job of its own
    constexpr int MF = EPI == EPI_ABS2_MAP ? ABS2_MAP_ROWS / BM : 1;
    auto next_job = [&](int j) {
      for (; j < jb1 * MF; ++j) {
        const GemmJob& q = g.jobs[j / MF];
        if (n0 >= q.n_lim || m0 >= q.m_lim) continue;
        // a tile holding no scan of the job's crop mask skips the job
        if (g.crop && !crop_rows_any(q, n0, min(n0 + BN - 1, g.P - 1), g.Sy, g.Sx)) continue;
        break;
      }
      return j;
    };
    int ij = next_job(jb0 * MF), ikc = 0, ink = 0, ibuf = 0, ahead = 0;  // ahead: chunks issued, not multiplied
    const char *iA = nullptr, *iB = nullptr;
    int64_t ilda = 0, ildb = 0;
    auto load_job = [&]() {
      if (ij >= jb1 * MF) return;
      const GemmJob& q = g.jobs[ij / MF];
      iA = (const char*)g.A + (q.a_off + (int64_t)(m0 + ij % MF * BM) * q.lda) * ESZ;
      iB = (const char*)g.B + (q.b_off + (int64_t)n0 * q.ldb) * ESZ;
      ilda = (int64_t)q.lda * ESZ;
      ildb = (int64_t)q.ldb * ESZ;
      ink = q.K / PT<PREC>::BK;
    };
    auto issue_next = [&]() {
      if (ij >= jb1 * MF) return;
      issue_chunk<PREC, EPI>(iA, g.a_plane * ESZ, ilda, iB, g.b_plane * ESZ, ildb, (int64_t)ikc * 64,
                             smem + ibuf * T::SB, wave, lane);
      ibuf = ibuf + 1 == NS ? 0 : ibuf + 1;
      ++ahead;
      if (++ikc == ink) {
        ij = next_job(ij + 1);
        ikc = 0;
        load_job();
      }
    };
    int cj = ij, ckc = 0, cbuf = 0;
    load_job();
    int cnk = ink;
    acc.zero();
#pragma unroll
    for (int i = 0; i < NS - 1; ++i) issue_next();
    while (ahead > 0) {
      wait_chunks<T::LPC, NS - 2>(ahead - 1);
      chunk_barrier();
      issue_next();
      mma_chunk<PREC, EPI, CONJA>(smem + cbuf * T::SB, wm, wn, lane, acc);
      cbuf = cbuf + 1 == NS ? 0 : cbuf + 1;
      --ahead;
      if (++ckc == cnk) {
#pragma unroll
        for (int j = 0; j < NBN; ++j) {
          // column n = scan rho of this lane's block j
          const bool keep = !g.crop || crop_in(g.jobs[cj / MF], n0 + wn * 16 * NBN + j * 16 + lr, g.Sy, g.Sx);
#pragma unroll
          for (int i = 0; i < NBM; ++i)
            if (keep) sq[i][j] += acc.re[i][j] * acc.re[i][j] + acc.im[i][j] * acc.im[i][j];
        }
        acc.zero();
        cj = next_job(cj + 1);
        ckc = 0;
        if (cj < jb1 * MF) cnk = g.jobs[cj / MF].K / PT<PREC>::BK;
      }
    }
    __syncthreads();
  } else {
    for (int jb = jb0; jb < jb1; ++jb) {
      const GemmJob job = g.jobs[jb];
      if (n0 >= job.n_lim || m0 >= job.m_lim) continue;  // uniform per workgroup
      // the block-triangular quadratic form runs K over r' >= the tile's first r
      int k0 = 0, k1 = job.K;
      if constexpr (EPI == EPI_QUAD) {
        const int nk = job.K / PT<PREC>::BK;
        k0 = max(g.qtri ? n0 : 0, (int)((int64_t)nk * kseg / g.ksplit) * PT<PREC>::BK);
        k1 = (int)((int64_t)nk * (kseg + 1) / g.ksplit) * PT<PREC>::BK;
        if (k0 >= k1) continue;
      } else if constexpr (GRAM) {
        const int nk = job.K / PT<PREC>::BK;
        k0 = (int)((int64_t)nk * kseg / g.ksplit) * PT<PREC>::BK;
        k1 = (int)((int64_t)nk * (kseg + 1) / g.ksplit) * PT<PREC>::BK;
      }
      const int64_t ch = (job.kstride ? (int64_t)job.kstride : (int64_t)PT<PREC>::BK) * ESZ;
      const int64_t kb = (int64_t)(k0 / PT<PREC>::BK) * ch;
      const char* Ap = (const char*)g.A + (job.a_off + (int64_t)m0 * job.lda) * ESZ + kb;
      const char* Bp = (const char*)g.B + (job.b_off + (int64_t)n0 * job.ldb) * ESZ + kb;
      acc.zero();
      if constexpr (k_segmented<PREC, EPI>()) {
        Acc<NBM, NBN> seg;
        for (int ks = 0; ks < k1 - k0; ks += KSEG) {
          seg.zero();
          const int64_t koff = (int64_t)(ks / PT<PREC>::BK) * ch;  // K chunks of the segment's start
          tile_product<PREC, EPI, CONJA>(Ap + koff, g.a_plane * ESZ, (int64_t)job.lda * ESZ, Bp + koff,
                                         g.b_plane * ESZ, (int64_t)job.ldb * ESZ, min(KSEG, k1 - k0 - ks), ch,
                                         smem, wave, lane, wm, wn, seg);
#pragma unroll
          for (int i = 0; i < NBM; ++i)
#pragma unroll
            for (int j = 0; j < NBN; ++j) {
              acc.re[i][j] += seg.re[i][j];
              acc.im[i][j] += seg.im[i][j];
            }
        }
      } else {
        tile_product<PREC, EPI, CONJA>(Ap, g.a_plane * ESZ, (int64_t)job.lda * ESZ, Bp, g.b_plane * ESZ,
                                       (int64_t)job.ldb * ESZ, k1 - k0, ch, smem, wave, lane, wm, wn, acc);
      }
      if constexpr (EPI == EPI_QUAD) {
        // Re conj(psi^T[rho][r]) (Q psi)^T[rho][r]; psi is read back from the A
        // operand: the tile's rows m0.. and columns n0.. (columns below the
        // row length lda, which K-chunks never straddle) go to LDS in 16-byte
        // coalesced pieces, then every lane reads its elements from there
        constexpr int QR = quad_row<PREC>(), QPL = BM * QR, CH = 16 / ESZ;
        constexpr int NCH = BN / CH;  // 16-byte pieces per row
        constexpr int NPC = PT<PREC>::PLANES * BM * NCH;  // pieces of the tile
        constexpr int QB = NPC / NT < 16 ? NPC / NT : 16;  // loads in flight per thread before their LDS stores
        static_assert(NPC % (NT * QB) == 0, "whole rounds of pieces");
        for (int i0 = tid; i0 < NPC; i0 += NT * QB) {
          uint4 val[QB];
#pragma unroll
          for (int u = 0; u < QB; ++u) {
            const int i = i0 + u * NT;
            const int pl = i / (BM * NCH), rem = i - pl * (BM * NCH);
            const int row = rem / NCH, ch = rem - row * NCH;
            const int r = n0 + ch * CH;
            val[u] = make_uint4(0u, 0u, 0u, 0u);
            if (r < job.lda)
              val[u] = *(const uint4*)((const char*)g.A +
                                       (job.a_off + (int64_t)(m0 + row) * job.lda + r + pl * g.a_plane) * ESZ);
          }
#pragma unroll
          for (int u = 0; u < QB; ++u) {
            const int i = i0 + u * NT;
            const int pl = i / (BM * NCH), rem = i - pl * (BM * NCH);
            const int row = rem / NCH, ch = rem - row * NCH;
            *(uint4*)(smem + ((int64_t)pl * QPL + row * QR + ch * CH) * ESZ) = val[u];
          }
        }
        __syncthreads();
#pragma unroll
        for (int bn = 0; bn < NBN; ++bn) {
          const int rl = wn * 16 * NBN + bn * 16 + lr;  // r - n0
          if (n0 + rl >= job.W2) continue;
#pragma unroll
          for (int bm = 0; bm < NBM; ++bm)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int rhol = wm * 16 * NBM + bm * 16 + kg * 4 + v;  // rho - m0
              const float2 ps = load_planes<PREC>(smem, (int64_t)rhol * QR + rl, QPL);
              sq[bm][bn][v] += ps.x * acc.re[bm][bn][v] + ps.y * acc.im[bm][bn][v];
            }
        }
        __syncthreads();  // the next job's K loop refills LDS
      } else if constexpr (EPI == EPI_STORE) {
        float2* o = (float2*)g.out;
#pragma unroll
        for (int bn = 0; bn < NBN; ++bn) {
          const int n = n0 + wn * 16 * NBN + bn * 16 + lr;
          if (n >= job.ldo) continue;
#pragma unroll
          for (int bm = 0; bm < NBM; ++bm)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int m = m0 + wm * 16 * NBM + bm * 16 + kg * 4 + v;
              if (m >= g.m_store) continue;
              const float s = g.rowscale ? g.rowscale[m] : 1.f;
              o[job.out_off + (int64_t)m * job.ldo + n] =
                  make_float2(s * acc.re[bm][bn][v], s * acc.im[bm][bn][v]);
            }
        }
      } else {
        // EPI_GRAMQ
        if (g.ksplit > 1) {  // partial tile in register order, summed by k_gram_finish
          float4* o = g.gpart + (int64_t)unit * T::QUADS * NT + tid;
#pragma unroll
          for (int bm = 0; bm < NBM; ++bm)
#pragma unroll
            for (int bn = 0; bn < NBN; ++bn) {
              o[(2 * (bm * NBN + bn)) * NT] = __builtin_bit_cast(float4, acc.re[bm][bn]);
              o[(2 * (bm * NBN + bn) + 1) * NT] = __builtin_bit_cast(float4, acc.im[bm][bn]);
            }
        } else {
          const bool hlds = g.n_ch * 2 * BM * (int)sizeof(float2) <= T::LDS;
          float2* sHm = (float2*)smem;
          float2* sHn = sHm + (hlds ? g.n_ch * BM : 0);
          if (hlds) {
            gram_stage_h<BM>(g, job, m0, n0, sHm, sHn, tid, NT);
            __syncthreads();
          }
#pragma unroll
          for (int bm = 0; bm < NBM; ++bm)
            gram_store<OPREC, BM, NBN>(g, job, m0, n0, wm * 16 * NBM + bm * 16 + kg * 4, wn * 16 * NBN + lr,
                                       acc.re[bm], acc.im[bm], hlds, sHm, sHn);
        }
      }
    }
  }
  if constexpr (EPI == EPI_ABS2_MAP) {
    // map partial sums over the tile's d (rows), fixed order
    __shared__ float red[T::WM][BN];
    float cs[NBN];
#pragma unroll
    for (int bn = 0; bn < NBN; ++bn) {
      float s = 0.f;
#pragma unroll
      for (int bm = 0; bm < NBM; ++bm)
        s += (sq[bm][bn][0] + sq[bm][bn][1]) + (sq[bm][bn][2] + sq[bm][bn][3]);
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      cs[bn] = s;
    }
    if (kg == 0) {
#pragma unroll
      for (int bn = 0; bn < NBN; ++bn) red[wm][wn * 16 * NBN + bn * 16 + lr] = cs[bn];
    }
    __syncthreads();
    if (tid < BN) {
      float s = red[0][tid];
#pragma unroll
      for (int w = 1; w < T::WM; ++w) s += red[w][tid];
      g.partial[((int64_t)blockIdx.z * g.mtiles + m0 / ABS2_MAP_ROWS) * g.Npad + n0 + tid] = g.oscale * s;
    }
  } else if constexpr (EPI == EPI_QUAD) {
    // rows rho = m0 + 16 NBM wm + 16 bm + 4 kg + v; sum over r (lanes lr, blocks bn, waves wn)
    __shared__ float red[T::WN][BM];
#pragma unroll
    for (int bm = 0; bm < NBM; ++bm)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        static_assert(EPI != EPI_QUAD || (NBN == 4 && T::WN == 2), "64-column waves, 128-column tiles");
        float s = (sq[bm][0][v] + sq[bm][1][v]) + (sq[bm][2][v] + sq[bm][3][v]);
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        s += __shfl_xor(s, 4);
        s += __shfl_xor(s, 8);
        if (lr == 0) red[wn][wm * 16 * NBM + bm * 16 + kg * 4 + v] = s;
      }
    __syncthreads();
    if (tid < BM)
      g.partial[((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * g.Mpad + m0 + tid] = red[0][tid] + red[1][tid];
  } else if constexpr (EPI == EPI_ABS2_BEAMS) {
    // one job group adds to the output, several store their own slices (summed
    // in group order by k_sum_slices)
    float* const out = g.zsplit > 1 ? g.slices + (int64_t)blockIdx.z * g.P * g.ndet : g.out_beams;
#pragma unroll
    for (int bn = 0; bn < NBN; ++bn) {
      const int rho = n0 + wn * 16 * NBN + bn * 16 + lr;
      if (rho >= g.P) continue;
#pragma unroll
      for (int bm = 0; bm < NBM; ++bm)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int d = m0 + wm * 16 * NBM + bm * 16 + kg * 4 + v;
          if (d >= g.ndet) continue;
          const float x = g.oscale * sq[bm][bn][v];
          float* o = out + (int64_t)rho * g.ndet + d;
          *o = g.zsplit > 1 ? x : *o + x;
        }
    }
  }
}

// K segments where the tiles alone leave the chip idle (gemm_gram_ksplit): one
// atom of 32 x 32 pixels and 2053 beams is 36 tiles of 65 chunks, 330 us on the
// 32 CUs of one XCD; in 7 segments on all of them 32 us, and 10 us for this
// kernel: the sum of a Gram tile's ksplit partial products (in segment order)
// and its epilogue.  A workgroup takes one row of the waves' blocks of a tile (grid y),
// with the thread layout of the product kernel.
template <int PREC, int OPREC>
__global__ __launch_bounds__((Tile<PREC, EPI_GRAMQ>::NT)) void k_gram_finish(const GemmArgs g, int hlds) {
  extern __shared__ char smem[];
  using T = Tile<PREC, EPI_GRAMQ>;
  constexpr int BM = T::BM, NT = T::NT, NBM = T::NBM, NBN = T::NBN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN, lr = lane & 15, kg = lane >> 4;
  const GramUnit r = gram_unit<BM>(g, (int)blockIdx.x, 1);  // tile blockIdx.x of the launch
  const GemmJob job = g.jobs[r.jb];
  const int m0 = r.m0, n0 = r.n0, bm = blockIdx.y;
  const int Tj = gram_tiles(job.n_lim, BM, g.whole_diag);
  const int64_t u0 = (int64_t)job.s0 * g.ksplit + ((int)blockIdx.x - job.s0);
  v4f re[NBN], im[NBN];
#pragma unroll
  for (int bn = 0; bn < NBN; ++bn) re[bn] = im[bn] = v4f{0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < g.ksplit; ++s) {
    const float4* p = g.gpart + (u0 + (int64_t)s * Tj) * T::QUADS * NT + tid;
#pragma unroll
    for (int bn = 0; bn < NBN; ++bn) {
      re[bn] += __builtin_bit_cast(v4f, p[(2 * (bm * NBN + bn)) * NT]);
      im[bn] += __builtin_bit_cast(v4f, p[(2 * (bm * NBN + bn) + 1) * NT]);
    }
  }
  float2* sHm = (float2*)smem;
  float2* sHn = sHm + (hlds ? g.n_ch * BM : 0);
  if (hlds) {
    gram_stage_h<BM>(g, job, m0, n0, sHm, sHn, tid, NT);
    __syncthreads();
  }
  gram_store<OPREC, BM, NBN>(g, job, m0, n0, wm * 16 * NBM + bm * 16 + kg * 4, wn * 16 * NBN + lr, re, im,
                             hlds != 0, sHm, sHn);
}

// -------------------------------------------------------------- helpers
__global__ void k_reduce_map(const float* __restrict__ partial, int ntiles, int Ppad, int P,
                             float* out, int accumulate) {
  const int rho = blockIdx.x * blockDim.x + threadIdx.x;
  if (rho >= P) return;
  float s = 0.f;
#pragma unroll 16  // loads in flight; the sum stays in order
  for (int t = 0; t < ntiles; ++t) s += partial[(int64_t)t * Ppad + rho];
  out[rho] = accumulate ? out[rho] + s : s;
}

// The quadratic form at f > 1 runs one job (atom) at a time over the scans of
// its crop mask; here every scan collects its atoms, in job order.
__global__ void k_reduce_crop(const float* __restrict__ partial, const GemmJob* __restrict__ jobs, int njobs, int ntiles,
                              int pitch, int Sy, int Sx, float* out) {
  const int rho = blockIdx.x * blockDim.x + threadIdx.x;
  if (rho >= Sy * Sx) return;
  const int u = rho / Sx, v = rho - u * Sx;
  float s = 0.f;
  for (int j = 0; j < njobs; ++j) {
    const GemmJob& q = jobs[j];
    const int iu = (u - q.cu0 + Sy) % Sy, iv = (v - q.cv0 + Sx) % Sx;
    if (iu >= q.cnu || iv >= q.cnv) continue;
    const int nt = min(ntiles, (q.n_lim + GRAM_TILE - 1) / GRAM_TILE);  // the job's column tiles
    const float* p = partial + (int64_t)j * ntiles * pitch + iu * q.cnv + iv;
    for (int t = 0; t < nt; ++t) s += p[(int64_t)t * pitch];
  }
  out[rho] += s;
}

// qEELS: sum the per-beam intensities over h_y at fixed h_x, in detector order
__global__ void k_qeels(const float* __restrict__ beams_out, const int32_t* __restrict__ bin_start,
                        const int32_t* __restrict__ bin_list, int ndet, int P, int nq,
                        float* out, int accumulate) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)P * nq) return;
  const int rho = (int)(i / nq);
  const int q = (int)(i - (int64_t)rho * nq);
  float s = 0.f;
  const int k1 = bin_start[q + 1];
#pragma unroll 8  // loads in flight, the sum in order: 426 us for 2304 scans of a 1024^2 field, 1390 one by one
  for (int k = bin_start[q]; k < k1; ++k)
    s += beams_out[(int64_t)rho * ndet + bin_list[k]];
  out[i] = accumulate ? out[i] + s : s;
}

// out += the slices of the job groups, in group order
__global__ void k_sum_slices(const float* __restrict__ slices, int z, int64_t n, float* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s = slices[i];
  for (int k = 1; k < z; ++k) s += slices[(int64_t)k * n + i];
  out[i] += s;
}

template <int PREC, int EPI, bool CONJA, int OPREC = PREC>
hipError_t zgemm_launch(const GemmArgs& g, dim3 grid, hipStream_t s) {
  const void* f = (const void*)k_zgemm<PREC, EPI, CONJA, OPREC>;
  constexpr int lds = kernel_lds_bytes<PREC, EPI>();
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_zgemm<PREC, EPI, CONJA, OPREC>), grid, dim3(Tile<PREC, EPI>::NT), lds, s, g);
  return hipGetLastError();
}

template <int PREC>
hipError_t zgemm_prec(int epi, const GemmArgs& g, dim3 grid, hipStream_t s) {
  switch (epi) {
    case EPI_ABS2_MAP: return zgemm_launch<PREC, EPI_ABS2_MAP, false>(g, grid, s);
    case EPI_ABS2_BEAMS: return zgemm_launch<PREC, EPI_ABS2_BEAMS, false>(g, grid, s);
    case EPI_QUAD: return zgemm_launch<PREC, EPI_QUAD, false>(g, grid, s);
    case EPI_STORE: return zgemm_launch<PREC, EPI_STORE, false>(g, grid, s);
    case EPI_STORE + EPI_CONJ_A: return zgemm_launch<PREC, EPI_STORE, true>(g, grid, s);
    default: return hipErrorInvalidValue;
  }
}

template <int PREC, int OPREC>
hipError_t gram_launch(const GemmArgs& g, int tiles, hipStream_t s) {
  using T = Tile<PREC, EPI_GRAMQ>;
  const dim3 grid((unsigned)((g.nunits + 7) / 8 * 8));
  if (g.gram_bm != T::BM) {
    if constexpr (PREC == BIP_PREC_FP32) {
      if (g.gram_bm == Tile<PREC, EPI_GRAMQ_SMALL>::BM && g.ksplit == 1)
        return zgemm_launch<PREC, EPI_GRAMQ_SMALL, true, OPREC>(g, grid, s);
    }
    return hipErrorInvalidValue;
  }
  hipError_t e = zgemm_launch<PREC, EPI_GRAMQ, true, OPREC>(g, grid, s);
  if (e != hipSuccess || g.ksplit == 1) return e;
  const int lds = g.n_ch * 2 * T::BM * (int)sizeof(float2);
  const int hlds = lds <= 65536;
  hipLaunchKernelGGL((k_gram_finish<PREC, OPREC>), dim3((unsigned)tiles, T::NBM), dim3(T::NT), hlds ? lds : 0, s, g,
                     hlds);
  return hipGetLastError();
}

constexpr int GRAM_SMALL = 32;
static_assert(Tile<BIP_PREC_FP32, EPI_GRAMQ_SMALL>::BM == GRAM_SMALL && Tile<BIP_PREC_FP32, EPI_GRAMQ_SMALL>::BN == GRAM_SMALL, "");
constexpr int gram_bm(int prec) { return prec == BIP_PREC_FP32 ? 64 : 128; }
static_assert(Tile<BIP_PREC_FP32, EPI_GRAMQ>::BM == 64 && Tile<BIP_PREC_SPLIT_BF16, EPI_GRAMQ>::BM == 128 &&
                  Tile<BIP_PREC_BF16, EPI_GRAMQ>::BM == 128 && Tile<BIP_PREC_FP16, EPI_GRAMQ>::BM == 128,
              "tiles of gram_bm");

}  // namespace

void gemm_tile(int prec, int epi, int& m, int& n) {
  m = n = prec == BIP_PREC_FP32 ? 64 : 128;
  if (epi == EPI_QUAD) n = 128;
  if (epi == EPI_ABS2_MAP) m = ABS2_MAP_ROWS;
}
static_assert(Tile<BIP_PREC_FP32, EPI_QUAD>::BM == 64 && Tile<BIP_PREC_SPLIT_BF16, EPI_QUAD>::BM == 128 &&
                  Tile<BIP_PREC_FP32, EPI_QUAD>::BN == 128 && Tile<BIP_PREC_SPLIT_BF16, EPI_QUAD>::BN == 128 &&
                  Tile<BIP_PREC_FP32, EPI_STORE>::BM == 64 && Tile<BIP_PREC_FP32, EPI_STORE>::BN == 64 &&
                  Tile<BIP_PREC_FP32, EPI_ABS2_BEAMS>::BM == 64 && Tile<BIP_PREC_FP32, EPI_ABS2_BEAMS>::BN == 64 &&
                  Tile<BIP_PREC_SPLIT_BF16, EPI_STORE>::BM == 128 && Tile<BIP_PREC_SPLIT_BF16, EPI_STORE>::BN == 128 &&
                  Tile<BIP_PREC_SPLIT_BF16, EPI_ABS2_BEAMS>::BM == 128 && Tile<BIP_PREC_SPLIT_BF16, EPI_ABS2_BEAMS>::BN == 128,
              "tiles of gemm_tile");

hipError_t launch_zgemm_gram(int in_prec, int out_prec, const GemmArgs& g0, int tiles, hipStream_t s) {
  if (tiles <= 0 || g0.njobs <= 0) return hipSuccess;
  if (!(g0.gscale > 0.f) || g0.ksplit < 1 || (g0.ksplit > 1 && !g0.gpart)) return hipErrorInvalidValue;
  if ((int64_t)tiles * g0.ksplit > INT32_MAX / 2) return hipErrorInvalidValue;
  GemmArgs g = g0;
  g.nunits = tiles * g.ksplit;
  if (in_prec == BIP_PREC_FP16 && out_prec == BIP_PREC_SPLIT_BF16)
    return gram_launch<BIP_PREC_FP16, BIP_PREC_SPLIT_BF16>(g, tiles, s);
  if (in_prec != out_prec) return hipErrorInvalidValue;
  switch (in_prec) {
    case BIP_PREC_FP32: return gram_launch<BIP_PREC_FP32, BIP_PREC_FP32>(g, tiles, s);
    case BIP_PREC_SPLIT_BF16: return gram_launch<BIP_PREC_SPLIT_BF16, BIP_PREC_SPLIT_BF16>(g, tiles, s);
    case BIP_PREC_BF16: return gram_launch<BIP_PREC_BF16, BIP_PREC_BF16>(g, tiles, s);
    case BIP_PREC_FP16: return gram_launch<BIP_PREC_FP16, BIP_PREC_FP16>(g, tiles, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_zgemm(int prec, int epi, const GemmArgs& g, int gx, int gy, int gz,
                        hipStream_t s) {
  if (gx <= 0 || gy <= 0 || gz <= 0 || g.njobs <= 0) return hipSuccess;
  if (epi == EPI_QUAD && (g.ksplit < 1 || g.zsplit != gz || gz % g.ksplit || gz / g.ksplit > g.njobs))
    return hipErrorInvalidValue;
  if (epi == EPI_GRAMQ) return hipErrorInvalidValue;  // launch_zgemm_gram
  dim3 grid(gx, gy, gz);
  GemmArgs ga = g;
  if (epi == EPI_ABS2_MAP || epi == EPI_ABS2_BEAMS) {
    if (g.zsplit != gz || gz > g.njobs || (epi == EPI_ABS2_BEAMS && gz > 1 && !g.slices)) return hipErrorInvalidValue;
    ga.mtiles = gx;
    ga.ntiles = gy;
    const int64_t n = ((int64_t)gx * gy + 7) / 8 * 8;
    if (n > INT32_MAX) return hipErrorInvalidValue;
    grid = dim3((unsigned)n, 1, gz);
  }
  hipError_t e = hipErrorInvalidValue;
  switch (prec) {
    case BIP_PREC_FP32: e = zgemm_prec<BIP_PREC_FP32>(epi, ga, grid, s); break;
    case BIP_PREC_SPLIT_BF16: e = zgemm_prec<BIP_PREC_SPLIT_BF16>(epi, ga, grid, s); break;
    case BIP_PREC_BF16: e = zgemm_prec<BIP_PREC_BF16>(epi, ga, grid, s); break;
    case BIP_PREC_FP16: e = zgemm_prec<BIP_PREC_FP16>(epi, ga, grid, s); break;
  }
  if (e == hipSuccess && epi == EPI_ABS2_BEAMS && gz > 1) {
    const int64_t n = (int64_t)g.P * g.ndet;
    hipLaunchKernelGGL(k_sum_slices, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g.slices, gz, n, g.out_beams);
    e = hipGetLastError();
  }
  return e;
}

int64_t gemm_gram_tiles(int n_lim, int prec, int whole_diag) { return gram_tiles(n_lim, gram_bm(prec), whole_diag); }

int64_t gemm_gram_plan(GemmJob* jobs, int njobs, int prec, int whole_diag, int n_cu, int& bm) {
  auto lay = [&] {
    int64_t n = 0;
    for (int j = 0; j < njobs; ++j) {
      jobs[j].s0 = (int32_t)n;
      n += gram_tiles(jobs[j].n_lim, bm, whole_diag);
    }
    return n;
  };
  bm = gram_bm(prec);
  const int64_t n = lay();
  // whole_diag: no K segments either, so few tiles are cut smaller (Cfg)
  if (!whole_diag || prec != BIP_PREC_FP32 || n >= n_cu) return n;
  bm = GRAM_SMALL;
  return lay();
}

int64_t gemm_gram_part_bytes(int prec) {
  return (int64_t)gram_bm(prec) * gram_bm(prec) * (int64_t)sizeof(float2);
}

int gemm_gram_ksplit(int prec, int64_t tiles, int K, int n_cu, int64_t part_bytes) {
  const int64_t cus = std::max<int64_t>(1, n_cu / 8);  // of an XCD
  const int64_t nk = K / gemm_bk(prec), per = gemm_gram_part_bytes(prec);
  int best = 1;
  double cost = 0;
  for (int q = 1; q <= 16 && q * 4 <= nk; ++q) {
    if (q > 1 && tiles * q * per > part_bytes) break;
    const int64_t mine = (tiles * q + 7) / 8;  // units of an XCD
    // units of a CU (they share its matrix cores), each its chunks and about GRAM_FILL chunk
    // times of filling and epilogue; the partial tiles' way out and back, and their sum
    const double c = (double)((mine + cus - 1) / cus) * ((double)((nk + q - 1) / q) + GRAM_FILL) +
                     (q > 1 ? GRAM_PART * (double)per / 131072 * (double)tiles * q + GRAM_FILL : 0.0);
    if (q == 1 || c < 0.97 * cost) {
      best = q;
      cost = c;
    }
  }
  return best;
}

int gemm_bk(int prec) { return prec == BIP_PREC_FP32 ? PT<BIP_PREC_FP32>::BK : 32; }

hipError_t launch_reduce_map(const float* partial, int ntiles, int Ppad, int P, float* out,
                             int accumulate, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_map, dim3((P + 255) / 256), dim3(256), 0, s, partial, ntiles, Ppad,
                     P, out, accumulate);
  return hipGetLastError();
}

hipError_t launch_reduce_crop(const float* partial, const GemmJob* jobs, int njobs, int ntiles, int pitch, int Sy,
                              int Sx, float* out, hipStream_t s) {
  if (njobs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_crop, dim3((Sy * Sx + 63) / 64), dim3(64), 0, s, partial, jobs, njobs, ntiles, pitch, Sy,
                     Sx, out);
  return hipGetLastError();
}

hipError_t launch_qeels_from_beams(const float* beams_out, const int32_t* bin_start,
                                   const int32_t* bin_list, int ndet, int P, int nq, float* out,
                                   int accumulate, hipStream_t s) {
  const int64_t n = (int64_t)P * nq;
  hipLaunchKernelGGL(k_qeels, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, beams_out,
                     bin_start, bin_list, ndet, P, nq, out, accumulate);
  return hipGetLastError();
}

}  // namespace bip
