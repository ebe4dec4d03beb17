// fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32) with the stage's fused
// epilogues: every product of an fp32 stage whose operands are 16-byte aligned.
//
// A block of WGM x WGN waves owns a BM x BN output tile, each wave 32 FM x 32 FN
// of it.  k-tiles of 32 values go from global memory through registers (the loads
// of tile kt + 2 are in flight while tile kt is multiplied and tile kt + 1 is in LDS)
// into a double-buffered LDS stage in the operand's own orientation:
//  - k-contiguous operands as [row][32 k] (16-byte chunks permuted by the row);
//    a lane reads 4 consecutive k of its row with one ds_read_b128;
//  - operands contiguous along m / n as [k][R]; a lane reads its column of one k
//    row with ds_read_b32 (32-column groups swapped on every other 4 k rows, so
//    the two lane halves use different banks).
// The reduction index of MFMA step (i, e) is 8 i + 4 G + e for lane half G in both.
//
// One 32 x 32 x 2 product occupies a SIMD's matrix core for 64 cycles, so a single
// fragment per operand already keeps LDS reads (32 B/clk/CU of 128) and the
// operand traffic of a 64 x 64 tile (16 B/clk/CU) below their limits: slice
// products take 64 x 64 tiles for the sake of many workgroups and split the
// reduction when they are still few, products of many tiles 128 x 128.
// Width 1024, 256-token slices, averages over a layer's products against the
// strided FMA kernel: forward 337 -> 23 us (+ 5 us reduction), dX 468 -> 22 us (+ 5),
// weight gradients over 1024 tokens 253 -> 69 us: 71, 74 and 94 TFLOP/s of 157 nominal;
// reading the fragments a step ahead, or one workgroup a CU without splits, was 2-4 %
// slower over the layer.
#include "tp_common.hpp"
#include "tp_epilogue.hpp"
#include "tp_kernels.hpp"

#include <algorithm>

namespace tp {

namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int BK = 32;

// LDS offset (floats) of element (row r, k) of a k-contiguous tile and of element
// (k, column r) of an m/n-contiguous tile of R columns
__device__ inline int kc_off(int r, int k) {
  return r * BK + ((((k >> 2) ^ r ^ (r >> 3)) & 7) << 2) + (k & 3);
}
template <int R>
__device__ inline int mc_off(int k, int r) {
  return k * R + (r ^ (((k >> 2) & 1) << 5));
}

// One R x 32 operand tile: X(r, k) = X[r * ld + k] (KC) or X[k * ld + r].
template <int R, int NTH, bool KC>
struct Tile32 {
  static constexpr int CH = R * BK / 4 / NTH;  // 16-byte chunks per thread
  float4 v[CH];
  // (row or column, k) of this thread's chunk i
  __device__ static int2 at(int i) {
    const int s = threadIdx.x + NTH * i;
    if constexpr (KC) return make_int2(s >> 3, (s & 7) * 4);
    else return make_int2((s % (R / 4)) * 4, s / (R / 4));
  }
  unsigned ok;  // bit i: chunk i lies inside the operand
  // A chunk is inside or outside as a whole (the contiguous extent is a multiple of
  // 4).  Outside ones load the nearest valid chunk and are cleared when stored: no
  // branch around a load, which would wait for it where the paths join.
  __device__ void load(const float* X, long ld, int r0, int rmax, int k0, int kmax) {
    ok = 0;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int2 p = at(i);
      const int r = r0 + p.x, k = k0 + p.y;
      ok |= (r < rmax && k < kmax ? 1u : 0u) << i;
      const int rc = min(r, KC ? rmax - 1 : rmax - 4), kc = min(k, KC ? kmax - 4 : kmax - 1);
      v[i] = *(const float4*)(KC ? X + (long)rc * ld + kc : X + (long)kc * ld + rc);
    }
  }
  __device__ void store(float* lds) const {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int2 p = at(i);
      const bool in = (ok >> i) & 1;
      const float4 x = make_float4(in ? v[i].x : 0.f, in ? v[i].y : 0.f, in ? v[i].z : 0.f,
                                   in ? v[i].w : 0.f);
      *(float4*)(lds + (KC ? kc_off(p.x, p.y) : mc_off<R>(p.y, p.x))) = x;
    }
  }
  // values k = 8 i + 4 G + e (e < 4) of row / column r
  __device__ static void frag(const float* lds, int r, int i, int G, float (&x)[4]) {
    const int k = 8 * i + 4 * G;
    if constexpr (KC) {
      const float4 u = *(const float4*)(lds + kc_off(r, k));
      x[0] = u.x, x[1] = u.y, x[2] = u.z, x[3] = u.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = lds[mc_off<R>(k + e, r)];
    }
  }
};

template <int BM, int BN, int WGM, int WGN, bool A_KC, bool B_KC, int EPI, bool SPLIT>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_f32_kernel(GemmArgs a) {
  constexpr int NTH = 64 * WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 32, FN = WN / 32;
  using TA = Tile32<BM, NTH, A_KC>;
  using TB = Tile32<BN, NTH, B_KC>;
  __shared__ __attribute__((aligned(16))) float As[2][BM * BK];
  __shared__ __attribute__((aligned(16))) float Bs[2][BN * BK];
  const float* A = (const float*)a.A;
  const float* B = (const float*)a.B;
  const long lda = A_KC ? a.sam : a.sak, ldb = B_KC ? a.sbn : a.sbk;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int G = lane >> 5, c = lane & 31;
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;
  const int kbeg = SPLIT ? blockIdx.z * a.k_split : 0;
  const int kend = SPLIT ? min(a.K, kbeg + a.k_split) : a.K;
  const int nk = (kend - kbeg + BK - 1) / BK;

  f32x16_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  TA ta;
  TB tb;
  auto load = [&](int kt) {
    ta.load(A, lda, m0, a.M, kbeg + kt * BK, kend);
    tb.load(B, ldb, n0, a.N, kbeg + kt * BK, kend);
  };
  if (nk > 0) {
    load(0);
    ta.store(As[0]);
    tb.store(Bs[0]);
    if (nk > 1) load(1);
  }
  for (int kt = 0; kt < nk; ++kt) {
    __syncthreads();  // tile kt is in LDS; every wave has left tile kt - 1
    if (kt + 1 < nk) {
      ta.store(As[(kt + 1) & 1]);
      tb.store(Bs[(kt + 1) & 1]);
    }
    if (kt + 2 < nk) load(kt + 2);
    const float* at = As[kt & 1];
    const float* bt = Bs[kt & 1];
#pragma unroll
    for (int i = 0; i < BK / 8; ++i) {
      float fa[FM][4], fb[FN][4];
#pragma unroll
      for (int x = 0; x < FM; ++x) TA::frag(at, wm0 + 32 * x + c, i, G, fa[x]);
#pragma unroll
      for (int y = 0; y < FN; ++y) TB::frag(bt, wn0 + 32 * y + c, i, G, fb[y]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int x = 0; x < FM; ++x)
#pragma unroll
          for (int y = 0; y < FN; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[x][e], fb[y][e], acc[x][y], 0, 0, 0);
    }
  }
  // acc[x][y][v]: row 8 (v / 4) + 4 G + v % 4, column c of the 32 x 32 tile
  float* part = SPLIT ? a.ws + (long)blockIdx.z * a.M * a.N : nullptr;
#pragma unroll
  for (int x = 0; x < FM; ++x)
#pragma unroll
    for (int y = 0; y < FN; ++y)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = m0 + wm0 + 32 * x + 8 * (v >> 2) + 4 * G + (v & 3);
        const int n = n0 + wn0 + 32 * y + c;
        if (m < a.M && n < a.N) {
          if constexpr (SPLIT)
            part[(long)m * a.N + n] = acc[x][y][v];
          else
            epi1<float, EPI>(a, m, n, acc[x][y][v]);
        }
      }
}

// Sums the split partials in split order and applies the epilogue.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_f32_kernel(GemmArgs a) {
  const long tot = (long)a.M * a.N;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < tot; e += (long)gridDim.x * 256) {
    float s = 0.f;
    for (int z = 0; z < a.splits; ++z) s += a.ws[z * tot + e];
    epi1<float, EPI>(a, (int)(e / a.N), (int)(e % a.N), s);
  }
}

#define TP_EPI_SWITCH(LAUNCH)                  \
  switch (a.epi) {                             \
    case EPI_STORE: LAUNCH(EPI_STORE); break;  \
    case EPI_QKV: LAUNCH(EPI_QKV); break;      \
    case EPI_RESID: LAUNCH(EPI_RESID); break;  \
    case EPI_GELU: LAUNCH(EPI_GELU); break;    \
    case EPI_DGELU: LAUNCH(EPI_DGELU); break;  \
    case EPI_ACC_F32: LAUNCH(EPI_ACC_F32); break; \
    default: return hipErrorInvalidValue;      \
  }

template <int BM, int BN, int WGM, int WGN, bool A_KC, bool B_KC>
hipError_t launch_f32(const GemmArgs& a, hipStream_t s) {
  constexpr int NTH = 64 * WGM * WGN;
  const dim3 grid(cdiv(a.N, BN), cdiv(a.M, BM), a.splits);
  if (a.splits > 1) {
    gemm_f32_kernel<BM, BN, WGM, WGN, A_KC, B_KC, EPI_STORE, true><<<grid, NTH, 0, s>>>(a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int blocks = (int)std::min<long>(cdiv((long)a.M * a.N, 256), 4096);
#define TP_RED(E) splitk_reduce_f32_kernel<E><<<blocks, 256, 0, s>>>(a)
    TP_EPI_SWITCH(TP_RED)
#undef TP_RED
    return hipGetLastError();
  }
#define TP_ONE(E) gemm_f32_kernel<BM, BN, WGM, WGN, A_KC, B_KC, E, false><<<grid, NTH, 0, s>>>(a)
  TP_EPI_SWITCH(TP_ONE)
#undef TP_ONE
  return hipGetLastError();
}

template <bool A_KC, bool B_KC>
hipError_t run_f32(GemmArgs a, hipStream_t s) {
  // 128 x 128 tiles (16 products per 4 fragment reads) once they fill the 256 CUs,
  // else 64 x 64 tiles, two to four workgroups of which share a CU
  if ((long)cdiv(a.M, 128) * cdiv(a.N, 128) >= 256) {
    if (!a.need) return launch_f32<128, 128, 2, 2, A_KC, B_KC>(a, s);
    return hipSuccess;
  }
  // Split count: a round is two workgroups on each CU, whose waves share the
  // matrix cores (about 0.9 us per k-tile); a split adds the reduction launch and
  // the partials' round trip.  The partials stay within the capacity of the static
  // scratch, so a split never makes the static forward refuse a slice.
  const long tiles = (long)cdiv(a.M, 64) * cdiv(a.N, 64);
  const int nkt = cdiv(a.K, BK);
  const long cap = std::min<long>(a.ws ? a.ws_elems : 0, STATIC_SCRATCH_ELEMS);
  double best = 1e30;
  for (int sp = 1; sp <= 16 && sp * 4 <= std::max(nkt, 4); ++sp) {
    if (sp > 1 && (long)sp * a.M * a.N > cap) break;
    const double t = cdiv(tiles * sp, 512) * (1.5 + 0.9 * cdiv(nkt, sp)) +
                     (sp > 1 ? 4.0 + (double)sp * a.M * a.N * 8.0 / 5e6 : 0.0);
    if (t < best) best = t, a.splits = sp;
  }
  a.k_split = cdiv(nkt, a.splits) * BK;
  a.splits = std::max(1, cdiv(a.K, a.k_split));
  if (a.need) {
    *a.need = a.splits > 1 ? (long)a.splits * a.M * a.N : 0;
    return hipSuccess;
  }
  return launch_f32<64, 64, 2, 2, A_KC, B_KC>(a, s);
}

}  // namespace

// fp32 operands with a unit stride, 16-byte-aligned bases, leading dimensions and
// contiguous extents of whole 16-byte chunks; anything else is left to the strided
// kernel.
hipError_t gemm_f32(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  const bool a_kc = a.sak == 1, b_kc = a.sbk == 1;
  if ((!a_kc && a.sam != 1) || (!b_kc && a.sbn != 1)) return hipErrorNotSupported;
  const long lda = a_kc ? a.sam : a.sak, ldb = b_kc ? a.sbn : a.sbk;
  if (((uintptr_t)a.A & 15) || ((uintptr_t)a.B & 15) || (lda & 3) || (ldb & 3))
    return hipErrorNotSupported;
  // whole 4-value chunks along the contiguous dimension of each operand
  if (a.K <= 0 || (a_kc ? a.K : a.M) % 4 || (b_kc ? a.K : a.N) % 4) return hipErrorNotSupported;
  if (a_kc && b_kc) return run_f32<true, true>(a, s);
  if (a_kc) return run_f32<true, false>(a, s);
  if (!b_kc) return run_f32<false, false>(a, s);
  return hipErrorNotSupported;
}

}  // namespace tp
