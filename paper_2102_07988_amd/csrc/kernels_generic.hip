// Generic kernels of the stage: a strided tiled-FMA GEMM with the fused epilogues
// for the operands the matrix-core GEMMs do not take (unaligned parameters),
// LayerNorm forward/backward, column reductions.
#include "tp_common.hpp"
#include "tp_epilogue.hpp"
#include "tp_kernels.hpp"

#include <algorithm>

namespace tp {

// ------------------------------------------------------------- generic GEMM

template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_generic_kernel(GemmArgs a) {
  __shared__ float As[16][65];
  __shared__ float Bs[16][65];
  const T* A = (const T*)a.A;
  const T* B = (const T*)a.B;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  // contiguous dimension of each operand decides the load order (coalescing)
  const bool a_k_fast = a.sak == 1;
  const bool b_n_fast = a.sbn == 1;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < a.K; k0 += 16) {
    for (int e = threadIdx.x; e < 1024; e += 256) {
      int kk, mm;
      if (a_k_fast) {
        kk = e & 15;
        mm = e >> 4;
      } else {
        kk = e >> 6;
        mm = e & 63;
      }
      const int gm = m0 + mm, gk = k0 + kk;
      As[kk][mm] = (gm < a.M && gk < a.K) ? ld(A + (long)gm * a.sam + (long)gk * a.sak) : 0.f;
      int kb, nn;
      if (b_n_fast) {
        kb = e >> 6;
        nn = e & 63;
      } else {
        kb = e & 15;
        nn = e >> 4;
      }
      const int gn = n0 + nn, gkb = k0 + kb;
      Bs[kb][nn] = (gn < a.N && gkb < a.K) ? ld(B + (long)gkb * a.sbk + (long)gn * a.sbn) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = As[kk][ty + 16 * i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bv[j] = Bs[kk][tx + 16 * j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += av[i] * bv[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + ty + 16 * i, n = n0 + tx + 16 * j;
      if (m < a.M && n < a.N) epi1<T, EPI>(a, m, n, acc[i][j]);
    }
}

template <typename T>
static hipError_t gemm_generic_t(const GemmArgs& a, hipStream_t s) {
  if (a.need || a.M <= 0 || a.N <= 0) return hipSuccess;  // no scratch
  dim3 grid(cdiv(a.N, 64), cdiv(a.M, 64));
  switch (a.epi) {
    case EPI_STORE: gemm_generic_kernel<T, EPI_STORE><<<grid, 256, 0, s>>>(a); break;
    case EPI_QKV: gemm_generic_kernel<T, EPI_QKV><<<grid, 256, 0, s>>>(a); break;
    case EPI_RESID: gemm_generic_kernel<T, EPI_RESID><<<grid, 256, 0, s>>>(a); break;
    case EPI_GELU: gemm_generic_kernel<T, EPI_GELU><<<grid, 256, 0, s>>>(a); break;
    case EPI_DGELU: gemm_generic_kernel<T, EPI_DGELU><<<grid, 256, 0, s>>>(a); break;
    case EPI_ACC_F32: gemm_generic_kernel<T, EPI_ACC_F32><<<grid, 256, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t gemm_generic(int dtype, const GemmArgs& a, hipStream_t s) {
  return dtype == DT_FP32 ? gemm_generic_t<float>(a, s) : gemm_generic_t<bf16>(a, s);
}

// ------------------------------------------------------------- LayerNorm

// 8 consecutive elements <-> 8 floats (16-byte loads for bf16, 2 x 16 for fp32).
__device__ inline void load8(const bf16* p, float* v) {
  const uint4 u = *(const uint4*)p;
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
__device__ inline void load8(const float* p, float* v) {
  const float4 a = ((const float4*)p)[0], b = ((const float4*)p)[1];
  v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
}
// Gain and offset parameters: 16-byte loads where the caller's tensors are aligned (AL),
// else element by element.
template <bool AL, typename T>
__device__ inline void load8_param(const T* p, float* v) {
  if constexpr (AL) {
    load8(p, v);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ld(p + e);
  }
}
__device__ inline void store8(bf16* p, const float* v) {
  uint4 u;
  u.x = f32_to_bf16_bits(v[0]) | ((uint32_t)f32_to_bf16_bits(v[1]) << 16);
  u.y = f32_to_bf16_bits(v[2]) | ((uint32_t)f32_to_bf16_bits(v[3]) << 16);
  u.z = f32_to_bf16_bits(v[4]) | ((uint32_t)f32_to_bf16_bits(v[5]) << 16);
  u.w = f32_to_bf16_bits(v[6]) | ((uint32_t)f32_to_bf16_bits(v[7]) << 16);
  *(uint4*)p = u;
}
__device__ inline void store8(float* p, const float* v) {
  ((float4*)p)[0] = make_float4(v[0], v[1], v[2], v[3]);
  ((float4*)p)[1] = make_float4(v[4], v[5], v[6], v[7]);
}

// One block per row; the row stays in registers (H % 8 == 0, H <= 16384).  The
// block has nt threads (a multiple of 64, <= 1024) and thread t owns the
// 8-element chunks t + nt * c, c < CPT; CPT = 2 only when H / 8 > 1024.  Every
// load a thread makes (row, gamma, beta, residual) is issued before the first
// reduction, so a row costs one memory latency instead of several.
struct LnShape {
  int cpt, nt;
};
inline LnShape ln_shape(int H) {
  const int nc = H / 8, cpt = nc > 1024 ? 2 : 1;
  return {cpt, cdiv(cdiv(nc, cpt), 64) * 64};
}

// T: stage dtype (gamma, beta, u); TX: type of the input rows x (fp32 for the
// residual stream of a mixed-precision stage).  x_copy (fp32 when copy_f32, else
// T) and u16 (fp16 copy of u) are optional.
template <typename T, typename TX, int CPT, bool AL>
__global__ __launch_bounds__(1024) void ln_fwd_kernel(int H, const TX* x, void* x_copy,
                                                      int copy_f32, const T* g, const T* b, T* u,
                                                      f16s* u16, float* mean, float* rstd,
                                                      float eps) {
  __shared__ float red[16];
  const int row = blockIdx.x, nc = H >> 3, nt = blockDim.x;
  const TX* xr = x + (long)row * H;
  float v[CPT][8], gg[CPT][8], bb[CPT][8];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ci = threadIdx.x + nt * c;
    if (ci < nc) {
      load8(xr + ci * 8, v[c]);
      load8_param<AL>(g + ci * 8, gg[c]);
      load8_param<AL>(b + ci * 8, bb[c]);
    }
  }
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < CPT; ++c)
    if (threadIdx.x + nt * c < nc)
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[c][e];
  const float mu = block_sum(s, red) / H;
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < CPT; ++c)
    if (threadIdx.x + nt * c < nc)
#pragma unroll
      for (int e = 0; e < 8; ++e) q += (v[c][e] - mu) * (v[c][e] - mu);
  const float rs = rsqrtf(block_sum(q, red) / H + eps);
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ci = threadIdx.x + nt * c;
    if (ci < nc) {
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = gg[c][e] * ((v[c][e] - mu) * rs) + bb[c][e];
      store8(u + (long)row * H + ci * 8, o);
      if (u16) st8(u16 + (long)row * H + ci * 8, o);
      if (x_copy) {
        if (copy_f32)
          store8((float*)x_copy + (long)row * H + ci * 8, v[c]);
        else
          store8((T*)x_copy + (long)row * H + ci * 8, v[c]);
      }
    }
  }
  if (threadIdx.x == 0) {
    mean[row] = mu;
    rstd[row] = rs;
  }
}

// Two block-wide sums in one pass (blockDim.x a multiple of 64, <= 1024).
__device__ inline float2 block_sum2(float a, float b, float* red /* >= 32 floats */) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  a = wave_sum(a);
  b = wave_sum(b);
  if (lane == 0) red[w] = a, red[16 + w] = b;
  __syncthreads();
  float sa = 0.f, sb = 0.f;
  for (int i = 0; i < nw; ++i) sa += red[i], sb += red[16 + i];
  return make_float2(sa, sb);
}

template <typename T, typename TX, int CPT, bool AL>
__global__ __launch_bounds__(1024) void ln_bwd_kernel(int H, const T* du, const TX* x,
                                                      const float* mean, const float* rstd,
                                                      const T* g, const T* resid, T* resid_copy,
                                                      T* dx) {
  __shared__ float red[32];
  const int row = blockIdx.x, nc = H >> 3, nt = blockDim.x;
  const float mu = mean[row], rs = rstd[row];
  float xh[CPT][8], dg[CPT][8], r[CPT][8];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ci = threadIdx.x + nt * c;
    if (ci < nc) {
      float gg[8];
      load8(x + (long)row * H + ci * 8, xh[c]);
      load8(du + (long)row * H + ci * 8, dg[c]);
      load8_param<AL>(g + ci * 8, gg);
      load8(resid + (long)row * H + ci * 8, r[c]);
#pragma unroll
      for (int e = 0; e < 8; ++e) dg[c][e] *= gg[e];
    }
  }
  float sa = 0.f, sb = 0.f;
#pragma unroll
  for (int c = 0; c < CPT; ++c)
    if (threadIdx.x + nt * c < nc)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xh[c][e] = (xh[c][e] - mu) * rs;
        sa += dg[c][e];
        sb += dg[c][e] * xh[c][e];
      }
  const float2 ab = block_sum2(sa, sb, red);
  const float a = ab.x / H, bm = ab.y / H;
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ci = threadIdx.x + nt * c;
    if (ci < nc) {
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        o[e] = rs * (dg[c][e] - a - xh[c][e] * bm) + r[c][e];
      store8(dx + (long)row * H + ci * 8, o);
      if (resid_copy) store8(resid_copy + (long)row * H + ci * 8, r[c]);
    }
  }
}

// Column reductions over rows: every bias and LayerNorm-parameter gradient of a
// layer in one launch.  A block owns 64 columns (8 chunks of 8: whole 128-byte
// lines of a bf16 row) of one job and one chunk of the rows; row group rg (of 32)
// sums rows rg, rg + 32, ... of the chunk in order, loading four rows at a time, then
// a column's 32 partial sums are added as 4 in-order groups of 8, the group sums in
// order.  With more than one row chunk the chunk sums go to `part` and a second
// launch adds them in order.  Deterministic.
// Bound by memory once enough blocks are in flight (11 H / 64 column blocks a layer
// are 352 at width 2048): one launch per tensor with 64-byte row pieces and no row
// split had H / 32 = 64 blocks for most tensors.  A layer's reductions, 2048 wide:
// 2048 tokens 104 -> 40 us, 8192 rows 381 -> 131 us (4 TB/s); 1024 wide, 256 tokens
// 21 us in 6 launches -> 8 us in one; 12288 wide, 2048 tokens 238 -> 168 us (4.5 TB/s).
constexpr int CR_RG = 32, CR_COLS = 64, CR_UNROLL = 4;

// The column totals of p[rg][col], in threads 0..63.
__device__ inline float col_partials_sum(float (*p)[CR_COLS + 1], float (*q)[CR_COLS]) {
  const int col = threadIdx.x & 63, grp = threadIdx.x >> 6;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) s += p[grp * 8 + i][col];
  q[grp][col] = s;
  __syncthreads();
  float t = 0.f;
  if (threadIdx.x < CR_COLS)
#pragma unroll
    for (int i = 0; i < 4; ++i) t += q[i][col];
  return t;
}

// Partial (or final) sum of one output column; slot: its column in `part`.
__device__ inline void col_out(const ColJobs& J, float* out, int col, int slot, float s) {
  if (J.chunks > 1)
    J.part[(long)blockIdx.y * J.slots + slot] = s;
  else
    out[col] = J.store ? s : out[col] + s;
}

// T: stage dtype; TX: type of the LayerNorm input rows
template <typename T, typename TX>
__global__ __launch_bounds__(256) void col_reduce_kernel(ColJobs J) {
  __shared__ float pa[CR_RG][CR_COLS + 1], pb[CR_RG][CR_COLS + 1], q[2][4][CR_COLS];
  int ji = 0;
  while (ji + 1 < J.count && (int)blockIdx.x >= J.job[ji + 1].block0) ++ji;
  const ColJob& j = J.job[ji];
  const int cc = threadIdx.x & 7, rg = threadIdx.x >> 3;
  const int col0 = (blockIdx.x - j.block0) * CR_COLS, c0 = col0 + cc * 8;
  const int r0 = blockIdx.y * J.rows_per, r1 = min(J.rows, r0 + J.rows_per);
  float sa[8] = {}, sb[8] = {};
  if (c0 < j.cols) {
    const T* A = (const T*)j.a + c0;
    const TX* X = j.x ? (const TX*)j.x + c0 : nullptr;
    for (int t0 = r0 + rg; t0 < r1; t0 += CR_UNROLL * CR_RG) {
      float d[CR_UNROLL][8], xv[CR_UNROLL][8], mu[CR_UNROLL], rs[CR_UNROLL];
#pragma unroll
      for (int k = 0; k < CR_UNROLL; ++k) {
        const int t = t0 + k * CR_RG;
        if (t < r1) {
          load8(A + (long)t * j.lda, d[k]);
          if (X) {
            load8(X + (long)t * j.lda, xv[k]);
            mu[k] = j.mean[t], rs[k] = j.rstd[t];
          }
        }
      }
#pragma unroll
      for (int k = 0; k < CR_UNROLL; ++k)
        if (t0 + k * CR_RG < r1)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            sa[e] += d[k][e];
            if (X) sb[e] += d[k][e] * ((xv[k][e] - mu[k]) * rs[k]);
          }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) pa[rg][cc * 8 + e] = sa[e], pb[rg][cc * 8 + e] = sb[e];
  __syncthreads();
  const float a = col_partials_sum(pa, q[0]);
  const float b = j.x ? col_partials_sum(pb, q[1]) : 0.f;  // uniform per block
  const int col = col0 + threadIdx.x;
  if (threadIdx.x < CR_COLS && col < j.cols) {
    col_out(J, j.sum, col, j.slot0 + col, a);
    if (j.x) col_out(J, j.xsum, col, j.slot0 + j.cols + col, b);
  }
}

// Adds the row chunks' partial sums in order; one thread per output column.
__global__ __launch_bounds__(256) void col_finish_kernel(ColJobs J) {
  const int slot = blockIdx.x * 256 + threadIdx.x;
  if (slot >= J.slots) return;
  int ji = 0;
  while (ji + 1 < J.count && slot >= J.job[ji + 1].slot0) ++ji;
  const ColJob& j = J.job[ji];
  float s = 0.f;
  for (int c = 0; c < J.chunks; ++c) s += J.part[(long)c * J.slots + slot];
  const int col = slot - j.slot0;
  float* out = col < j.cols ? j.sum + col : j.xsum + (col - j.cols);
  *out = J.store ? s : *out + s;
}

__global__ void fill_f32_kernel(float* p, size_t n, float v) {
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (size_t)gridDim.x * blockDim.x)
    p[e] = v;
}

hipError_t ln_fwd(int dtype, int n, int H, const void* x, int x_f32, void* x_copy, int copy_f32,
                  const void* g, const void* b, void* u, void* u16, float* mean, float* rstd,
                  float eps, hipStream_t s) {
  clear_stale_error();
  if (n <= 0) return hipSuccess;
  const LnShape sh = ln_shape(H);
  const bool al = !(((uintptr_t)g | (uintptr_t)b) & 15);
#define TP_LN(TT, TX, C)                                                                   \
  (al ? ln_fwd_kernel<TT, TX, C, true> : ln_fwd_kernel<TT, TX, C, false>)                  \
      <<<n, sh.nt, 0, s>>>(H, (const TX*)x, x_copy, copy_f32, (const TT*)g, (const TT*)b,   \
                           (TT*)u, (f16s*)u16, mean, rstd, eps)
  if (dtype == DT_FP32) {
    if (sh.cpt == 1) TP_LN(float, float, 1); else TP_LN(float, float, 2);
  } else if (x_f32) {
    if (sh.cpt == 1) TP_LN(bf16, float, 1); else TP_LN(bf16, float, 2);
  } else {
    if (sh.cpt == 1) TP_LN(bf16, bf16, 1); else TP_LN(bf16, bf16, 2);
  }
#undef TP_LN
  return hipGetLastError();
}

hipError_t ln_bwd(int dtype, int n, int H, const void* du, const void* x, int x_f32,
                  const float* mean, const float* rstd, const void* g, const void* resid,
                  void* resid_copy, void* dx, hipStream_t s) {
  clear_stale_error();
  if (n <= 0) return hipSuccess;
  const LnShape sh = ln_shape(H);
  const bool al = !((uintptr_t)g & 15);
#define TP_LN(TT, TX, C)                                                                   \
  (al ? ln_bwd_kernel<TT, TX, C, true> : ln_bwd_kernel<TT, TX, C, false>)                  \
      <<<n, sh.nt, 0, s>>>(H, (const TT*)du, (const TX*)x, mean, rstd, (const TT*)g,        \
                           (const TT*)resid, (TT*)resid_copy, (TT*)dx)
  if (dtype == DT_FP32) {
    if (sh.cpt == 1) TP_LN(float, float, 1); else TP_LN(float, float, 2);
  } else if (x_f32) {
    if (sh.cpt == 1) TP_LN(bf16, float, 1); else TP_LN(bf16, float, 2);
  } else {
    if (sh.cpt == 1) TP_LN(bf16, bf16, 1); else TP_LN(bf16, bf16, 2);
  }
#undef TP_LN
  return hipGetLastError();
}

hipError_t col_reduce(int dtype, int x_f32, ColJobs J, hipStream_t s) {
  clear_stale_error();
  if (J.rows <= 0 || J.count <= 0) return hipSuccess;
  int blocks = 0, slots = 0;
  for (int i = 0; i < J.count; ++i) {
    ColJob& j = J.job[i];
    j.block0 = blocks, j.slot0 = slots;
    blocks += cdiv(j.cols, CR_COLS);
    slots += j.cols * (j.x ? 2 : 1);
  }
  J.slots = slots;
  // about 1024 blocks (4 per CU), at most 16 chunks of at least 256 rows (a 256-row
  // slice in two chunks, with their second launch, took 10 us for 8; 300 rows in two of
  // 150, 1024 wide, 2.2 us more than in one); the partials must fit
  J.chunks = (int)std::min<long>({16, std::max(1, J.rows / 256), std::max(1, cdiv(1024, blocks))});
  while (J.chunks > 1 && (!J.part || (long)J.chunks * slots > J.part_elems)) --J.chunks;
  J.rows_per = cdiv(J.rows, J.chunks);
  J.chunks = cdiv(J.rows, J.rows_per);
  const dim3 grid(blocks, J.chunks);
  if (dtype == DT_FP32)
    col_reduce_kernel<float, float><<<grid, 256, 0, s>>>(J);
  else if (x_f32)
    col_reduce_kernel<bf16, float><<<grid, 256, 0, s>>>(J);
  else
    col_reduce_kernel<bf16, bf16><<<grid, 256, 0, s>>>(J);
  if (J.chunks > 1) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    col_finish_kernel<<<cdiv(slots, 256), 256, 0, s>>>(J);
  }
  return hipGetLastError();
}

// 8 bf16 values per thread as fp16 (n % 8 == 0, 16-byte aligned), else one.
__global__ void cvt_bf16_f16_kernel(size_t n, const uint16_t* src, uint16_t* dst, int vec) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  if (vec) {
    const size_t n8 = n / 8;
    size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    // four independent 16-byte loads in flight per thread
    for (; e + 3 * stride < n8; e += 4 * stride) {
      float v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) ld8((const bf16*)src + 8 * (e + u * stride), v[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) st8((f16s*)dst + 8 * (e + u * stride), v[u]);
    }
    for (; e < n8; e += stride) {
      float v[8];
      ld8((const bf16*)src + 8 * e, v);
      st8((f16s*)dst + 8 * e, v);
    }
  } else {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride)
      dst[e] = f32_to_f16_bits(to_f32(bf16{src[e]}));
  }
}

hipError_t cvt_bf16_f16(size_t n, const void* src, void* dst, hipStream_t s) {
  clear_stale_error();
  if (n == 0) return hipSuccess;
  const int vec = n % 8 == 0 && ((uintptr_t)src & 15) == 0 && ((uintptr_t)dst & 15) == 0;
  const size_t work = vec ? n / 8 : n;
  const int blocks = (int)((work + 255) / 256 < 8192 ? (work + 255) / 256 : 8192);
  cvt_bf16_f16_kernel<<<blocks, 256, 0, s>>>(n, (const uint16_t*)src, (uint16_t*)dst, vec);
  return hipGetLastError();
}

hipError_t fill_f32(float* p, size_t n, float v, hipStream_t s) {
  clear_stale_error();
  if (n == 0) return hipSuccess;
  const int blocks = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
  fill_f32_kernel<<<blocks, 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

}  // namespace tp
