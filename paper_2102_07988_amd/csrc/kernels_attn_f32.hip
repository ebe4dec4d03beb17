// Prefix-causal attention of a token slice with every product on the fp32
// matrix cores (v_mfma_f32_32x32x2_f32): fp32 stages of any head width, and bf16
// stages with narrow heads (16, 32), whose bf16 operands are widened to fp32 as
// they are loaded.  Scores, softmax weights, dP, dS and every sum stay in fp32.
//
// MFMA fragment conventions (32 x 32 x 2): lane l = 32 G + c supplies row c of the
// left operand and column c of the right one at reduction index G; accumulator
// element v of lane l is D[8 (v / 4) + 4 G + v % 4][c].  The order of a reduction
// is free, so
//  - a product over the head width takes step (i, e) at columns 8 i + 4 G + e:
//    each lane reads 4 consecutive values of its row at a time;
//  - a score tile is fed back as an operand straight from its accumulator: step v
//    stands for row 8 (v / 4) + 4 G + v % 4 of the tile.
//
// These stages are narrow (heads x queries / 32 is near the CU count) and their
// slices short, so latency bounds them, not the matrix cores: one block owns 32
// queries (forward, dQ) or 32 keys (dK, dV) of one head, its NW waves take the
// 32-row tiles of the other side in turn (tile % NW) straight from the caches
// into registers, and the waves' partial results meet in LDS in wave order at
// the end (deterministic, no atomics).  Slices of 256 tokens after up to 768,
// against one block per query row with a serial key loop and atomic dK/dV:
// 16 heads of 64 in fp32, forward 130 -> 19 us, backward 1099 -> 70 us a slice;
// 16 heads of 32 in bf16, forward 72 -> 13 us, backward 543 -> 45 us.
#include "tp_common.hpp"
#include "tp_kernels.hpp"

namespace tp {

namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

__device__ inline f32x16_t mfma32(float a, float b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ inline f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}
// row of accumulator element v for lane half G
__device__ inline int acc_row(int v, int G) { return 8 * (v >> 2) + 4 * G + (v & 3); }

// 4 consecutive values as fp32 (p aligned to 4 elements)
__device__ inline void ld4(const float* p, float* x) {
  const float4 u = *(const float4*)p;
  x[0] = u.x, x[1] = u.y, x[2] = u.z, x[3] = u.w;
}
__device__ inline void ld4(const bf16* p, float* x) {
  const uint2 u = *(const uint2*)p;
  x[0] = __uint_as_float(u.x << 16), x[1] = __uint_as_float(u.x & 0xffff0000u);
  x[2] = __uint_as_float(u.y << 16), x[3] = __uint_as_float(u.y & 0xffff0000u);
}

// sum / maximum over the lane pair (l, l ^ 32)
__device__ inline float pair_sum(float v) { return v + __shfl_xor(v, 32, 64); }
__device__ inline float pair_max(float v) { return fmaxf(v, __shfl_xor(v, 32, 64)); }

// This lane's part of one row of D values: values 8 i + 4 G + e, i < D / 8.
template <int D, typename T>
__device__ inline void row_frag(const T* row, int G, float (&x)[D / 2]) {
#pragma unroll
  for (int i = 0; i < D / 8; ++i) ld4(row + 8 * i + 4 * G, x + 4 * i);
}
template <int D>
__device__ inline f32x16_t dot_tile(const float (&a)[D / 2], const float (&b)[D / 2]) {
  f32x16_t s = zero16();
#pragma unroll
  for (int i = 0; i < D / 2; ++i) s = mfma32(a[i], b[i], s);
  return s;
}

template <int D>
struct Shape {
  static constexpr int JB = (D + 31) / 32;        // 32-column blocks
  static constexpr int W = 32 * JB;               // padded width
  static constexpr int NW = D == 128 ? 4 : 8;     // waves per block
  static constexpr size_t part = (size_t)NW * 32 * W * 4;  // bytes of the waves' partials
};

__device__ inline bool nonfinite(float x) {
  return (__float_as_uint(x) & 0x7f800000u) == 0x7f800000u;
}

// The part of acc_cols that X's infinities and NaNs contribute: w * X of every pair
// that `sees` (tile row, lane's or accumulator row's column) admits.  Rarely run.
template <int D, bool LEFT, typename T, typename S>
__device__ inline void acc_nonfinite(const T* X, long ld, int rows, const f32x16_t& w, int G,
                                     int c, f32x16_t (&acc)[Shape<D>::JB], S sees) {
  constexpr int JB = Shape<D>::JB;
#pragma unroll 1
  for (int rr = 0; rr < rows; ++rr) {
    const int vr = 4 * (rr >> 3) + (rr & 3), half = ((rr >> 2) & 1) << 5;  // rr = acc_row(vr, half)
    float wr = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) wr = v == vr ? w[v] : wr;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int other = LEFT ? c : acc_row(v, G);  // the pair's query (LEFT) or key
      const float p = __shfl(wr, half + other, 64);
#pragma unroll
      for (int j = 0; j < JB; ++j) {
        const int col = 32 * j + (LEFT ? acc_row(v, G) : c);
        const float x = tp::ld(X + (long)rr * ld + (col & (D - 1)));
        if (nonfinite(x) && sees(rr, other)) acc[j][v] += p * x;
      }
      __builtin_amdgcn_sched_barrier(0);  // few registers rather than many loads in flight
    }
  }
}

// acc[j][v] += sum over the 32 rows of X (from row 0 of the tile, rows past
// rows - 1 repeat it; their weights are 0): X[row][32 j + c] * w[v].  As the left
// operand: acc^T (columns of X by lanes' columns).  `left` picks the side of X.
// part: some weights of the tile are 0 because the mask or the tile's end took the
// pair out (sees(row, other) is false).  Such a pair adds nothing also where X is
// infinite or NaN, so a tile with such values multiplies zeros in their place and adds
// what the admitted pairs make of them.
template <int D, bool LEFT, typename T, typename S>
__device__ inline void acc_cols(const T* X, long ld, int rows, const f32x16_t& w, int G, int c,
                                f32x16_t (&acc)[Shape<D>::JB], bool part, S sees) {
  constexpr int JB = Shape<D>::JB;
  const int cc = D < 32 ? c & (D - 1) : c;  // width 16: columns 16..31 are discarded
  float x[JB][16];
  auto load = [&](bool finite) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const T* r = X + (long)min(acc_row(v, G), rows - 1) * ld + cc;
#pragma unroll
      for (int j = 0; j < JB; ++j) {
        const float y = tp::ld(r + 32 * j);
        x[j][v] = finite && nonfinite(y) ? 0.f : y;
      }
    }
  };
  load(false);
  if (part) {
    bool bad = false;
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
      for (int j = 0; j < JB; ++j) bad |= nonfinite(x[j][v]);
    if (__any(bad)) {
      acc_nonfinite<D, LEFT>(X, ld, rows, w, G, c, acc, sees);
      load(true);
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v)
#pragma unroll
    for (int j = 0; j < JB; ++j)
      acc[j] = LEFT ? mfma32(x[j][v], w[v], acc[j]) : mfma32(w[v], x[j][v], acc[j]);
}

// The waves' [32 rows][W] partials in LDS, rows of W floats whose 16-byte chunks
// are permuted by the row, so that lanes that each write their own row spread
// over the banks.
template <int D>
__device__ inline float* part_at(float* base, int w, int row, int col) {
  constexpr int W = Shape<D>::W;
  return base + ((w * 32 + row) * W) + ((((col >> 2) ^ row) & (W / 4 - 1)) << 2) + (col & 3);
}
// lane = row c, acc[j][v] = column 32 j + acc_row(v)
template <int D>
__device__ inline void put_rows(float* base, int w, int G, int c,
                                const f32x16_t (&acc)[Shape<D>::JB]) {
#pragma unroll
  for (int j = 0; j < Shape<D>::JB; ++j)
#pragma unroll
    for (int v = 0; v < 16; v += 4)
      *(float4*)part_at<D>(base, w, c, 32 * j + 8 * (v >> 2) + 4 * G) =
          make_float4(acc[j][v], acc[j][v + 1], acc[j][v + 2], acc[j][v + 3]);
}
// lane = column c, acc[j][v] = row acc_row(v)
template <int D>
__device__ inline void put_cols(float* base, int w, int G, int c,
                                const f32x16_t (&acc)[Shape<D>::JB]) {
#pragma unroll
  for (int j = 0; j < Shape<D>::JB; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) *part_at<D>(base, w, acc_row(v, G), 32 * j + c) = acc[j][v];
}

// ------------------------------------------------------------------ forward

template <int D, typename T>
__global__ __launch_bounds__(64 * Shape<D>::NW) void attn_fwd_f32_kernel(AttnArgs a0) {
  constexpr int NW = Shape<D>::NW, JB = Shape<D>::JB, NTH = 64 * NW;
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ float ms[NW][32], ls[NW][32];
  const AttnArgs a = attn_seq_view<T>(a0);
  const int h = blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int G = lane >> 5, c = lane & 31;
  const long H = a.ld;  // row stride
  const int q_lo = a.l + blockIdx.x * 32, t = q_lo + c, kend = min(a.r, q_lo + 32);
  const T* K = (const T*)a.kc + h * D;
  const T* V = (const T*)a.vc + h * D;
  float qf[D / 2];
  row_frag<D>((const T*)a.q + (long)(min(t, a.r - 1) - a.l) * H + h * D, G, qf);
  const float sl2 = a.scale * LOG2E;
  float m = -INFINITY, lsum = 0.f;  // running maximum (log2 units) and sum of weights
  f32x16_t o[JB];
#pragma unroll
  for (int j = 0; j < JB; ++j) o[j] = zero16();
  for (int k0 = 32 * w; k0 < kend; k0 += 32 * NW) {
    const int rows = min(32, kend - k0);
    float kf[D / 2];
    row_frag<D>(K + (long)(k0 + min(c, rows - 1)) * H, G, kf);
    f32x16_t p = dot_tile<D>(kf, qf);  // p[v]: key k0 + acc_row(v), query t
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p[v] = k0 + acc_row(v, G) <= t ? p[v] * sl2 : -INFINITY;
      mx = fmaxf(mx, p[v]);
    }
    const float mnew = fmaxf(m, pair_max(mx));
    // no visible key yet for this query: nothing to scale, weights 0
    const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mnew);
    const float mo = mnew == -INFINITY ? 0.f : mnew;
    float rs = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p[v] = __builtin_amdgcn_exp2f(p[v] - mo);
      rs += p[v];
    }
    lsum = lsum * alpha + pair_sum(rs);
    m = mnew;
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[j][v] *= alpha;
    acc_cols<D, true>(V + (long)k0 * H, H, rows, p, G, c, o, k0 + 31 > q_lo,
                      [&](int row, int q) { return k0 + row <= q_lo + q; });
  }
  if (G == 0) ms[w][c] = m, ls[w][c] = lsum;
  put_rows<D>(sm, w, G, c, o);
  __syncthreads();
  // merge in wave order: M = max_w m_w, O = sum_w O_w 2^(m_w - M) / sum_w l_w 2^(m_w - M)
  for (int e = threadIdx.x; e < 32 * D; e += NTH) {
    const int row = e / D, col = e % D, tt = q_lo + row;
    if (tt >= a.r) continue;
    float M = -INFINITY, L = 0.f, acc = 0.f;
#pragma unroll
    for (int x = 0; x < NW; ++x) M = fmaxf(M, ms[x][row]);
#pragma unroll
    for (int x = 0; x < NW; ++x) {
      const float f = ms[x][row] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms[x][row] - M);
      L += ls[x][row] * f;
      acc += *part_at<D>(sm, x, row, col) * f;
    }
    st((T*)a.o + (long)(tt - a.l) * H + h * D + col, acc / L);
    if (col == 0) a.lse[(long)h * a.Lmax + tt] = (M + log2f(L)) * LN2;
  }
}

// --------------------------------------------------------------------- dQ

// Also leaves D = rowsum(dO * O) = sum over keys of P dP of its queries for the
// dK/dV kernel: from the fp32 O, or, where O was rounded to bf16, from a first
// pass over the keys.
template <int D, typename T>
__global__ __launch_bounds__(64 * Shape<D>::NW) void attn_dq_f32_kernel(AttnArgs a0) {
  constexpr int NW = Shape<D>::NW, JB = Shape<D>::JB, NTH = 64 * NW;
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ float ds_[NW][32];
  const AttnArgs a = attn_seq_view<T>(a0);
  const int h = blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int G = lane >> 5, c = lane & 31;
  const long H = a.ld;  // row stride
  const int q_lo = a.l + blockIdx.x * 32, t = q_lo + c, kend = min(a.r, q_lo + 32);
  const T* K = (const T*)a.kc + h * D;
  const T* V = (const T*)a.vc + h * D;
  const int tc = min(t, a.r - 1);
  const long qoff = (long)(tc - a.l) * H + h * D;
  float qf[D / 2], of[D / 2];
  row_frag<D>((const T*)a.q + qoff, G, qf);
  row_frag<D>((const T*)a.dout + qoff, G, of);
  const float sl2 = a.scale * LOG2E, lse2 = a.lse[(long)h * a.Lmax + tc] * LOG2E;
  // P and dP of keys [k0, k0 + 32): element v is key k0 + acc_row(v)
  auto scores = [&](int k0, int rows, f32x16_t& p, f32x16_t& dp) {
    const long off = (long)(k0 + min(c, rows - 1)) * H;
    float kf[D / 2], vf[D / 2];
    row_frag<D>(K + off, G, kf);
    row_frag<D>(V + off, G, vf);
    p = dot_tile<D>(kf, qf);
    dp = dot_tile<D>(vf, of);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const bool ok = k0 + acc_row(v, G) <= t;
      p[v] = ok ? __builtin_amdgcn_exp2f(__builtin_fmaf(p[v], sl2, -lse2)) : 0.f;
      dp[v] = ok ? dp[v] : 0.f;  // a later token's value may be infinite or NaN
    }
  };
  float Dt = 0.f;
  if constexpr (sizeof(T) == 4) {
    float o[D / 2];
    row_frag<D>((const T*)a.o + qoff, G, o);
#pragma unroll
    for (int i = 0; i < D / 2; ++i) Dt += of[i] * o[i];
    Dt = pair_sum(Dt);
  } else {
    for (int k0 = 32 * w; k0 < kend; k0 += 32 * NW) {
      f32x16_t p, dp;
      scores(k0, min(32, kend - k0), p, dp);
#pragma unroll
      for (int v = 0; v < 16; ++v) Dt += p[v] * dp[v];
    }
    Dt = pair_sum(Dt);
    if (G == 0) ds_[w][c] = Dt;
    __syncthreads();
    Dt = 0.f;
#pragma unroll
    for (int x = 0; x < NW; ++x) Dt += ds_[x][c];
  }
  if (w == 0 && G == 0 && t < a.r) a.D[(long)h * a.Lmax + t] = Dt;
  f32x16_t dq[JB];
#pragma unroll
  for (int j = 0; j < JB; ++j) dq[j] = zero16();
  for (int k0 = 32 * w; k0 < kend; k0 += 32 * NW) {
    const int rows = min(32, kend - k0);
    f32x16_t p, dp;
    scores(k0, rows, p, dp);
#pragma unroll
    for (int v = 0; v < 16; ++v) p[v] *= dp[v] - Dt;
    acc_cols<D, true>(K + (long)k0 * H, H, rows, p, G, c, dq, k0 + 31 > q_lo,
                      [&](int row, int q) { return k0 + row <= q_lo + q; });
  }
  put_rows<D>(sm, w, G, c, dq);
  __syncthreads();
  for (int e = threadIdx.x; e < 32 * D; e += NTH) {
    const int row = e / D, col = e % D, tt = q_lo + row;
    if (tt >= a.r) continue;
    float acc = 0.f;
#pragma unroll
    for (int x = 0; x < NW; ++x) acc += *part_at<D>(sm, x, row, col);
    st((T*)a.dq + (long)(tt - a.l) * a.ld_dq + h * D + col, acc * a.scale);
  }
}

// ------------------------------------------------------------------ dK, dV

template <int D, typename T>
__global__ __launch_bounds__(64 * Shape<D>::NW) void attn_dkdv_f32_kernel(AttnArgs a0) {
  constexpr int NW = Shape<D>::NW, JB = Shape<D>::JB, NTH = 64 * NW;
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const AttnArgs a = attn_seq_view<T>(a0);
  const int h = blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int G = lane >> 5, c = lane & 31;
  const long H = a.ld;  // row stride
  const int k_lo = blockIdx.x * 32, key = k_lo + c, n = a.r - a.l;
  const T* Q = (const T*)a.q + h * D;
  const T* dO = (const T*)a.dout + h * D;
  const long koff = (long)min(key, a.r - 1) * H + h * D;
  float kf[D / 2], vf[D / 2];
  row_frag<D>((const T*)a.kc + koff, G, kf);
  row_frag<D>((const T*)a.vc + koff, G, vf);
  const float sl2 = a.scale * LOG2E;
  const float* lse = a.lse + (long)h * a.Lmax + a.l;
  const float* Dr = a.D + (long)h * a.Lmax + a.l;
  f32x16_t dk[JB], dv[JB];
#pragma unroll
  for (int j = 0; j < JB; ++j) dk[j] = dv[j] = zero16();
  // query rows i = t - l from the first that sees a key of this block
  for (int i0 = max(0, k_lo - a.l) + 32 * w; i0 < n; i0 += 32 * NW) {
    const int rows = min(32, n - i0);
    const long off = (long)(i0 + min(c, rows - 1)) * H;
    float lq[16], dr[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = i0 + min(acc_row(v, G), rows - 1);
      lq[v] = lse[i] * LOG2E;
      dr[v] = Dr[i];
    }
    f32x16_t p, ds;
    {
      float x[D / 2];
      row_frag<D>(Q + off, G, x);
      p = dot_tile<D>(x, kf);  // p[v]: query i0 + acc_row(v), key `key`
    }
    {
      float x[D / 2];
      row_frag<D>(dO + off, G, x);
      ds = dot_tile<D>(x, vf);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int i = acc_row(v, G);
      const bool ok = i < rows && key <= a.l + i0 + i;
      p[v] = ok ? __builtin_amdgcn_exp2f(__builtin_fmaf(p[v], sl2, -lq[v])) : 0.f;
      ds[v] = ok ? p[v] * (ds[v] - dr[v]) : 0.f;
    }
    const bool part = k_lo + 31 > a.l + i0 || rows < 32;
    auto sees = [&](int row, int k) { return k_lo + k <= a.l + i0 + row; };
    acc_cols<D, false>(dO + (long)i0 * H, H, rows, p, G, c, dv, part, sees);
    acc_cols<D, false>(Q + (long)i0 * H, H, rows, ds, G, c, dk, part, sees);
  }
  // dk[j][v], dv[j][v]: key k_lo + acc_row(v), column 32 j + c; each element of the
  // fp32 buffers (or, once final, of the dqkv rows) belongs to one thread
  auto add = [&](const f32x16_t(&acc)[JB], float* buf, float mul, int third) {
    put_cols<D>(sm, w, G, c, acc);
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * D; e += NTH) {
      const int row = e / D, col = e % D, s = k_lo + row;
      if (s >= a.r) continue;
      float x = 0.f;
#pragma unroll
      for (int z = 0; z < NW; ++z) x += *part_at<D>(sm, z, row, col);
      x *= mul;
      float* dst = buf + (long)s * H + h * D + col;
      if (s < a.dkv_init) x += *dst;
      if (s >= a.pack_l)
        st((T*)a.pack + (long)(s - a.pack_l) * a.ld_dq + third * a.H + h * D + col, x);
      else
        *dst = x;
    }
    __syncthreads();
  };
  add(dk, a.dk, a.scale, 1);
  add(dv, a.dv, 1.f, 2);
}

template <typename K>
hipError_t set_lds(K* fn, size_t bytes) {
  if (bytes < 60 * 1024) return hipSuccess;  // with the static part, within the default 64 KB
  return hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

template <int D, typename T>
hipError_t fwd_t(const AttnArgs& a, hipStream_t s) {
  constexpr size_t lds = Shape<D>::part;
  hipError_t e = set_lds(attn_fwd_f32_kernel<D, T>, lds);
  if (e != hipSuccess) return e;
  attn_fwd_f32_kernel<D, T>
      <<<dim3(cdiv(a.r - a.l, 32), a.heads, a.bs), 64 * Shape<D>::NW, lds, s>>>(a);
  return hipGetLastError();
}

template <int D, typename T>
hipError_t bwd_t(const AttnArgs& a, hipStream_t s) {
  constexpr size_t lds = Shape<D>::part;
  constexpr int NTH = 64 * Shape<D>::NW;
  hipError_t e = set_lds(attn_dq_f32_kernel<D, T>, lds);
  if (e == hipSuccess) e = set_lds(attn_dkdv_f32_kernel<D, T>, lds);
  if (e != hipSuccess) return e;
  attn_dq_f32_kernel<D, T><<<dim3(cdiv(a.r - a.l, 32), a.heads, a.bs), NTH, lds, s>>>(a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  attn_dkdv_f32_kernel<D, T><<<dim3(cdiv(a.r, 32), a.heads, a.bs), NTH, lds, s>>>(a);
  return hipGetLastError();
}

template <typename T>
hipError_t pick(const AttnArgs& a, bool bwd, hipStream_t s) {
  if (a.need) return hipSuccess;  // no scratch
  switch (a.d) {
    case 16: return bwd ? bwd_t<16, T>(a, s) : fwd_t<16, T>(a, s);
    case 32: return bwd ? bwd_t<32, T>(a, s) : fwd_t<32, T>(a, s);
    case 64:
      if constexpr (sizeof(T) == 4) return bwd ? bwd_t<64, T>(a, s) : fwd_t<64, T>(a, s);
      break;
    case 128:
      if constexpr (sizeof(T) == 4) return bwd ? bwd_t<128, T>(a, s) : fwd_t<128, T>(a, s);
      break;
  }
  return hipErrorNotSupported;
}

}  // namespace

// Every attention operand lies in the stage's workspace: rows are multiples of 16
// elements from 256-byte-aligned arenas, so the 4-element loads are aligned.
hipError_t attn_fwd_f32(int dtype, const AttnArgs& a, hipStream_t s) {
  return dtype == DT_FP32 ? pick<float>(a, false, s) : pick<bf16>(a, false, s);
}
hipError_t attn_bwd_f32(int dtype, const AttnArgs& a, hipStream_t s) {
  return dtype == DT_FP32 ? pick<float>(a, true, s) : pick<bf16>(a, true, s);
}

}  // namespace tp
