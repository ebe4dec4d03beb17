// bf16 (and fp16) GEMM of aligned operands, any number of rows, a last k-tile that need
// not be whole: global -> LDS by the CDNA4 LDS DMA (global_load_lds_dwordx4, 16
// bytes per lane straight into LDS), a ring of STAGES k-tiles in flight, and
// matrix-core reads straight from LDS:
//  - k-contiguous operand tiles ([row][64 k], 128-byte rows) are read with
//    ds_read_b128 (8 consecutive k for one row);
//  - operands contiguous along m/n stay in their global orientation in LDS
//    ([64 k][R], k-major) and are read with two ds_read_b64_tr_b16, the
//    transposing LDS read: within each 16-lane group, lane j addresses 4
//    consecutive columns of row k0 + j/4, and lane i receives column i of the
//    group's 16 columns at the 4 rows -- exactly 4 reduction values of one
//    MFMA row/column.
// Both layouts permute 16-byte chunks by an XOR of the row so that the DMA
// writes stay contiguous and the fragment reads avoid bank conflicts; the
// DMA lane order implements the permutation (each lane picks the global chunk
// that belongs at its LDS slot).
//
// LDS reads are issued as inline assembly with explicit lgkmcnt waits, and the
// DMA completion with explicit vmcnt waits before each barrier, so the
// compiler's conservative wait-for-all-DMA before LDS reads does not serialise
// the pipeline.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "tp_common.hpp"
#include "tp_epilogue.hpp"
#include "tp_kernels.hpp"

namespace tp {

hipError_t gemm_splitk_reduce(const GemmArgs& a, hipStream_t s);

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ inline uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// k-contiguous tile of BK k per row: row r, 16-byte chunk c (k = 8c..8c+7) at
// r*2BK + 16*(c ^ swz_kc(r)).  Any 16 consecutive rows read at one chunk land
// on 16 distinct 16-byte bank groups.
template <int BK>
__device__ inline int swz_kc(int r) {
  if constexpr (BK == 64) return (r ^ (r >> 3)) & 7;
  else return (r >> 2) & 3;
}
// m/n-contiguous tile of R columns: k-row k, 16-byte chunk c at k*2R + 16*(c ^ swz_mc<R>(k)).
// A transposing read takes 32 bytes from each of 4 consecutive k-rows.  Rows of
// 256 or 512 bytes all start on bank 0, so the row's chunk index is XORed with
// 4 (k mod 4) (64-byte steps); rows of 384 bytes (R = 192) already alternate
// between bank 0 and bank 32, so XOR 4 on rows 2 and 3 of each 4 suffices and
// keeps the 24 chunks of a row within range.
// Rows of 128 bytes (R = 64) alternate between bank 0 and bank 32 too and take the
// same XOR.
template <int R>
__device__ inline int swz_mc(int k) {
  static_assert(R % 128 == 0 || R == 192 || R == 64, "no transposing-read swizzle");
  if constexpr (R == 192 || R == 64) return ((k >> 1) & 1) << 2;
  else return (k & 3) << 2;
}

typedef float f32x4v __attribute__((ext_vector_type(4)));

__device__ inline void dma16(const uint16_t* g, uint16_t* lds_wave_base) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)lds_wave_base, 16, 0,
                                   0);
}

// DMA of one R x BK operand tile into LDS.  KC: X(r, k) = X[r * ld + k];
// MC: X(r, k) = X[k * ld + r].  Rows/columns past rmax are clamped to valid
// memory (their products are never stored); issue takes whole k-tiles, issue_tail and
// zero_tail a last one that is not.  The per-lane part of every chunk address is a
// byte offset from the k-origin of the tile, computed once per output tile;
// each k-tile only moves the wave-uniform origin (X + k for KC, X + k * ld for
// MC), so the loads take the scalar-base + 32-bit vector-offset form.  The
// caller guarantees the offsets fit in 32 bits.
template <int R, int BK, int NTH, bool KC>
struct DmaPlan {
  static constexpr int CH = R * BK / 8 / NTH;  // 16-byte chunks per thread
  uint32_t off[CH];
  __device__ DmaPlan(long ld, int r0, int rmax, int w, int lane) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int s = i * NTH + w * 64 + lane;  // LDS slot of this lane
      if constexpr (KC) {
        constexpr int CPR = BK / 8;  // chunks per row
        const int row = s / CPR, phys = s % CPR;
        const int logical = phys ^ swz_kc<BK>(row);
        const int gr = min(r0 + row, rmax - 1);
        off[i] = (uint32_t)(((long)gr * ld + logical * 8) * 2);
      } else {
        constexpr int CPR = R / 8;  // chunks per k-row
        const int krow = s / CPR, phys = s % CPR;
        const int logical = phys ^ swz_mc<R>(krow);
        const int gc = min(r0 + logical * 8, rmax - 8);
        off[i] = (uint32_t)(((long)krow * ld + gc) * 2);
      }
    }
  }
  // The last k-tile of a reduction that is not whole k-tiles (kvalid < BK values,
  // a multiple of 8 for KC): chunks past it repeat the last valid one, so every
  // address stays inside the operand; zero_tail clears them once they landed.
  __device__ static void issue_tail(const uint16_t* origin, long ld, int r0, int rmax, int kvalid,
                                    uint16_t* lds, int w, int lane) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int s = i * NTH + w * 64 + lane;
      long o;
      if constexpr (KC) {
        constexpr int CPR = BK / 8;
        const int row = s / CPR, logical = (s % CPR) ^ swz_kc<BK>(row);
        o = (long)min(r0 + row, rmax - 1) * ld + min(logical * 8, kvalid - 8);
      } else {
        constexpr int CPR = R / 8;
        const int krow = s / CPR, logical = (s % CPR) ^ swz_mc<R>(krow);
        o = (long)min(krow, kvalid - 1) * ld + min(r0 + logical * 8, rmax - 8);
      }
      dma16(origin + o, lds + (i * NTH + w * 64) * 8);
    }
  }
  __device__ static void zero_tail(int kvalid, uint16_t* lds) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int s = i * NTH + threadIdx.x;
      const int k = KC ? ((s % (BK / 8)) ^ swz_kc<BK>(s / (BK / 8))) * 8 : s / (R / 8);
      if (k >= kvalid) *(uint4*)(lds + s * 8) = make_uint4(0, 0, 0, 0);
    }
  }
  // origin: X + k0 (KC) or X + k0 * ld (MC), wave-uniform; w: wave index (uniform)
  __device__ void issue(const uint16_t* origin, uint16_t* lds, int w) const {
#pragma unroll
    for (int i = 0; i < CH; ++i)
      dma16((const uint16_t*)((const char*)origin + off[i]), lds + (i * NTH + w * 64) * 8);
  }
};

__device__ inline u32x4 ds_read128(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr));
  return v;
}
__device__ inline u32x2 ds_read_tr(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(v) : "v"(addr));
  return v;
}

// Fragment (8 reduction values at k0 + 8 G) of operand row/column `rc` for lane
// (G = lane / 32).  KC tiles: one 16-byte read; MC tiles: two transposing reads.
template <int R, int BK, bool KC>
__device__ inline u32x4 frag_read(uint32_t tile, int rc_base, int k0, int lane) {
  if constexpr (KC) {
    const int row = rc_base + (lane & 31), c = (k0 >> 3) + (lane >> 5);
    return ds_read128(tile + row * (2 * BK) + ((c ^ swz_kc<BK>(row)) << 4));
  } else {
    const int g = lane >> 4, j = lane & 15;
    const int col = rc_base + 16 * (g & 1) + 4 * (j & 3);
    const int kr0 = k0 + 8 * (g >> 1) + (j >> 2);
    u32x2 lo, hi;
    {
      const int kr = kr0;
      lo = ds_read_tr(tile + kr * (2 * R) + (((col >> 3) ^ swz_mc<R>(kr)) << 4) + ((col & 7) << 1));
    }
    {
      const int kr = kr0 + 4;
      hi = ds_read_tr(tile + kr * (2 * R) + (((col >> 3) ^ swz_mc<R>(kr)) << 4) + ((col & 7) << 1));
    }
    u32x4 r;
    r.x = lo.x;
    r.y = lo.y;
    r.z = hi.x;
    r.w = hi.y;
    return r;
  }
}

template <int N>
__device__ inline void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Wait until at most `pending` k-tiles (LPT DMA instructions each) are in flight.
template <int LPT, int MAXP>
__device__ inline void wait_tiles(int pending) {
  if constexpr (MAXP >= 1) {
    if (pending >= MAXP) {
      wait_vm<LPT * MAXP>();
      return;
    }
    wait_tiles<LPT, MAXP - 1>(pending);
  } else {
    wait_vm<0>();
  }
}

// XCD-aware output-tile order for launches of many tiles.  Workgroups are
// dispatched round-robin over the 8 XCDs (workgroup g runs on XCD g % 8) and
// each CU holds one workgroup, so the j-th workgroup of an XCD belongs to
// "round" j / 32 of that XCD's 32 CUs.  The 32 workgroups of one XCD and
// round cover a 4 x 8 super-tile of output tiles, so each k-slice of its 4
// A-panels and 8 B-panels is fetched into that XCD's L2 once while they run
// side by side.  Super-tile s of round r is r * 8 + xcd.
constexpr int WALK_PER_XCD = 32;

struct TileWalk {
  static constexpr int SM = 4, SN = 8;
  int tm, tn, stm, stn, sm, sn;
  // a super-tile is 4 x 8 tiles, or 8 x 4 where `turn` is set
  __host__ __device__ TileWalk(int tiles_m, int tiles_n, bool turn = false)
      : tm(tiles_m), tn(tiles_n), sm(turn ? SN : SM), sn(turn ? SM : SN) {
    stm = (tm + sm - 1) / sm, stn = (tn + sn - 1) / sn;
  }
  __host__ __device__ int supers() const { return stm * stn; }
  // output tile of slot `slot` of super-tile s; -1 if that slot is idle
  __device__ int tile_of(int s, int slot) const {
    if (s >= supers()) return -1;
    const int im = (s / stn) * sm + slot / sn, in = (s % stn) * sn + slot % sn;
    if (im >= tm || in >= tn) return -1;
    return im * tn + in;
  }
  // output tile of workgroup (xcd, slot) in round r
  __device__ int tile(int r, int xcd, int slot) const { return tile_of(r * 8 + xcd, slot); }
};

// Up to four weight-gradient products over the same tokens in one launch: the
// products of a layer differ in width, and each alone leaves a part-empty last round
// of workgroups (or, when narrow, most CUs idle).  first[p]: the first workgroup of
// product p in grid order, or its first super-tile (walk).
struct GemmGroup {
  GemmArgs g[4];
  int first[5];
  int count, walk;
};
// the product of this workgroup (uniform) and its index within it
__device__ inline const GemmArgs& my_product(const GemmArgs& a, int, int*) { return a; }
__device__ inline const GemmArgs& my_product(const GemmGroup& a, int i, int* local) {
  int p = 0;
  while (p + 1 < a.count && i >= a.first[p + 1]) ++p;
  *local = i - a.first[p];
  return a.g[p];
}

// STAGES k-tiles of A and SB of B are buffered.  SB == STAGES: one ring of
// (A, B) stages.  SB == STAGES + 1 == 3 ("B leads"): separate rings, the B
// operand (the weights of a slice-shaped product, streamed from HBM) one
// k-tile further ahead than A (activations, L2-resident).
// F16: both operands are fp16 (the mixed-precision query/key/value product),
// otherwise bf16.  TAIL: K need not be whole k-tiles; the values of the last tile
// past K are zeroed in LDS, in both operands, between two barriers.
// WGK: wave groups over the reduction: group wk of WGK takes its 1/WGK of every
// k-tile's 16-value steps, and the groups' accumulators are added in LDS before the
// epilogue.
// KEEP: fp32 outputs stay in the caches (GemmArgs::keep); an instance of its own, as both
// kinds of store in one epilogue cost the wide gradients 1 % (12288 wide, deferred, 2
// slices: 7235 -> 7319 us).
template <int BM, int BN, int BK, int WGM, int WGN, int WGK, bool A_KC, bool B_KC, int EPI,
          bool SPLIT, int STAGES, int SB, bool F16, bool TAIL, typename ARGS, bool KEEP = false>
__global__ __launch_bounds__(64 * WGM * WGN * WGK) void gemm_dma_kernel(ARGS args) {
  constexpr bool GROUP = std::is_same<ARGS, GemmGroup>::value;
  constexpr int NTH = 64 * WGM * WGN * WGK;
  constexpr int KSP = BK / 16 / WGK;  // 16-value steps of a wave per k-tile
  constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 32, FN = WN / 32;
  constexpr int TILE_A = BM * BK, TILE_B = BN * BK, STAGE = TILE_A + TILE_B;  // elements
  constexpr int LPT = BK * (BM + BN) / 8 / NTH;  // DMA instructions per thread per k-tile
  static_assert(FM >= 1 && FN >= 1, "wave tile below 32 x 32");
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile not a multiple of 32 x 32");
  static_assert((BK * BM / 8) % NTH == 0 && (BK * BN / 8) % NTH == 0, "uneven DMA split");
  static_assert(LPT * (STAGES - 2) <= 63, "vmcnt range");
  constexpr bool BLEAD = SB > STAGES;
  static_assert(SB == STAGES || (STAGES == 2 && SB == 3), "unsupported ring shape");
  static_assert(KSP % 2 == 0, "fragment buffers alternate per k-step across k-tiles");
  static_assert(WGK == 1 || WGK == 2, "one or two wave groups over the reduction");
  constexpr int LPT_B = BK * BN / 8 / NTH;
  // the epilogue's wave patches take the ring stage no wave reads in the last
  // k-tile; with separate rings, or where they are larger than a stage, the LDS
  // base once every wave has left the loop
  constexpr int PATCH = WGM * WGN * WGK * 32 * 36 * 2;  // elements
  constexpr bool PATCH_AT_BASE = BLEAD || WGK > 1 || PATCH > STAGE;
  static_assert(PATCH <= (BLEAD && WGK == 1 ? STAGES * TILE_A : STAGES * STAGE), "epilogue patch exceeds LDS");
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

  int local = 0;  // GROUP: tile or super-tile within this workgroup's product
  int gi = blockIdx.x;
  if constexpr (GROUP) {
    if (args.walk) {
      gi = (blockIdx.x / 8 / WALK_PER_XCD) * 8 + blockIdx.x % 8;
      if (gi >= args.first[args.count]) return;  // uniform per workgroup
    }
  }
  const GemmArgs& a = my_product(args, gi, &local);
  const uint16_t* A = (const uint16_t*)a.A;
  const uint16_t* B = (const uint16_t*)a.B;
  const long lda = A_KC ? a.sam : a.sak;
  const long ldb = B_KC ? a.sbn : a.sbk;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wk = WGK > 1 ? wave / (WGM * WGN) : 0;  // wave group over the reduction
  const int wmn = WGK > 1 ? wave % (WGM * WGN) : wave, kofs = wk * KSP * 16;
  const int wm0 = (wmn / WGN) * WM, wn0 = (wmn % WGN) * WN;
  const int kbeg = SPLIT ? blockIdx.z * a.k_split : 0;
  const int kend = SPLIT ? min(a.K, kbeg + a.k_split) : a.K;
  const int nk = TAIL ? (kend - kbeg + BK - 1) / BK : (kend - kbeg) / BK;
  const int kvalid = kend - kbeg - (nk - 1) * BK;  // TAIL: values of the last k-tile
  const uint32_t sbase = lds_addr(smem);

  int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  if constexpr (GROUP) {
    const TileWalk walk(cdiv(a.M, BM), cdiv(a.N, BN), a.walk == 2);
    const int tile =
        args.walk ? walk.tile_of(local, blockIdx.x / 8 % WALK_PER_XCD) : local;
    if (tile < 0) return;  // uniform per workgroup
    m0 = (tile / walk.tn) * BM;
    n0 = (tile % walk.tn) * BN;
  } else if (!SPLIT && a.walk) {
    const TileWalk walk(cdiv(a.M, BM), cdiv(a.N, BN));
    const int j = blockIdx.x / 8;
    const int tile = walk.tile(j / WALK_PER_XCD, blockIdx.x % 8, j % WALK_PER_XCD);
    if (tile < 0) return;  // uniform per workgroup
    m0 = (tile / walk.tn) * BM;
    n0 = (tile % walk.tn) * BN;
  }

  const int wu = __builtin_amdgcn_readfirstlane(wave);
  const DmaPlan<BM, BK, NTH, A_KC> plan_a(lda, m0, a.M, wu, lane);
  const DmaPlan<BN, BK, NTH, B_KC> plan_b(ldb, n0, a.N, wu, lane);
  auto issue_a = [&](int kt) {
    uint16_t* st = smem + (kt % STAGES) * (BLEAD ? TILE_A : STAGE);
    const long k = kbeg + kt * BK;
    if (TAIL && kt == nk - 1 && kvalid < BK)
      plan_a.issue_tail(A + (A_KC ? k : k * lda), lda, m0, a.M, kvalid, st, wu, lane);
    else
      plan_a.issue(A + (A_KC ? k : k * lda), st, wu);
  };
  auto issue_b = [&](int kt) {
    uint16_t* st = BLEAD ? smem + STAGES * TILE_A + (kt % SB) * TILE_B
                         : smem + (kt % STAGES) * STAGE + TILE_A;
    const long k = kbeg + kt * BK;
    if (TAIL && kt == nk - 1 && kvalid < BK)
      plan_b.issue_tail(B + (B_KC ? k : k * ldb), ldb, n0, a.N, kvalid, st, wu, lane);
    else
      plan_b.issue(B + (B_KC ? k : k * ldb), st, wu);
  };
  // DMA of the k-tiles that iteration kt brings in (their stages were last read
  // in iteration kt - 1, before its closing barrier)
  auto issue_next = [&](int kt) {
    if constexpr (BLEAD) {
      if (kt + 1 < nk) issue_a(kt + 1);
      if (kt + 2 < nk) issue_b(kt + 2);
    } else if (kt + STAGES - 1 < nk) {
      issue_a(kt + STAGES - 1);
      issue_b(kt + STAGES - 1);
    }
  };

  f32x16_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  if constexpr (BLEAD) {
    // issue order B0, A0, B1, then per iteration A(kt+1), B(kt+2): when
    // iteration kt starts, only B(kt+1) was issued after A(kt)
    issue_b(0);
    issue_a(0);
    if (nk > 1) issue_b(1);
  } else {
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
      if (s < nk) {
        issue_a(s);
        issue_b(s);
      }
  }

  // k-tile j has landed for every wave once at most the DMAs issued after it
  // are in flight (they complete in issue order) and the workgroup has met at
  // a barrier
  auto wait_tile = [&](int j) {
    if constexpr (BLEAD) {
      if (j + 1 < nk) wait_vm<LPT_B>();
      else wait_vm<0>();
    } else {
      wait_tiles<LPT, STAGES - 2>(min(STAGES - 2, nk - 1 - j));
    }
    __builtin_amdgcn_s_barrier();
    if constexpr (TAIL) {
      static_assert(!BLEAD, "the tail is cleared in single-ring kernels only");
      if (j == nk - 1 && kvalid < BK) {
        uint16_t* st = smem + (j % STAGES) * STAGE;
        plan_a.zero_tail(kvalid, st);
        plan_b.zero_tail(kvalid, st + TILE_A);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
      }
    }
  };
  auto tile_a = [&](int j) { return sbase + (j % STAGES) * (BLEAD ? TILE_A : STAGE) * 2; };
  auto tile_b = [&](int j) {
    return BLEAD ? sbase + (STAGES * TILE_A + (j % SB) * TILE_B) * 2 : tile_a(j) + TILE_A * 2;
  };
  u32x4 fa[2][FM], fb[2][FN];
  auto read_frags = [&](int buf, int j, int k0) {
    const uint32_t ta = tile_a(j), tb = tile_b(j);
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[buf][i] = frag_read<BM, BK, A_KC>(ta, wm0 + 32 * i, k0, lane);
#pragma unroll
    for (int jj = 0; jj < FN; ++jj) fb[buf][jj] = frag_read<BN, BK, B_KC>(tb, wn0 + 32 * jj, k0, lane);
  };
  // wait for every LDS read issued so far, every fragment register of `buf` tied to the wait
  auto frags_ready = [&](int buf) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fa[buf][0]));
#pragma unroll
    for (int i = 1; i < FM; ++i) asm volatile("" : "+v"(fa[buf][i]));
#pragma unroll
    for (int jj = 0; jj < FN; ++jj) asm volatile("" : "+v"(fb[buf][jj]));
  };

  // One k-step runs the FM x FN matrix-core products of fragment buffer `cur`
  // and, one per product from the first product on, the fragment reads of the
  // next step into the other buffer, so the reads complete under the products
  // and the step ends with a single LDS wait.  Scheduling barriers pin that
  // order: the reads are inline assembly, which the scheduler would otherwise
  // let the products pass, leaving a wait in front of most of them.
  //
  // The k-tile boundary is software-pipelined: half of the last step's
  // products go out, then the wait and barrier for tile kt+1, then its first
  // fragment reads interleaved with the other half.  The DMA of the tile after
  // goes out right after the barrier for split (slice-shaped, weight-streaming)
  // products, after the last step's products for the others; either way into
  // the stage of tile kt, which every wave finished reading before the barrier.
  // The final k-tile is peeled (no next tile to wait for or read), so no
  // branch inside the loop holds products.
  constexpr int NR = FM + FN, NM = FM * FN;
  auto mfma_at = [&](int buf, int t) {
    const int i = t / FN, j = t % FN;
    if constexpr (F16)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
          __builtin_bit_cast(f16x8_t, fa[buf][i]), __builtin_bit_cast(f16x8_t, fb[buf][j]),
          acc[i][j], 0, 0, 0);
    else
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          __builtin_bit_cast(bf16x8_t, fa[buf][i]), __builtin_bit_cast(bf16x8_t, fb[buf][j]),
          acc[i][j], 0, 0, 0);
  };
  auto read_at = [&](int buf, uint32_t ta, uint32_t tb, int k0, int r) {
    if (r < FM) fa[buf][r] = frag_read<BM, BK, A_KC>(ta, wm0 + 32 * r, k0, lane);
    else fb[buf][r - FM] = frag_read<BN, BK, B_KC>(tb, wn0 + 32 * (r - FM), k0, lane);
  };
  // products [T0, NM) of `cur`; with RD, the reads of `nxt` (tile j, k-offset
  // k0) one per product from T0 on, any left over after the last product
  auto interleave = [&](auto t0c, auto rdc, int cur, int nxt, int j, int k0) {
    constexpr int T0 = decltype(t0c)::value;
    constexpr bool RD = decltype(rdc)::value;
    const uint32_t ta = tile_a(j), tb = tile_b(j);
#pragma unroll
    for (int t = T0; t < NM; ++t) {
      if constexpr (RD) {
        if (t - T0 < NR) read_at(nxt, ta, tb, k0, t - T0);
      }
      mfma_at(cur, t);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (RD) {
#pragma unroll
      for (int r = NM - T0; r < NR; ++r) read_at(nxt, ta, tb, k0, r);
    }
  };
  using First = std::integral_constant<int, 0>;
  using Half = std::integral_constant<int, NM / 2>;
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;
  auto ktile = [&](int kt, auto finalc) {
    constexpr bool FINAL = decltype(finalc)::value;
#pragma unroll
    for (int ks = 0; ks < KSP; ++ks) {
      const int cur = ks & 1, nxt = cur ^ 1;
      const bool last = ks + 1 == KSP;
      if (!last) {
        interleave(First{}, Yes{}, cur, nxt, kt, kofs + 16 * (ks + 1));
      } else if constexpr (!FINAL) {
#pragma unroll
        for (int t = 0; t < NM / 2; ++t) mfma_at(cur, t);
        __builtin_amdgcn_sched_barrier(0);
        wait_tile(kt + 1);
        if (SPLIT) issue_next(kt + 1);
        interleave(Half{}, Yes{}, cur, nxt, kt + 1, kofs);
      } else {
        interleave(First{}, No{}, cur, nxt, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (!FINAL && !SPLIT && last) issue_next(kt + 1);
      if (!(FINAL && last)) frags_ready(nxt);
    }
  };

  wait_tile(0);
  issue_next(0);
  read_frags(0, 0, kofs);
  frags_ready(0);
  if (nk > 0) {
    for (int kt = 0; kt + 1 < nk; ++kt) ktile(kt, No{});
    ktile(nk - 1, Yes{});
  }
  // every outstanding DMA has been waited for: the last iteration waited for 0

  // Two wave groups: a sub-tile t of the wave tile belongs to group t % 2 (a single
  // one to group 0); each wave leaves its sums of the partner's sub-tiles in LDS and
  // adds the partner's to its own.
  constexpr int T = FM * FN;
  auto mine = [&](int t) { return WGK == 1 || (T == 1 ? wk == 0 : t % 2 == wk); };
  if constexpr (WGK > 1) {
    constexpr int HT = (T + 1) / 2;  // sub-tiles a wave gives away at most
    static_assert(WGM * WGN * WGK * HT * 4096 <= 2 * ((long)STAGES * TILE_A + (long)SB * TILE_B),
                  "exchange exceeds LDS");
    __builtin_amdgcn_s_barrier();  // every wave has read its last fragments
    float* ex = (float*)smem;
    const int partner = wave ^ (WGM * WGN);
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (!mine(t)) {
#pragma unroll
        for (int v = 0; v < 16; v += 4)
          *(float4*)(ex + ((wave * HT + t / 2) * 4 + v / 4) * 256 + lane * 4) =
              make_float4(acc[t / FN][t % FN][v], acc[t / FN][t % FN][v + 1],
                          acc[t / FN][t % FN][v + 2], acc[t / FN][t % FN][v + 3]);
      }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (mine(t)) {
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
          const float4 x =
              *(const float4*)(ex + ((partner * HT + t / 2) * 4 + v / 4) * 256 + lane * 4);
          f32x16_t& c = acc[t / FN][t % FN];
          c[v] += x.x, c[v + 1] += x.y, c[v + 2] += x.z, c[v + 3] += x.w;
        }
      }
    __syncthreads();
  }

  if constexpr (SPLIT || EPI == EPI_ACC_F32) {
    // fp32 outputs: each 32 x 32 sub-tile goes through a wave-private LDS patch
    if constexpr (PATCH_AT_BASE) __builtin_amdgcn_s_barrier();
    float* patch = (float*)(smem + (PATCH_AT_BASE ? 0 : (nk % STAGES) * STAGE)) + wave * (32 * 36);
    float* out = SPLIT ? a.ws + (long)blockIdx.z * a.M * a.N : (float*)a.C;
    const long ldo = SPLIT ? a.N : a.ldc;
    // sub-tile rows leave as whole 128-byte lines: in step q (0..3) lane l
    // takes row 8q + l/8, 16-byte chunk l%8
    const int er = lane >> 3, ec = (lane & 7) * 4;
    const bool full = m0 + wm0 + WM <= a.M && n0 + wn0 + WN <= a.N;
    auto dst_of = [&](int t, int q) {
      return out + (long)(m0 + wm0 + (t / FN) * 32 + 8 * q + er) * ldo + n0 + wn0 + (t % FN) * 32 +
             ec;
    };
    // fp32 +=: the destination values of the next P sub-tiles are in flight
    // while one is combined (a plain store with a.overwrite)
    constexpr int P = T < 4 ? T : 4;
    const bool add = !SPLIT && !a.overwrite;
    float4 pre[P][4];
    if (add && full) {
#pragma unroll
      for (int t = 0; t < P; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) pre[t][q] = *(const float4*)dst_of(t, q);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (!mine(t)) continue;
      const int i = t / FN, j = t % FN;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        patch[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 36 + (lane & 31)] = acc[i][j][v];
      float4 x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = *(const float4*)(patch + (8 * q + er) * 36 + ec);
      if (full) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (add) {
            const float4 o = pre[t % P][q];
            x[q].x += o.x, x[q].y += o.y, x[q].z += o.z, x[q].w += o.w;
          }
          if constexpr (SPLIT || KEEP) {
            *(float4*)dst_of(t, q) = x[q];
          } else {
            // a stored fp32 weight gradient is not read again by this sequence's
            // kernels, or not before the caches have moved on: a non-temporal store
            // keeps it from displacing their operands
            const f32x4v v = {x[q].x, x[q].y, x[q].z, x[q].w};
            __builtin_nontemporal_store(v, (f32x4v*)dst_of(t, q));
          }
        }
        if (add && t + P < T) {
#pragma unroll
          for (int q = 0; q < 4; ++q) pre[t % P][q] = *(const float4*)dst_of(t + P, q);
        }
      } else {
        const int n = n0 + wn0 + j * 32 + ec;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = m0 + wm0 + i * 32 + 8 * q + er;
          if (m < a.M) {
            float* dst = out + (long)m * ldo + n;
            const float xs[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (n + e < a.N) dst[e] = add ? dst[e] + xs[e] : xs[e];
          }
        }
      }
    }
  } else {
    // bf16 outputs: each 32 x 32 sub-tile goes through the LDS patch and leaves
    // as 8-column row segments (in step q of 2, lane l takes row 16q + l/4,
    // columns 8 (l%4) .. +7), one 16-byte access per operand; N % 8 == 0, so a
    // segment is either inside the output or past its edge
    if constexpr (PATCH_AT_BASE) __builtin_amdgcn_s_barrier();
    float* patch = (float*)(smem + (PATCH_AT_BASE ? 0 : (nk % STAGES) * STAGE)) + wave * (32 * 36);
    const int er = lane >> 2, ec = (lane & 3) * 8;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        if (!mine(i * FN + j)) continue;
#pragma unroll
        for (int v = 0; v < 16; ++v)
          patch[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 36 + (lane & 31)] = acc[i][j][v];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int r = 16 * q + er;
          const float4 u = *(const float4*)(patch + r * 36 + ec);
          const float4 w = *(const float4*)(patch + r * 36 + ec + 4);
          float x[8] = {u.x, u.y, u.z, u.w, w.x, w.y, w.z, w.w};
          const int m = m0 + wm0 + 32 * i + r, n = n0 + wn0 + 32 * j + ec;
          if (m < a.M && n < a.N) epi8<EPI>(a, m, n, x);
        }
      }
  }
}

// Raises a kernel's dynamic-LDS limit, once per kernel and device (bit d of a
// per-kernel mask; devices past 31 set it on every launch).
template <auto* FN>
hipError_t raise_lds(size_t lds) {
  static std::atomic<uint32_t> done{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = 32;
  const uint32_t bit = dev < 32 ? 1u << dev : 0u;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute((const void*)FN,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

template <int BM, int BN, int BK, int WGM, int WGN, int WGK, bool A_KC, bool B_KC, int STAGES,
          int SB, bool SPLIT, bool F16, bool TAIL>
hipError_t launch_dma(const GemmArgs& a, hipStream_t s) {
  constexpr int NTH = 64 * WGM * WGN * WGK;
  constexpr size_t lds = ((size_t)STAGES * BM + (size_t)SB * BN) * BK * 2;
  dim3 grid(cdiv(a.N, BN), cdiv(a.M, BM), SPLIT ? a.splits : 1);
  if (!SPLIT && a.walk) {
    // rounds of 8 super-tiles (one per XCD), 256 workgroups per round
    const int rounds =
        (cdiv(cdiv(a.M, BM), TileWalk::SM) * cdiv(cdiv(a.N, BN), TileWalk::SN) + 7) / 8;
    grid = dim3(rounds * 8 * WALK_PER_XCD, 1, 1);
  }
#define TP_LAUNCH(E)                                                                         \
  do {                                                                                       \
    constexpr auto* fn = &gemm_dma_kernel<BM, BN, BK, WGM, WGN, WGK, A_KC, B_KC, E, SPLIT,   \
                                          STAGES, SB, F16, TAIL, GemmArgs>;                  \
    const hipError_t e = raise_lds<fn>(lds);                                                 \
    if (e != hipSuccess) return e;                                                           \
    fn<<<grid, NTH, lds, s>>>(a);                                                            \
  } while (0)
  if constexpr (SPLIT) {
    TP_LAUNCH(EPI_STORE);
  } else if constexpr (F16) {
    // fp16 operands: only the query/key/value product
    if (a.epi != EPI_QKV) return hipErrorNotSupported;
    TP_LAUNCH(EPI_QKV);
  } else if constexpr (!A_KC && !B_KC) {
    // m/n-contiguous operands on both sides: the weight-gradient products
    if (a.epi != EPI_ACC_F32) return hipErrorNotSupported;
    TP_LAUNCH(EPI_ACC_F32);
  } else if constexpr (B_KC) {
    // the forward's products
    switch (a.epi) {
      case EPI_QKV: TP_LAUNCH(EPI_QKV); break;
      case EPI_RESID: TP_LAUNCH(EPI_RESID); break;
      case EPI_GELU: TP_LAUNCH(EPI_GELU); break;
      default: return hipErrorNotSupported;
    }
  } else {
    // the backward's products with a weight matrix
    switch (a.epi) {
      case EPI_STORE: TP_LAUNCH(EPI_STORE); break;
      case EPI_DGELU: TP_LAUNCH(EPI_DGELU); break;
      default: return hipErrorNotSupported;
    }
  }
#undef TP_LAUNCH
  return hipGetLastError();
}


// One DMA GEMM product with the given number of splits over the reduction (whole
// k-tiles, the last split may be shorter), 1 = no partial sums.  With splits2 > 0
// and 0 < cols1 < the column-tile count, the product runs as two split launches:
// column tiles [0, cols1) with `splits`, the rest with splits2, and one reduction
// over both.  The caller has checked that the partials fit the workspace.
template <int BM, int BN, int BK, int WGM, int WGN, int WGK, bool A_KC, bool B_KC, int STAGES,
          int SB, bool F16, bool TAIL>
hipError_t run_dma(GemmArgs a, hipStream_t s, int splits, int splits2, int cols1) {
  constexpr int CUS = 256;
  const long tiles = (long)cdiv(a.M, BM) * cdiv(a.N, BN);
  const int nkt = cdiv(a.K, BK);
  if (splits2 > 0 && cols1 > 0 && (long)cols1 * BN < a.N) {
    const int n1 = cols1 * BN, n2 = a.N - n1;
    const int ks1 = cdiv(nkt, splits) * BK, ks2 = cdiv(nkt, splits2) * BK;
    const int s1 = cdiv(a.K, ks1), s2 = cdiv(a.K, ks2);
    const long p1 = (long)s1 * a.M * n1;
    GemmArgs g = a;
    g.N = n1, g.k_split = ks1, g.splits = s1;
    hipError_t e = launch_dma<BM, BN, BK, WGM, WGN, WGK, A_KC, B_KC, STAGES, SB, true, F16, TAIL>(g, s);
    if (e != hipSuccess) return e;
    g = a;
    g.N = n2, g.k_split = ks2, g.splits = s2;
    g.B = (const uint16_t*)a.B + (long)n1 * a.sbn;
    g.ws = a.ws + p1, g.ws_elems = a.ws_elems - p1;
    e = launch_dma<BM, BN, BK, WGM, WGN, WGK, A_KC, B_KC, STAGES, SB, true, F16, TAIL>(g, s);
    if (e != hipSuccess) return e;
    GemmArgs r = a;
    r.splits = s1, r.splits2 = s2, r.split_cols = n1;
    return gemm_splitk_reduce(r, s);
  }
  if (splits > 1) {
    a.k_split = cdiv(nkt, splits) * BK;
    a.splits = cdiv(a.K, a.k_split);
    hipError_t e = launch_dma<BM, BN, BK, WGM, WGN, WGK, A_KC, B_KC, STAGES, SB, true, F16, TAIL>(a, s);
    if (e != hipSuccess) return e;
    return gemm_splitk_reduce(a, s);
  }
  // many tiles: XCD-aware super-tile order
  if (tiles >= 2 * CUS) a.walk = 1;
  return launch_dma<BM, BN, BK, WGM, WGN, WGK, A_KC, B_KC, STAGES, SB, false, F16, TAIL>(a, s);
}

// Tile configurations.  All hold 64-value k-tiles; wpc workgroups fit a CU's LDS.
enum TileCfg { T256x256, T256x192, T256x128, T128x128, T64x128, T64x64, T32x128, T_DW256 };

template <bool A_KC, bool B_KC, bool F16, bool TAIL>
hipError_t run_cfg(int cfg, const GemmArgs& a, hipStream_t s, int splits, int splits2, int cols1) {
  constexpr bool SLICE = A_KC;  // a slice's activations or gradients times a weight matrix
  if constexpr (!SLICE) {
    if (cfg == T128x128)
      return run_dma<128, 128, 64, 4, 2, 1, A_KC, B_KC, 4, 4, F16, TAIL>(a, s, splits, 0, 0);
    if (cfg == T64x64)
      return run_dma<64, 64, 64, 2, 2, 1, A_KC, B_KC, 3, 3, F16, TAIL>(a, s, splits, 0, 0);
    if (cfg == T_DW256)
      return run_dma<256, 256, 64, 2, 4, 1, A_KC, B_KC, 2, 2, F16, TAIL>(a, s, splits, 0, 0);
  } else {
    // Two wave groups over the reduction: a wave tile twice as large reads fewer
    // LDS bytes per product (64x128 tiles of eight waves: 48 instead of 64 KB a
    // k-tile), which with the DMA's writes bounds these tiles: 256 x 6144 x 2048 17.4 ->
    // 15.8 us, 256 x 2048 x 2048 13.2 -> 11.7 us (graph replays of one product; the first
    // takes 19 us among a stage's other kernels).
    switch (cfg) {
      case T128x128:
        return run_dma<128, 128, 64, 2, 2, 2, A_KC, B_KC, 4, 4, F16, TAIL>(a, s, splits, 0, 0);
      case T64x64:
        return run_dma<64, 64, 64, 2, 2, 2, A_KC, B_KC, 3, 3, F16, TAIL>(a, s, splits, 0, 0);
    }
  }
  if constexpr (SLICE && !TAIL) {
    switch (cfg) {
      case T256x256:
        return run_dma<256, 256, 64, 2, 4, 1, A_KC, B_KC, 2, 3, F16, false>(a, s, splits, splits2, cols1);
      // 256 tiles for a 256-row product of width 49152, 64 for 12288
      case T256x192:
        return run_dma<256, 192, 64, 4, 2, 1, A_KC, B_KC, 2, 3, F16, false>(a, s, splits, splits2, cols1);
      case T256x128:
        return run_dma<256, 128, 64, 4, 2, 1, A_KC, B_KC, 3, 3, F16, false>(a, s, splits, 0, 0);
      case T64x128:
        return run_dma<64, 128, 64, 2, 2, 2, A_KC, B_KC, 3, 3, F16, false>(a, s, splits, 0, 0);
      case T32x128: return run_dma<32, 128, 64, 1, 4, 1, A_KC, B_KC, 4, 4, F16, false>(a, s, splits, 0, 0);
    }
  }
  return hipErrorNotSupported;
}

// ------------------------------------------------------- tile shape and splits

constexpr int kSplits[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};

// Modelled main loop (us) of `wgs` workgroups of kt k-tiles each: a workgroup
// costs a + kt * c alone on its CU (c_cold where the weights come from HBM), and
// kt * c_more (plus a) for every further workgroup that shares the CU.
struct Cand {
  int cfg, bm, bn, wpc;
  double a, c, c_cold, c_more;
  double main_us(long wgs, int kt, bool cold) const {
    const long load = cdiv(wgs, 256), rounds = cdiv(wgs, 256l * wpc);
    return rounds * kt * (cold ? c_cold : c) + (load - rounds) * kt * c_more + load * a;
  }
};

struct TileChoice {
  int cfg, splits;
  int splits2 = 0, cols1 = 0;  // two column groups (see run_dma), 0: one launch
  long partials = 0;           // fp32 partial sums it takes at most
};

// The partial sums of the reference plan, which defines together with the plan that
// runs which slices tp_slice_forward_static admits: four tile shapes (128x128 ..
// 256x256; for row counts off the 8-row grid or a K off the 64-value grid, three
// workgroups a CU) with fixed costs.  No launch follows it; it keeps that call's
// answers the same when the tiles of choose_tiles change.  choose_tiles in turn takes
// no more than the larger of the array and this, so an admitted slice's own plan fits.
long reference_partials(const GemmArgs& a) {
  if (a.M % 8 || a.K % 64) {
    const int bm = a.M <= 64 ? 64 : a.M <= 128 ? 128 : a.M <= 256 ? 256 : 128;
    const long tiles = (long)cdiv(a.M, bm) * cdiv(a.N, 128);
    if (tiles >= 768 || !a.ws) return 0;
    int sp = (int)std::min<long>(8, cdiv(768, tiles));
    while (sp > 1 && (a.K / sp < 512 || (long)sp * a.M * a.N > a.ws_elems)) --sp;
    return sp > 1 ? (long)cdiv(a.K, cdiv(cdiv(a.K, sp), 64) * 64) * a.M * a.N : 0;
  }
  struct Ref {
    int bm, bn;
    double c_kt;
  };
  static const Ref kRefs[] = {{128, 128, 0.5931}, {256, 128, 0.9088}, {256, 192, 1.2088},
                              {256, 256, 1.4367}};
  const int nkt = a.K / 64;
  double best = 1e300;
  long pick = 0;
  for (const Ref& c : kRefs) {
    const long mt = cdiv(a.M, c.bm), tiles = mt * cdiv(a.N, c.bn);
    const double hbm = (double)mt * a.N * a.K * 2.0 / 1e6 * 0.1773;
    for (int sp : kSplits) {
      if (sp > nkt) break;
      if (sp > 1 && (!a.ws || (long)sp * a.M * a.N > a.ws_elems)) break;
      const int ks = cdiv(nkt, sp), s = cdiv(nkt, ks);
      double t = std::max(cdiv(tiles * s, 256) * (0.7377 + ks * c.c_kt), hbm);
      if (s > 1) t += 5.6764 + (double)s * a.M * a.N * 8.0 / 1e6 / 5.7874;
      if (t < best) best = t, pick = s > 1 ? (long)s * a.M * a.N : 0;
    }
  }
  const double single = best;
  for (const Ref& c : kRefs) {
    if (c.bn < 192) continue;
    const long mt = cdiv(a.M, c.bm), tn = cdiv(a.N, c.bn);
    for (int sp1 : kSplits) {
      if (sp1 > nkt) break;
      const int ks1 = cdiv(nkt, sp1), e1 = cdiv(nkt, ks1);
      for (long r1 = 1;; ++r1) {
        const long cols1 = r1 * 256 / (mt * e1);
        if (cols1 >= tn) break;
        if (cols1 * mt * e1 != r1 * 256) continue;
        const long n1 = cols1 * c.bn, n2 = a.N - n1;
        const double h1 = (double)mt * n1 * a.K * 2.0 / 1e6 * 0.1773;
        const double h2 = (double)mt * n2 * a.K * 2.0 / 1e6 * 0.1773;
        for (int sp2 : kSplits) {
          if (sp2 > nkt) break;
          const int ks2 = cdiv(nkt, sp2), e2 = cdiv(nkt, ks2);
          const double part = (double)e1 * a.M * n1 + (double)e2 * a.M * n2;
          if (!a.ws || part > (double)a.ws_elems) break;
          const double t = std::max(r1 * (0.7377 + ks1 * c.c_kt), h1) +
                           std::max(cdiv(mt * (tn - cols1) * e2, 256) * (0.7377 + ks2 * c.c_kt), h2) +
                           5.6764 + part * 8.0 / 1e6 / 5.7874;
          if (t < best && t < 0.97 * single) best = t, pick = (long)part;
        }
      }
    }
  }
  return pick;
}

// Tile shape and split count of a product whose A operand is k-contiguous (slice
// activations or output gradients times a weight matrix): the candidate with the
// smallest modelled time.  The model was fitted (log least squares, rms error 7 %)
// to a sweep of every candidate (graph replays, rotating weights) on the 8 products
// of a layer for widths 256-12288 and 8- and 4-way shards, 16-4096 rows; its pick
// is on average 1.1 % (at worst 32 %) over the best candidate of each product,
// where four shapes of 128x128 and up, one workgroup a CU, were 22 % over.
// What decides: a CU moves operands at 45-65 GB/s, more with two or three
// workgroups on it, so narrow products want small tiles that use every CU without
// partial sums (256 x 3072 x 1024: 14.5 -> 9 us, 256 x 8192 x 2048 with a GELU: 23 ->
// 17.5 us, replays as in the sweep; 22 us among a stage's other kernels), wide ones large
// tiles that move few bytes per flop.
//   t = 3.6 + |(main + GELU, stream)| + epilogue bytes + (split: 2.1 + 0.16 per
//   split + partials)
// with stream = the weights (once from HBM, again from the caches for every further
// row tile) and A (for every column tile).
TileChoice choose_tiles(const GemmArgs& a, bool tail) {
  static const Cand kCands[] = {{T32x128, 32, 128, 2, 0.281, 0.2644, 0.3440, 0.1016},
                                {T64x64, 64, 64, 3, 0.378, 0.2191, 0.3375, 0.0986},
                                {T64x128, 64, 128, 2, 0.730, 0.3103, 0.3947, 0.1583},
                                {T128x128, 128, 128, 1, 2.326, 0.4158, 0.4605, 0.0},
                                {T256x128, 256, 128, 1, 1.887, 0.8262, 0.8117, 0.0},
                                {T256x192, 256, 192, 1, 3.001, 1.1034, 1.1131, 0.0},
                                {T256x256, 256, 256, 1, 3.427, 1.3320, 1.3828, 0.0}};
  const int nkt = cdiv(a.K, 64);
  const double wmb = (double)a.N * a.K * 2e-6, amb = (double)a.M * a.K * 2e-6;
  // Weights that the caches no longer hold when their next slice comes.  What else a
  // layer touches is not known here, so the line was placed by measuring stages on both
  // sides of it (8e6 / 18e6 / 40e6, 256-token slices, one layer, us): 1536 wide 793 / 793
  // / 793, 2048 1012 / 966 / 966, 2560 1329 / 1333 / 1332, 3072 1610 / 1616 / 1624, 4096
  // 2255 / 2270 / 2268, 5120 3153 / 3165 / 3158; 64-token forward 3072 wide 734 / 733 /
  // 770; two layers alike.
  const bool cold = (double)a.N * a.K >= 18e6;
  const long room = a.ws ? a.ws_elems : 0;
  const bool gelu = a.epi == EPI_GELU || a.epi == EPI_DGELU;
  // MB the epilogue reads and writes
  const double outmb = (double)a.M * a.N * 1e-6 * (a.epi == EPI_RESID ? 8 : gelu ? 4 : 2);
  auto stream_us = [&](const Cand& c, double cols) {  // for `cols` of the N columns
    const long mt = cdiv(a.M, c.bm);
    return wmb * cols / a.N * (0.1512 + 0.0253 * (mt - 1)) + amb * 0.0362 * cdiv((long)cols, c.bn);
  };
  long limit = -1;  // partial sums the plan may take; the reference plan only where needed
  auto fits = [&](double part) {
    if (part > room) return false;
    if (part <= STATIC_SCRATCH_ELEMS) return true;
    if (limit < 0) limit = std::max(STATIC_SCRATCH_ELEMS, reference_partials(a));
    return part <= limit;
  };
  double best = 1e300;
  TileChoice pick{T128x128, 1};
  for (const Cand& c : kCands) {
    if (tail && c.cfg != T64x64 && c.cfg != T128x128) continue;
    const long tiles = (long)cdiv(a.M, c.bm) * cdiv(a.N, c.bn);
    const double stream = stream_us(c, a.N);
    for (int sp : kSplits) {
      if (sp > nkt) break;
      const int ks = cdiv(nkt, sp), s = cdiv(nkt, ks);
      double t = c.main_us(tiles * s, ks, cold);
      if (s == 1 && gelu) t += 1.457 * cdiv(tiles, 256) * c.bm * c.bn / 16384.0;
      t = std::sqrt(t * t + stream * stream) + 3.563;
      const double part = s > 1 ? (double)s * a.M * a.N : 0.0;
      if (s > 1) t += 2.142 + 0.1614 * s + part * 8e-6 * 0.1364 + outmb * 0.1356;
      // a LayerNorm (or D) that follows costs a launch of its own after an unsplit
      // product
      else t += outmb * 0.1449 + (a.norm ? 2.0 + (double)a.M * a.N * 8e-6 * 0.12 : 0.0) +
                (a.dot ? 2.5 + (double)a.M * a.N * 4e-6 * 0.12 : 0.0);
      if (t < best && (s == 1 || fits(part))) {
        best = t;
        pick = {c.cfg, s, 0, 0, (long)part};
      }
    }
  }
  // Two launches over column groups: the first group's workgroups fill whole
  // rounds, the second group takes its own split count, so no round runs
  // part-empty the way a uniform split leaves the last one (the query/key/value
  // product of 144 tiles of 256 x 256: 2 x 128 + 16 x 16 workgroups against 3
  // x 144).  Taken when the model puts it 3 % under the best single launch, and
  // looked for only where 3 % outweighs the further launch.
  const double single = best;
  if (tail || single < 100.0) return pick;
  for (const Cand& c : kCands) {
    if (c.bm != 256 || c.bn < 192) continue;
    const long mt = cdiv(a.M, c.bm), tn = cdiv(a.N, c.bn);
    for (int sp1 : kSplits) {
      if (sp1 > nkt) break;
      const int ks1 = cdiv(nkt, sp1), e1 = cdiv(nkt, ks1);
      for (long r1 = 1;; ++r1) {
        const long cols1 = r1 * 256 / (mt * e1);
        if (cols1 >= tn) break;
        if (cols1 * mt * e1 != r1 * 256) continue;
        const long n1 = cols1 * c.bn, n2 = a.N - n1;
        const double t1 = std::hypot(c.main_us(r1 * 256, ks1, cold), stream_us(c, n1));
        for (int sp2 : kSplits) {
          if (sp2 > nkt) break;
          const int ks2 = cdiv(nkt, sp2), e2 = cdiv(nkt, ks2);
          const double part = (double)e1 * a.M * n1 + (double)e2 * a.M * n2;
          const double t = t1 + 2 * 3.563 + 2.142 + 0.1614 * (e1 + e2) +
                           part * 8e-6 * 0.1364 + outmb * 0.1356 +
                           std::hypot(c.main_us(mt * (tn - cols1) * e2, ks2, cold),
                                      stream_us(c, n2));
          if (t < best && t < 0.97 * single && fits(part)) {
            best = t;
            pick = {c.cfg, e1, e2, (int)cols1, (long)part};
          }
        }
      }
    }
  }
  return pick;
}

// The same for the weight-gradient products (both operands m/n-contiguous, a
// reduction over tokens, fp32 output read and written or only written): 256 x 256
// tiles where they fill the CUs, smaller ones (or splits) for narrow gradients,
// which left most CUs idle (2048 x 2048 over 2048 tokens: 64 tiles of 256 x 256 46
// us, 256 tiles of 128 x 128 28 us; 512 x 2048: 16 tiles 44 us, 64 x 64 tiles 16
// us).  Fitted like choose_tiles (rms error 8 %): on average 2.7 % over the best
// candidate, always 256 x 256 was 74 % over on the same sweep (widths 512-5120,
// 64-8192 tokens).
constexpr Cand kDwCands[] = {{T64x64, 64, 64, 3, 0.0, 0.3745, 0.3745, 0.1047},
                             {T128x128, 128, 128, 1, 0.598, 0.5815, 0.5815, 0.0},
                             {T_DW256, 256, 256, 1, 1.841, 1.3978, 1.3978, 0.0}};
TileChoice choose_dw(const GemmArgs& a, double* us = nullptr) {
  const int nkt = cdiv(a.K, 64);
  const double out = (double)a.M * a.N * 4e-6 * (a.overwrite ? 1 : 2);
  double best = 1e300;
  TileChoice pick{T_DW256, 1};
  for (const Cand& c : kDwCands) {
    const long tiles = (long)cdiv(a.M, c.bm) * cdiv(a.N, c.bn);
    for (int sp : kSplits) {
      if (sp > nkt || sp > 8) break;
      const int ks = cdiv(nkt, sp), s = cdiv(nkt, ks);
      if (s > 1 && (!a.ws || (long)s * a.M * a.N > a.ws_elems)) break;
      double t = c.main_us(tiles * s, ks, false);
      t += s > 1 ? 3.2 + ((double)s * a.M * a.N * 8e-6 + out) * 0.1659 : out * 0.1437;
      if (t < best) {
        best = t;
        pick = {c.cfg, s};
      }
    }
  }
  if (us) *us = best;
  return pick;
}

// One launch over the products of a group with tiles of BM x BN.
template <int BM, int BN, int WGM, int WGN, int STAGES, bool TAIL, bool KEEP = false>
hipError_t launch_group(GemmGroup& g, hipStream_t s) {
  if constexpr (!KEEP)
    if (g.g[0].keep) return launch_group<BM, BN, WGM, WGN, STAGES, TAIL, true>(g, s);
  constexpr int NTH = 64 * WGM * WGN;
  constexpr size_t lds = (size_t)STAGES * (BM + BN) * 64 * 2;
  long tiles = 0;
  for (int p = 0; p < g.count; ++p) tiles += (long)cdiv(g.g[p].M, BM) * cdiv(g.g[p].N, BN);
  g.walk = tiles >= 512;
  g.first[0] = 0;
  for (int p = 0; p < g.count; ++p) {
    const int tm = cdiv(g.g[p].M, BM), tn = cdiv(g.g[p].N, BN);
    // the super-tile orientation that leaves fewer idle slots
    const int up = TileWalk(tm, tn, false).supers(), side = TileWalk(tm, tn, true).supers();
    g.g[p].walk = side < up ? 2 : 1;
    g.first[p + 1] = g.first[p] + (g.walk ? std::min(up, side) : tm * tn);
  }
  const int n = g.first[g.count], blocks = g.walk ? cdiv(n, 8) * 8 * WALK_PER_XCD : n;
  constexpr auto* fn = &gemm_dma_kernel<BM, BN, 64, WGM, WGN, 1, false, false, EPI_ACC_F32, false,
                                        STAGES, STAGES, false, TAIL, GemmGroup, KEEP>;
  const hipError_t e = raise_lds<fn>(lds);
  if (e != hipSuccess) return e;
  fn<<<blocks, NTH, lds, s>>>(g);
  return hipGetLastError();
}

// shapes of gemm_dma_bf16 for a weight-gradient product
bool dw_covered(const GemmArgs& a) {
  return a.M > 0 && a.N > 0 && a.K > 0 && a.epi == EPI_ACC_F32 && a.sam == 1 && a.sbn == 1 &&
         a.sak != 1 && a.sbk != 1 && a.M % 8 == 0 && a.N % 8 == 0 && !(a.sak & 7) && !(a.sbk & 7) &&
         !((uintptr_t)a.A & 15) && !((uintptr_t)a.B & 15) && !((uintptr_t)a.C & 15) &&
         !(a.ldc & 3) && 65 * a.sak * 2 < (1l << 32) && 65 * a.sbk * 2 < (1l << 32);
}

}  // namespace

// The weight-gradient products of a layer (count <= 4, one reduction length) in one
// launch, where that is modelled faster than one launch each with its own tiles and
// splits: narrow gradients fill the chip together (1024 wide, 256 tokens a slice: 36 ->
// 27 us, 3.7 TB/s of gradient read and written), wide ones share their part-empty last
// rounds (2048 wide, 2048 tokens: 238 -> 202 us; 8-way shard of 12288: 1038 -> 963 us).
// hipErrorNotSupported: not covered, or separate launches are better.
hipError_t gemm_dw_group(const GemmArgs* g, int count, hipStream_t s) {
  clear_stale_error();
  if (count < 2 || count > 4) return hipErrorNotSupported;
  double apart = 0, out = 0;
  for (int p = 0; p < count; ++p) {
    if (!dw_covered(g[p]) || g[p].K != g[0].K) return hipErrorNotSupported;
    double t;
    choose_dw(g[p], &t);
    apart += t + 3.13;  // launch and drain
    out += (double)g[p].M * g[p].N * 4e-6 * (g[p].overwrite ? 1 : 2);
  }
  const int nkt = cdiv(g[0].K, 64);
  double best = apart;
  int pick = -1;
  for (const Cand& c : kDwCands) {
    long tiles = 0;
    for (int p = 0; p < count; ++p) tiles += (long)cdiv(g[p].M, c.bm) * cdiv(g[p].N, c.bn);
    const double t = 3.13 + c.main_us(tiles, nkt, false) + out * 0.1437;
    if (t < best) best = t, pick = c.cfg;
  }
  if (pick < 0) return hipErrorNotSupported;
  GemmGroup G;
  for (int p = 0; p < count; ++p) G.g[p] = g[p];
  G.count = count;
  const bool tail = g[0].K % 64 != 0;
  switch (pick) {
    case T64x64:
      return tail ? launch_group<64, 64, 2, 2, 3, true>(G, s)
                  : launch_group<64, 64, 2, 2, 3, false>(G, s);
    case T128x128:
      return tail ? launch_group<128, 128, 4, 2, 4, true>(G, s)
                  : launch_group<128, 128, 4, 2, 4, false>(G, s);
    case T_DW256:
      return tail ? launch_group<256, 256, 2, 4, 2, true>(G, s)
                  : launch_group<256, 256, 2, 4, 2, false>(G, s);
  }
  return hipErrorNotSupported;
}

// Shapes the DMA path takes: 16-byte-aligned operands with a unit stride and
// leading dimensions of whole 16-byte chunks; N, and M where A is contiguous along
// it, multiples of 8 (a k-contiguous A takes any number of rows); K any multiple
// of 8, or any number of tokens for the weight-gradient products.
hipError_t gemm_dma_bf16(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  const bool a_kc = a.sak == 1, b_kc = a.sbk == 1, a_mc = a.sam == 1, b_nc = a.sbn == 1;
  if (a.N % 8 || a.K <= 0) return hipErrorNotSupported;
  if (((uintptr_t)a.A & 15) || ((uintptr_t)a.B & 15)) return hipErrorNotSupported;
  const long lda = a_kc ? a.sam : a.sak, ldb = b_kc ? a.sbn : a.sbk;
  if ((lda & 7) || (ldb & 7)) return hipErrorNotSupported;
  // per-lane DMA offsets are 32-bit byte offsets from a k-origin
  auto fits = [](long rows, long ld) { return (rows + 1) * ld * 2 < (1l << 32); };
  if (!fits(a_kc ? a.M : 64, lda) || !fits(b_kc ? a.N : 64, ldb)) return hipErrorNotSupported;
  // fp32 outputs leave as 16-byte row segments, bf16 outputs (and their
  // operands) as 8-column segments
  if (a.epi == EPI_ACC_F32 && (((uintptr_t)a.C & 15) || (a.ldc & 3))) return hipErrorNotSupported;
  if (a.epi != EPI_ACC_F32 && !vec8_ok(a)) return hipErrorNotSupported;
  const bool tail = a.K % 64 != 0;
  if (a_mc && b_nc && !a_kc) {
    if (a.M % 8 || a.epi != EPI_ACC_F32) return hipErrorNotSupported;
    const TileChoice c = choose_dw(a);
    return tail ? run_cfg<false, false, false, true>(c.cfg, a, s, c.splits, 0, 0)
                : run_cfg<false, false, false, false>(c.cfg, a, s, c.splits, 0, 0);
  }
  if (!a_kc || (!b_kc && !b_nc) || a.K % 8) return hipErrorNotSupported;
  const bool fwd = a.epi == EPI_QKV || a.epi == EPI_RESID || a.epi == EPI_GELU;
  if (b_kc ? !fwd : (a.epi != EPI_STORE && a.epi != EPI_DGELU)) return hipErrorNotSupported;
  // fp16 operands: the query/key/value product (activations times the fp16 weight
  // copy) of stages whose widths are whole k-tiles
  if (a.in_f16 && (!b_kc || a.epi != EPI_QKV || tail)) return hipErrorNotSupported;
  const TileChoice c = choose_tiles(a, tail);
  if (a.need) {
    // neither plan takes more than 16 splits: below that the reference plan's search
    // cannot change the admission
    const bool small = 16l * a.M * a.N <= STATIC_SCRATCH_ELEMS;
    *a.need = small ? c.partials : std::max(c.partials, reference_partials(a));
    return hipSuccess;
  }
  if (a.in_f16)
    return run_cfg<true, true, true, false>(c.cfg, a, s, c.splits, c.splits2, c.cols1);
  if (tail)
    return b_kc ? run_cfg<true, true, false, true>(c.cfg, a, s, c.splits, 0, 0)
                : run_cfg<true, false, false, true>(c.cfg, a, s, c.splits, 0, 0);
  return b_kc ? run_cfg<true, true, false, false>(c.cfg, a, s, c.splits, c.splits2, c.cols1)
              : run_cfg<true, false, false, false>(c.cfg, a, s, c.splits, c.splits2, c.cols1);
}

}  // namespace tp
