// CPU-only driver (tests/test_static_plan.py builds and links it against the stage
// library): the scratch by which tp_slice_forward_static admits a product
// (GemmArgs::need) against the split partials of the launch that the same arguments
// make.  The HIP runtime's entry points below stand in for the real ones and record
// the arguments of every launch; no device is touched.
//
// Prints one line per product whose launch takes more scratch than the admission said
// or writes past the array that the admission grants, and "products N, split S".
// Also the least work of a part: column sums over rows in chunks of at least 256 rows,
// the streaming dQ kernel in key splits of at least 256 keys; and a GEMM kernel's
// attributes are set by its first launch alone.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>

#include "../../paper_2102_07988_amd/csrc/tp_kernels.hpp"

namespace {
long recorded = 0;  // most fp32 partial sums among the launches since it was cleared
int launches = 0, attribute_calls = 0;
enum { GEMM, COLSUM, ATTN, GROUP } kind = GEMM;  // what the launches' first argument is
int least = 0;                            // rows of a chunk, keys of a split (0: unsplit)
dim3 grid_, block_;
size_t lds_;
hipStream_t stream_;
}  // namespace

// The GEMM and reduction kernels take their GemmArgs first (k_split, splits,
// split_cols and splits2 as set by the launcher).
extern "C" hipError_t hipLaunchKernel(const void*, dim3 grid, dim3, void** args, size_t,
                                      hipStream_t) {
  if (kind == COLSUM) {
    const tp::ColJobs& j = *(const tp::ColJobs*)args[0];
    least = j.chunks > 1 ? j.rows_per : 0;
    return hipSuccess;
  }
  if (kind == GROUP) return hipSuccess;
  if (kind == ATTN) {
    const tp::AttnArgs& a = *(const tp::AttnArgs*)args[0];
    if (a.nsplit > 1) least = a.kv_chunk;
    return hipSuccess;
  }
  const tp::GemmArgs& a = *(const tp::GemmArgs*)args[0];
  long n = 0;
  if (a.split_cols)
    n = (long)a.splits * a.M * a.split_cols + (long)a.splits2 * a.M * (a.N - a.split_cols);
  else if (a.splits > 1)
    n = (long)a.splits * a.M * a.N;
  if (grid.z > 1 && (int)grid.z != a.splits) n = INT64_MAX;  // not what this driver expects
  recorded = std::max(recorded, n);
  ++launches;
  return hipSuccess;
}
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
  ++attribute_calls;
  return hipSuccess;
}
extern "C" hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  grid_ = g, block_ = b, lds_ = lds, stream_ = s;
  return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = grid_, *b = block_, *lds = lds_, *s = stream_;
  return hipSuccess;
}

int main() {
  using namespace tp;
  char* base = (char*)0x7e0000000000;  // never dereferenced
  int bad = 0, products = 0, split = 0;
  // the forward's products of a slice of n rows: widths and shards as the stage takes them
  for (int H : {64, 96, 256, 512, 768, 1024, 1536, 2048, 2560, 3072, 4096, 5120, 8192, 12288, 16384})
    for (int parts : {1, 2, 8})
      for (int n : {1, 7, 8, 16, 31, 64, 80, 100, 128, 144, 200, 256, 257, 300, 400, 512, 777, 1024, 2048, 4096})
        for (int dtype : {DT_BF16, DT_FP32})
          for (int which = 0; which < 4; ++which) {
            if (H % (16 * parts)) continue;
            const int A = H / parts, F = 4 * H / parts;
            GemmArgs g;
            g.M = n;
            g.N = which == 0 ? 3 * A : which == 2 ? F : H;
            g.K = which == 1 ? A : which == 3 ? F : H;
            g.A = base, g.sam = g.K, g.sak = 1;
            g.B = base, g.sbk = 1, g.sbn = g.K;
            g.epi = which == 0 ? EPI_QKV : which == 2 ? EPI_GELU : EPI_RESID;
            g.bias = base, g.C = base, g.ldc = g.N, g.R = base, g.ldr = g.N;
            g.C2 = base, g.ldc2 = g.N, g.q = g.k = g.v = g.vb = base, g.H = A;
            RowNorm nm;
            nm.g = nm.b = base;
            bool done = false;
            if (which == 1) g.norm = &nm, g.norm_done = &done;
            // the stage's split scratch
            g.ws = (float*)base;
            g.ws_elems = 8l * std::min(n, 256) * std::max(std::max(F, H), 3 * A);
            long need = 0;
            g.need = &need;
            if (gemm(dtype, g, nullptr) != hipSuccess) continue;  // not covered
            g.need = nullptr;
            recorded = 0, launches = 0;
            const hipError_t e = gemm(dtype, g, nullptr);
            ++products;
            split += recorded > 0;
            const bool over = recorded > need || (need <= STATIC_SCRATCH_ELEMS && recorded > STATIC_SCRATCH_ELEMS);
            if (e != hipSuccess || !launches || over) {
              ++bad;
              if (bad <= 20)
                std::printf("M %d N %d K %d dtype %d: admitted by %ld, launches take %ld (%d launches, status %d)\n",
                            g.M, g.N, g.K, dtype, need, recorded, launches, (int)e);
            }
          }
  std::printf("products %d, split %d\n", products, split);
  int chunked = 0, kv_split = 0;
  kind = COLSUM;
  for (int H : {64, 256, 512, 1024, 2048, 4096, 12288})
    for (int rows = 1; rows <= 4200; rows += rows < 1100 ? 1 : 97) {
      ColJobs J;
      const int cols[6] = {H, 4 * H, H, H, 3 * H, H};
      for (int i = 0; i < 6; ++i) {
        J.job[i].a = base, J.job[i].cols = J.job[i].lda = cols[i], J.job[i].sum = (float*)base;
        if (i == 2 || i == 5) J.job[i].x = base, J.job[i].xsum = (float*)base;
      }
      J.count = 6, J.rows = rows, J.part = (float*)base;
      J.part_elems = 8l * std::min(rows, 256) * 4 * H;
      least = 0;
      if (col_reduce(DT_BF16, 1, J, nullptr) != hipSuccess) ++bad;
      chunked += least > 0;
      if (least > 0 && least < 256 && ++bad <= 20)
        std::printf("column sums: H %d, %d rows in chunks of %d\n", H, rows, least);
    }
  kind = ATTN;
  for (int heads : {8, 16, 32, 64, 128})
    for (int n : {1, 16, 100, 128, 256, 512})
      for (int r = n; r <= 4096; r += r < 1100 ? 1 : 37) {
        // shorter prefixes take the recomputing dQ kernel
        if ((r + 127) / 128 * heads < 128) continue;
        AttnArgs a;
        a.l = r - n, a.r = r, a.d = 128, a.heads = heads, a.H = a.ld = heads * 128;
        a.Lmax = r, a.f16 = 1, a.have_D = true;
        a.o = a.dq = a.pack = base, a.q = a.kc = a.vc = a.dout = base;
        a.ld_dq = 3 * a.H, a.dq_seq = 3 * a.H, a.pack_l = a.l;
        a.lse = a.D = a.dk = a.dv = a.ws = (float*)base;
        a.ws_elems = 8 * (16384l * 128 + 2 * 16384);
        // the stage's dS planes at the longest slice of the shortest stage that has it
        a.pd = (uint16_t*)base, a.pd_elems = (long)heads * r * std::min(1024, (r + 255) / 256 * 256);
        least = 0;
        if (attn_bwd(DT_BF16, a, nullptr) != hipSuccess && ++bad <= 40)
          std::printf("dQ: %d heads, %d queries, %d keys not taken\n", heads, n, r);
        kv_split += least > 0;
        if (least > 0 && least < 256 && ++bad <= 40)
          std::printf("dQ: %d heads, %d queries, %d keys in splits of %d\n", heads, n, r, least);
      }
  kind = GROUP;
  for (int H : {1024, 2048, 12288})
    for (int pass = 0; pass < 2; ++pass) {
      GemmArgs g[4];
      for (int i = 0; i < 4; ++i) {
        g[i].M = i == 1 ? 4 * H : i == 3 ? 3 * H : H, g[i].N = i == 0 ? 4 * H : H, g[i].K = 256;
        g[i].A = g[i].B = base, g[i].sam = g[i].sbn = 1, g[i].sak = g[i].M, g[i].sbk = g[i].N;
        g[i].epi = EPI_ACC_F32, g[i].C = base, g[i].ldc = g[i].N;
      }
      attribute_calls = 0;
      const bool run = gemm_dw_group(g, 4, nullptr) == hipSuccess;
      if (pass && run && attribute_calls && ++bad)
        std::printf("grouped products, H %d: %d attribute calls in the second launch\n", H, attribute_calls);
    }
  std::printf("column sums in chunks %d, dQ launches split %d\n", chunked, kv_split);
  if (bad) std::printf("FAILED %d\n", bad);
  return bad ? 1 : 0;
}
