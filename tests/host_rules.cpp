// Host side of the library's index and launch rules, compiled without device
// code and called through ctypes by test_host_rules.py.
#include "../paper_2608_23463_amd/csrc/decode.hpp"
#include "../paper_2608_23463_amd/csrc/gemm.hpp"

using namespace pf;

// Largest byte past the staged A that the fragment reads of one projection
// workgroup touch (<= 0: all of them stay inside), and how many of them read a
// chunk that is not the one asked for of the row that stands in for theirs.
template <typename T>
static int64_t staged_reads(int d, int rows, int64_t* wrong) {
  constexpr int kV = 16 / (int)sizeof(T);
  int64_t past = INT64_MIN;
  *wrong = 0;
  const int kq = d / 4;
  for (int wave = 0; wave < 4; ++wave)
    for (int st = 0; st < kq / 16; ++st)
      for (int lane = 0; lane < 64; ++lane) {
        const int g = lane >> 5, l32 = lane & 31, k = wave * kq + st * 16 + g * 8;
        for (int c = k / kV; c < (k + 8) / kV; ++c) {
          const int64_t at = staged_offset<T>(l32, c, rows, d);
          past = std::max<int64_t>(past, (at + kV - (int64_t)rows * d) * (int64_t)sizeof(T));
          // the write of the same chunk: row l32 mod rows is staged by its own index
          if (at != staged_offset<T>(l32 % rows, c, rows, d) || at / d != l32 % rows) ++*wrong;
        }
      }
  return past;
}

extern "C" int64_t host_staged_reads(int esize, int d, int rows, int64_t* wrong) {
  return esize == 2 ? staged_reads<bf16>(d, rows, wrong) : staged_reads<float>(d, rows, wrong);
}

// 1 if the register-path kernel takes a product with this many batches, column
// sums of A, or A and B read from a third source from K index ksplit3 on.
extern "C" int host_register_path(int K, int batch, int colsum, int ksplit3) {
  static float sums[1];
  GemmProblem pr{};
  pr.M = pr.N = 40;
  pr.K = K;
  pr.batch = batch;
  pr.colsum = colsum ? sums : nullptr;
  if (ksplit3 >= 0) pr.ksplit3 = ksplit3;
  return gemm_runs_register(pr);
}

// How an append's product of `rows` rows cuts K and joins the slices, planned as
// for `plan_rows` rows (0: for its own): slices, their length, lanes per chunk,
// and in fp32, whose tiles sum in different chains, the tile.
template <typename T>
static void row_plan(int rows, int n, int k, int plan_rows, int count, int* out) {
  GemmProblem pr[2];
  for (GemmProblem& q : pr) q.M = rows, q.N = n, q.K = k;
  const GemmPlan pl = plan_rows ? plan_gemm_rows<T>(pr, count, plan_rows, 256) : plan_gemm<T>(pr, count, 256);
  int zl = pl.zl, blocks;
  plan_reduce((int64_t)rows * n / 8 * count, pl.splits, &zl, &blocks);
  out[0] = plan_splits(pr[0], pl);
  out[1] = plan_k_slice(pr[0], pl);
  out[2] = zl;
  out[3] = sizeof(T) == 4 ? pl.tile : 0;
}

extern "C" void host_row_plan(int esize, int rows, int n, int k, int plan_rows, int count, int* out) {
  esize == 2 ? row_plan<bf16>(rows, n, k, plan_rows, count, out) : row_plan<float>(rows, n, k, plan_rows, count, out);
}
