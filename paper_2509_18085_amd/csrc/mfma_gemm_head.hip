// The LM head (mfma_gemm_kernel.h, EPI_LMHEAD): one launch whatever the number of rows in use, which only the device knows.
#include "mfma_gemm_kernel.h"

namespace spiffy {

namespace {

// One workgroup a compute unit, so a launch takes whole rounds of 256 workgroups, and the shape of the tile decides how full
// they are.  Every workgroup reads the row count and picks the shape of the launch:
//   vocabulary x tokens   time of a round, relative (products 1024 .. 4096 deep)
//   256 x 192             50
//   256 x 256             61      385 .. 512 rows: two token tiles instead of three
//   128 x 256             35      half the vocabulary: fills rounds that 256 leave half empty
//   128 x 128             25      the same up to 128 rows, where the weight stream is the bound
// The times are the ones with the least regret over 76 measured launches (vocabularies of 32000, 126464 and 152064, 8 .. 1000
// rows), 0.3% over the best shape of each launch, 256 x 192 alone 10.2%, and over 128 of 512 .. 6144 rows (1280 .. 200000
// tokens), where a round of 128 x 256 at 34 was chosen at 1640 rows of 32000 (241 us, 256 x 256 229).  Whole heads, us, 256 x 192 alone -> this rule:
// 152064 x 3584 at 24 rows 246 -> 223, at 250 rows 378 -> 308, at 440 rows 529 -> 470; 126464 x 4096 at 250 rows 358 -> 258, at
// 1000 rows 958 -> 837; 32000 x 2048 at 24 rows 57 -> 49.  256 x 128 (250 rows of 126464 302, of 32000 59) is ahead of none of
// them by more than 3%.
// The summaries are per 128 vocabulary rows in every shape and added up in the same order: a row's bits do not depend on it.
constexpr int T_256_192 = 50, T_256_256 = 61, T_128_256 = 35, T_128_128 = 25;

enum Shape { S_256_192, S_256_256, S_128_256, S_128_128 };
__host__ __device__ __forceinline__ Shape head_shape(int rows, int tiles) {       // tiles of 256 vocabulary rows
  const auto rounds = [](int workgroups) { return (workgroups + 255) / 256; };
  const int c192 = T_256_192 * rounds(tiles * ((rows + 191) / 192)), n256 = (rows + 255) / 256;
  const int whole = T_256_256 * rounds(tiles * n256) < c192 ? T_256_256 * rounds(tiles * n256) : c192;
  const int half = rows <= 128 ? T_128_128 * rounds(2 * tiles) : T_128_256 * rounds(2 * tiles * n256);
  return half < whole ? (rows <= 128 ? S_128_128 : S_128_256) : (whole < c192 ? S_256_256 : S_256_192);
}
__host__ __device__ __forceinline__ int head_workgroups(Shape s, int rows, int tiles) {
  return s == S_128_128 ? 2 * tiles : s == S_128_256 ? 2 * tiles * ((rows + 255) / 256)
       : s == S_256_256 ? tiles * ((rows + 255) / 256) : tiles * ((rows + 191) / 192);
}

__global__ __launch_bounds__(256) void lmhead_mfma_kernel(GemmArgs a, int tiles) {
  const int wave = wave_id();
  switch (head_shape(a.M_dev ? min(*a.M_dev, a.M) : a.M, tiles)) {
    case S_128_128: return gemm_tile<EPI_LMHEAD, 128, 5, 128, 5>(a, 2 * tiles, 1, wave);
    case S_128_256: return gemm_tile<EPI_LMHEAD, 256, 3, 128, 3>(a, 2 * tiles, 1, wave);
    case S_256_256: return gemm_tile<EPI_LMHEAD, 256, 3, 256, 0>(a, tiles, 1, wave);
    default: return gemm_tile<EPI_LMHEAD, 192, 3, 256, 0>(a, tiles, 1, wave);
  }
}

}  // namespace

hipError_t launch_gemm_head(const GemmArgs& a, hipStream_t st) {
  // As many workgroups as the shape of any number of rows up to a.M takes: a shape and its tiles change at multiples of 64 rows
  // (128, 192, 256) only.  Those beyond the tiles in use leave at once, which takes about 1 us per 256.
  const int tiles = cdiv(a.N, BM);
  int grid = 1;
  bool choice = false;
  for (int rows = 64; rows < a.M + 64; rows += 64) {
    const Shape s = head_shape(rows, tiles);
    const int n = head_workgroups(s, rows, tiles);
    grid = n > grid ? n : grid;
    choice = choice || s != S_256_192;
  }
  if (!choice) return launch_t<EPI_LMHEAD, 192, 3>(a, tiles, cdiv(a.M, 192), st);     // (2 - 3 us less than the kernel of four)
  constexpr size_t lds = smem_bytes<EPI_LMHEAD, 256, 3, 256, 0>();       // one allocation for every shape
  static_assert(lds <= 160 * 1024 && lds >= smem_bytes<EPI_LMHEAD, 192, 3, 256, 0>() &&
                lds >= smem_bytes<EPI_LMHEAD, 128, 5, 128, 5>() && lds >= smem_bytes<EPI_LMHEAD, 256, 3, 128, 3>(), "LDS");
  static std::atomic<unsigned long long> lds_ok{0};
  const hipError_t e = allow_dynamic_lds((const void*)lmhead_mfma_kernel, (int)lds, lds_ok);
  if (e != hipSuccess) return e;
  lmhead_mfma_kernel<<<grid, 256, lds, st>>>(a, tiles);
  return hipGetLastError();
}

}  // namespace spiffy
