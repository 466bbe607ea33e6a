// Host side of the bf16 MFMA GEMM: which tile shapes a projection is launched with, the residual epilogue's instantiations,
// and the reduction of the K slices.  The kernel is in mfma_gemm_kernel.h; the instantiations of the other epilogues are in
// mfma_gemm_{store,qkv,swiglu,partial,head}.hip (one compilation each).
#include "mfma_gemm_kernel.h"

namespace spiffy {

namespace {

// out[m,:] = R[m,:] + sum_z P[z][m,:]  (fixed order), optionally followed by RMSNorm of that row.
// One workgroup per row, of 256 or 1024 threads: with few rows the launch is latency-bound and 1024 threads have every
// load of a row in flight at once.  The thread count is scheduling only.  The row's sum of squares is defined by the
// 256-thread order: a lane adds the sums of its four elements over the 256-element chunks w, w+4, w+8, .. (w = its
// wavefront), the 64 lanes of a wavefront are summed, then the four wavefront sums.  With 1024 threads every
// (chunk, lane) sum goes through LDS and the first four wavefronts add them in that same order.
//
// HEAD: the last layer's masked rows, which the head starts from.  Their RMSNorm is taken from the rounded row in the order of
// rmsnorm_row (256 threads, eight elements each at a time), the bits that a launch of its own gave (4.7 us).
enum { RED_PLAIN = 0, RED_NORM = 1, RED_HEAD = 2 };
template <int MODE>
__global__ __launch_bounds__(1024) void splitk_reduce_kernel(const float* __restrict__ P, int ksplit,
                                                            const bf16_t* __restrict__ R, bf16_t* __restrict__ out,
                                                            const bf16_t* __restrict__ gain, float eps,
                                                            bf16_t* __restrict__ normed, int M, int N,
                                                            const int32_t* __restrict__ n_rows_dev,
                                                            const int32_t* __restrict__ out_rows,
                                                            const int32_t* __restrict__ r_rows,
                                                            int32_t* __restrict__ head_rows, int32_t* __restrict__ head_count) {
  constexpr bool NORM = MODE == RED_NORM;
  __shared__ float red[4];
  extern __shared__ float rowbuf[];               // NORM: the row in fp32; 1024 threads: then one sum per (chunk, lane)
  const int m = blockIdx.x;
  if (MODE == RED_HEAD && m == 0 && threadIdx.x == 0) *head_count = *n_rows_dev;
  if (n_rows_dev && m >= *n_rows_dev) return;
  const size_t mo = out_rows ? (size_t)out_rows[m] : (size_t)m;     // where the row goes (compacted rows scatter back)
  const size_t mr = r_rows ? (size_t)r_rows[m] : (size_t)m;
  if (MODE == RED_HEAD && threadIdx.x == 0) head_rows[m] = (int32_t)mo;
  const int stride = 4 * (int)blockDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool wide = blockDim.x > 256;
  float* lane_ss = rowbuf + N;
  float ss = 0.f;
  for (int base = wave * 256; base < N; base += stride) {     // wavefront-uniform: one chunk per trip
    const int n = base + lane * 4;
    float c = 0.f;
    if (n < N) {
      f32x4 s = *reinterpret_cast<const f32x4*>(P + (size_t)m * N + n);
      for (int z = 1; z < ksplit; ++z) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(P + ((size_t)z * M + m) * N + n);
        s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] += p[3];
      }
      const bf16x4 r = *reinterpret_cast<const bf16x4*>(R + mr * N + n);
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[e] += static_cast<float>(r[e]);
        o[e] = static_cast<bf16_t>(s[e]);
        if (NORM) { rowbuf[n + e] = s[e]; c += s[e] * s[e]; }
      }
      *reinterpret_cast<bf16x4*>(out + mo * N + n) = o;
      if (MODE == RED_HEAD) *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(rowbuf) + n) = o;
    }
    if (NORM) {
      if (wide) lane_ss[(base >> 8) * 64 + lane] = c; else ss += c;
    }
  }
  if (MODE == RED_HEAD) {
    const bf16x8* row = reinterpret_cast<const bf16x8*>(rowbuf);
    const bf16x8* g8 = reinterpret_cast<const bf16x8*>(gain);
    bf16x8* n8 = reinterpret_cast<bf16x8*>(normed + (size_t)m * N);
    const int nv = N / 8;
    __syncthreads();
    if (wave < 4) {
      for (int i = threadIdx.x; i < nv; i += 256) {
        const bf16x8 v = row[i];
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float f = static_cast<float>(v[e]); ss += f * f; }
      }
      ss = wave_sum(ss);
      if (lane == 0) red[wave] = ss;
    }
    __syncthreads();
    const float inv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)N + eps);
    for (int i = threadIdx.x; i < nv; i += (int)blockDim.x) {
      const bf16x8 v = row[i], g = g8[i];
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = static_cast<bf16_t>(static_cast<float>(v[e]) * inv * static_cast<float>(g[e]));
      n8[i] = o;
    }
    return;
  }
  if (!NORM) return;
  if (wide) {
    __syncthreads();
    if (wave < 4)
      for (int k = wave; k < (N + 255) / 256; k += 4) ss += lane_ss[k * 64 + lane];
  }
  if (wave < 4) {
    ss = wave_sum(ss);
    if (lane == 0) red[wave] = ss;
  }
  __syncthreads();
  const float inv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)N + eps);
  for (int n = threadIdx.x * 4; n < N; n += stride) {
    const bf16x4 g = *reinterpret_cast<const bf16x4*>(gain + n);
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16_t>(rowbuf[n + e] * inv * static_cast<float>(g[e]));
    *reinterpret_cast<bf16x4*>(normed + (size_t)m * N + n) = o;
  }
}

}  // namespace

// number of K slices for the narrow-N projections: a function of (N, K) only
int mfma_ksplit(int N, int K) {
  const int n_tiles = cdiv(N, 128), kt = K / BKK;
  int ks = 1;
  while (ks < 4 && 4 * n_tiles * ks < 224 && kt / (ks + 1) >= 8) ++ks;
  // and no slice longer than 128 K-tiles (8192 elements): a split-K launch is one round of workgroups whose time is the
  // slice length.  K = 18944 over 768 rows and 3584 columns: 118.5 us with two slices (168 workgroups), 97.2 us with
  // three (252), 129.7 us with four (two rounds); 1024 rows of that shape pay for it (336 workgroups with three).
  const int by_length = cdiv(kt, 128);
  if (by_length > ks) ks = by_length < 4 ? by_length : 4;
  return ks;
}

bool mfma_gemm_supported(int epi, const GemmArgs& a) {
  if (a.K % BKK != 0 || a.K < BKK || a.M < 1) return false;
  // per-lane byte offsets inside an operand are 32-bit
  const size_t lim = (size_t)1 << 32;
  const size_t ldw = a.ldw ? a.ldw : a.K;
  if ((size_t)a.M * a.lda * 2 >= lim || (size_t)a.N * ldw * 2 >= lim) return false;
  if (epi == EPI_SWIGLU) return a.N % 32 == 0;
  if (epi == EPI_LMHEAD) return a.N >= 1;
  if (epi == EPI_QKV)      // whole heads of 128 columns: the epilogue pairs columns of a head
    return a.Nseg[0] > 0 && a.Nseg[1] > 0 && a.Nseg[2] > 0 && (a.Nseg[0] | a.Nseg[1] | a.Nseg[2]) % 128 == 0 &&
           a.Nseg[0] + a.Nseg[1] + a.Nseg[2] == a.N;
  return a.N % 64 == 0 && a.Nseg[0] == a.N && !a.bias[0];      // one weight matrix
}

int mfma_lmhead_partials_per_row(int V) { return cdiv(V, BM) * 2; }

// Tile shape: a pure scheduling choice (it never changes the K order of any output element, so a row's result
// is bit-identical whatever shape runs it).  Estimated cost = rounds over the 256 CUs x time of one K-tile of
// one workgroup, the larger of its matrix-pipe time (32 cycles per 32x32x16 MFMA, 4 K steps, a penalty for
// narrow tiles) and the time to bring its operands in (about 40 bytes per clock per CU).  With few rows
// (one or a few states) the projections are weight-streaming problems: 64- and 128-row tiles spend a quarter
// or half of the matrix work of a 256-row tile on them and cover more CUs.
static const int kTileWidths[5] = {192, 128, 96, 64, 32};
// estimated time of one K-tile of one workgroup of shape bm x kTileWidths[wi]
static float tile_cost(int bm, int wi) {
  const float eff[5] = {1.0f, 0.85f, 0.6f, 0.55f, 0.4f};
  const int bn = kTileWidths[wi];
  const float mfma = (float)(bm / 64) * ((float)bn / 64.0f) * 128.0f / eff[wi];
  const float load = (float)(bm + bn) * 3.2f;
  return mfma > load ? mfma : load;
}
static TileShape choose_tile(int M, int n_cols, int unit, int ksplit, bool allow192, bool allow32 = false, bool allow96 = false,
                             bool allow96_two_rows = false, float* cost_out = nullptr) {
  const int heights[4] = {256, 128, 64, 32};
  const int* widths = kTileWidths;
  TileShape best = {256, 0};
  float best_cost = 1e30f;
  for (int h = 0; h < 4; ++h)
    for (int i = 0; i < 5; ++i) {
      const int bm = heights[h], bn = widths[i];
      const int cols = bn / unit;                 // output columns (or SwiGLU features) per tile
      if ((bn == 192 && (!allow192 || bm <= 64)) || (bn == 64 && bm == 128) || n_cols % cols != 0) continue;
      // 96-wide tiles: one row of tiles over few rows (weight streaming), where they turn 192 workgroups into 256
      // (the QKV projection also takes them over two rows of 128- or 64-row tiles: 256 workgroups where 128 columns
      // give 192; 41.4 against 43.3 us at 256 rows, 31.9 against 35.2 us at 128 rows in interleaved runs)
      if (bn == 96 && !((allow96 && (bm == 64 || bm == 128) && M <= bm) ||
                        (allow96_two_rows && (bm == 64 || bm == 128) && M <= 2 * bm))) continue;
      // 32-wide tiles (one or two wavefronts per workgroup) exist for the split-K projections of one or two states
      if ((bn == 32 || bm == 32) && !(allow32 && bn == 32 && bm <= 64)) continue;
      const int tiles = cdiv(M, bm) * (n_cols / cols) * ksplit;
      const float cost = (float)cdiv(tiles, 256) * tile_cost(bm, i);
      if (cost < best_cost) { best_cost = cost; best = {bm, bn}; }
    }
  if (cost_out) *cost_out = best_cost;
  return best;
}

// The launches of one projection: one, or two column ranges (the two-part schedule of the gate/up projection).
// Host arithmetic only; launch_gemm_mfma executes exactly this plan.
GemmPlan plan_gemm_mfma(int epi, int M, int N, int ksplit) {
  GemmPlan p = {};
  if (ksplit < 1) ksplit = 1;
  auto one = [&](TileShape t, int unit) {
    p.n_parts = 1;
    p.part[0] = {t.bm, t.bn, 0, N, cdiv(M, t.bm) * (N / (t.bn / unit)) * ksplit};
  };
  switch (epi) {
    case EPI_STORE:
    case EPI_QKV:
      one(choose_tile(M, N, 1, 1, true, false, false, true), 1);
      break;
    case EPI_RESID: {
      // 256-row tiles only; 128 columns wide unless N is an odd multiple of 64 or the narrower tile fills the chip better
      const TileShape t = choose_tile(M, N, 1, 1, false);
      one(TileShape{256, (N % 128 != 0 || (t.bm == 256 && t.bn == 64)) ? 64 : 128}, 1);
      break;
    }
    case EPI_PARTIAL:
      one(choose_tile(M, N, 1, ksplit, false, true), 1);
      break;
    case EPI_SWIGLU: {
      float whole = 0.f;
      const TileShape t = choose_tile(M, N, 2, 1, true, false, true, false, &whole);   // a tile of width w holds w/2 features
      one(t, 2);
      // Two-part column schedule, for widths whose best single shape leaves the last round of workgroups mostly empty
      // (18944 features over 768 rows: 888 tiles of 256 x 128 = 3.47 rounds, and 96 does not divide the width; over 128
      // rows: 296 tiles of 128 x 128, 1.16 rounds): one shape over as many leading features as fill whole rounds of the
      // 256 CUs - 256 x 192 tiles, or the best single shape - then the best shape for the rest, as a second launch on
      // the same stream.  Same K order in every shape, so the output bits are those of the single launch; measured
      // 207.8 -> 190.5 us at 768 rows (170 column tiles of 256 x 192, then 246 tiles of 128 x 128) and 83.9 -> 69.7 us
      // at 128 rows (256 tiles of 128 x 128, then 160 of 64 x 64).
      float best = 0.9f * whole;          // a second launch has to promise at least a tenth
      auto try_main = [&](TileShape tm) {
        int wi = 0;
        while (wi < 5 && kTileWidths[wi] != tm.bn) ++wi;
        if (wi == 5) return;
        const int per = tm.bn / 2, mt = cdiv(M, tm.bm);               // features per tile, row tiles
        const int rounds = (int)(((long long)mt * (N / per)) / 256);
        if (rounds < 1) return;
        const int main_tiles = (256 * rounds) / mt;                    // column tiles of the first part
        const int rest = N - per * main_tiles;                         // features left; a multiple of 32 as N is
        if (rest <= 0) return;
        float rest_cost = 0.f;
        const TileShape tr = choose_tile(M, rest, 2, 1, true, false, true, false, &rest_cost);
        const float cost = (float)rounds * tile_cost(tm.bm, wi) + rest_cost;
        if (tr.bn == 0 || cost > best) return;
        best = cost;
        p.n_parts = 2;
        p.part[0] = {tm.bm, tm.bn, 0, per * main_tiles, mt * main_tiles};
        p.part[1] = {tr.bm, tr.bn, per * main_tiles, rest, cdiv(M, tr.bm) * (rest / (tr.bn / 2))};
      };
      try_main(TileShape{256, 192});
      if (t.bn != 0 && !(t.bm == 256 && t.bn == 192)) try_main(t);
      break;
    }
    default:
      break;
  }
  return p;
}

// Tile shapes of a layer's projections.  Every shape's time is taken as
//   3.5 us + 1 us per further round + K-tiles x (c0 r + c1 w + c2 w / mt + c3 r fill)
// r = rounds over the 256 compute units, w = rounds in workgroups (the last one not rounded up), mt = row tiles (workgroups
// that share a weight tile), fill = rows per tile row.  The coefficients (us per K-tile of 64) are a non-negative least
// squares fit to 5,500 measured launches: rows 16 .. 1088, the projections of three models (K slices of 11 .. 99 tiles,
// 2048 .. 37888 columns), 7 - 11% rms of a launch for the small shapes, 2 - 5% for the large ones.  Picking by them
// costs 1.7% over the best shape of each launch, the rule of plan_gemm_mfma 5.4%; its shape stays where the fit
// does not promise 3%.  It holds beyond the fit: over 6,400 launches of 16 .. 16384 rows (QKV with its own epilogue, two more
// models) it costs 0.2% up to 128 rows, 0.5% up to 1088, 1.3% above, the other rule 6.1% over all.  Measured, us, its shape ->
// this one: gate/up at 352 rows 78 -> 68 (256 x 192 -> 192 x 192), 768 rows 142 -> 128; down at 192 rows 49.8 -> 40.9 (64 x 128 ->
// 128 x 64); QKV of 4608 columns at 320 rows 27.9 -> 22.4.
struct ShapeCost { int bm, bn; float c[4]; };
static const ShapeCost kShapeCost[] = {
    {256, 256, {0.943f, 0.329f, 0.143f, 0.076f}}, {256, 192, {0.743f, 0.232f, 0.118f, 0.083f}},
    {256, 128, {0.497f, 0.057f, 0.198f, 0.179f}}, {256, 64, {0.478f, 0.110f, 0.062f, 0.076f}},
    {384, 128, {0.816f, 0.198f, 0.071f, 0.069f}}, {320, 192, {0.868f, 0.379f, 0.064f, 0.081f}},
    {320, 128, {0.706f, 0.151f, 0.132f, 0.059f}}, {192, 192, {0.520f, 0.154f, 0.225f, 0.164f}},
    {192, 128, {0.296f, 0.000f, 0.343f, 0.279f}}, {128, 192, {0.475f, 0.000f, 0.350f, 0.164f}},
    {128, 128, {0.206f, 0.000f, 0.382f, 0.245f}}, {128, 96, {0.477f, 0.091f, 0.026f, 0.013f}},
    {128, 64, {0.189f, 0.000f, 0.134f, 0.168f}},  {64, 128, {0.260f, 0.000f, 0.295f, 0.109f}},
    {64, 96, {0.290f, 0.024f, 0.156f, 0.047f}},   {64, 64, {0.128f, 0.000f, 0.139f, 0.125f}},
    {64, 32, {0.204f, 0.017f, 0.020f, 0.024f}},   {32, 32, {0.054f, 0.016f, 0.097f, 0.046f}}};

static float shape_cost(const ShapeCost& s, int M, int n_cols, int unit, int k_tiles, int ksplit) {
  const int mt = cdiv(M, s.bm), tiles = mt * (n_cols / (s.bn / unit)) * ksplit, r = cdiv(tiles, 256);
  const float w = (float)tiles / 256.f, fill = (float)M / (float)(mt * s.bm), kt = (float)k_tiles / (float)ksplit;
  return 3.5f + (float)(r - 1) + kt * (s.c[0] * (float)r + s.c[1] * w + s.c[2] * w / (float)mt + s.c[3] * (float)r * fill);
}
// Tiles of 192 rows that are one full round of four slices take longer than the fit says: a layer of width 2048 with 608 .. 768 rows
// 133 - 138 us instead of 125 - 135.  With fewer or more of them they are the better ones (layers: 544 rows of width 2048 122 -> 116
// us, 1440 rows 231 -> 219, 1280 rows of width 1024 158 -> 145).
static bool mispriced(const ShapeCost& s, int M, int n_cols, int ksplit) {
  return s.bm == 192 && ksplit == 4 && cdiv(M, s.bm) * (n_cols / s.bn) * ksplit == 256;
}
GemmPlan plan_gemm_layer(int epi, int M, int N, int K, int ksplit, float* cost_us) {
  GemmPlan p = plan_gemm_mfma(epi, M, N, ksplit);
  if (ksplit < 1) ksplit = 1;
  const int unit = epi == EPI_SWIGLU ? 2 : 1, kt = K / BKK;
  auto cost_of = [&](int bm, int bn, int n) {
    for (const ShapeCost& s : kShapeCost)
      if (s.bm == bm && s.bn == bn) return shape_cost(s, M, n, unit, kt, ksplit);
    return 1e30f;
  };
  auto best_shape = [&](int n, TileShape& t) {
    float best = 1e30f;
    for (const ShapeCost& s : kShapeCost) {
      if (n % (s.bn / unit) != 0 || !has_shape(epi, s.bm, s.bn)) continue;
      if (mispriced(s, M, n, ksplit)) continue;
      const float c = shape_cost(s, M, n, unit, kt, ksplit);
      if (c < best) { best = c; t = {s.bm, s.bn}; }
    }
    return best;
  };
  float now = 0.f;
  for (int i = 0; i < p.n_parts; ++i) now += cost_of(p.part[i].bm, p.part[i].bn, p.part[i].ncols);
  if (cost_us) *cost_us = now;
  if (epi != EPI_QKV && epi != EPI_PARTIAL && epi != EPI_SWIGLU) return p;
  float best = 0.97f * now;
  TileShape t = {0, 0};
  const float whole = best_shape(N, t);
  if (whole < best) {
    best = whole;
    p.n_parts = 1;
    p.part[0] = {t.bm, t.bn, 0, N, cdiv(M, t.bm) * (N / (t.bn / unit)) * ksplit};
  }
  // gate/up in two column ranges: whole rounds of one shape, then the rest (plan_gemm_mfma says why)
  if (epi == EPI_SWIGLU) {
    best = best < 0.97f * whole ? best : 0.97f * whole;
    for (const ShapeCost& s : kShapeCost) {
      if (!has_shape(epi, s.bm, s.bn)) continue;
      const int per = s.bn / 2, mt = cdiv(M, s.bm);
      for (int r = 1; r <= (int)((long long)mt * (N / per) / 256); ++r) {
        const int main_tiles = 256 * r / mt, rest = N - per * main_tiles;
        if (rest <= 0 || rest % 32 != 0) continue;
        const float c_main = shape_cost(s, M, per * main_tiles, 2, kt, 1);
        if (c_main >= best) break;
        TileShape tr = {0, 0};
        const float c = c_main + best_shape(rest, tr);
        if (tr.bn == 0 || c >= best) continue;
        best = c;
        p.n_parts = 2;
        p.part[0] = {s.bm, s.bn, 0, per * main_tiles, mt * main_tiles};
        p.part[1] = {tr.bm, tr.bn, per * main_tiles, rest, cdiv(M, tr.bm) * (rest / (tr.bn / 2))};
      }
    }
  }
  if (cost_us) {
    *cost_us = 0.f;
    for (int i = 0; i < p.n_parts; ++i) *cost_us += cost_of(p.part[i].bm, p.part[i].bn, p.part[i].ncols);
  }
  return p;
}

// The same for a launch of which only the device knows how many of the M rows are in use (the masked rows of a last layer).  What is
// best for all of them can be far off for some: with 67 of 1280 rows of width 4096 a layer takes 388 us in tiles of 320 rows and 303 in
// plan_gemm_mfma's tiles of 256.  Above 512 rows that rule's plan therefore gives way only to one shape that is no taller and is priced
// no higher for any number of rows (prices change where a row tile begins, every 64 rows), and lower by 3% on average.  Over 3,092 last
// layers of 513 .. 2048 rows (five models, 5 .. 100% of the rows masked), against plan_gemm_mfma's: 2.1% less on average, 1.6% more at
// most; plan_gemm_layer's 2.2% less, 32% more at most.  Up to 512 rows, 2,068 layers, that one is 2.9% less, 4.8% more at most.
GemmPlan plan_gemm_masked(int epi, int M, int N, int K, int ksplit) {
  if (M <= kMaskedLikeLayerRows) return plan_gemm_layer(epi, M, N, K, ksplit);
  const GemmPlan general = plan_gemm_mfma(epi, M, N, ksplit);
  if (epi != EPI_PARTIAL && epi != EPI_SWIGLU) return general;
  if (ksplit < 1) ksplit = 1;
  const int unit = epi == EPI_SWIGLU ? 2 : 1, kt = K / BKK, step = 64 * cdiv(M, 2048);      // at most 33 row counts
  const auto price = [&](int bm, int bn, int rows, int n) {
    for (const ShapeCost& s : kShapeCost)
      if (s.bm == bm && s.bn == bn) return shape_cost(s, rows, n, unit, kt, ksplit);
    return 1e30f;
  };
  int tallest = 0, points = 0;
  float now[33], sum = 0.f;
  for (int rows = 1; points < 33; rows += step) {
    const int m = rows < M ? rows : M;
    now[points] = 0.f;
    for (int i = 0; i < general.n_parts; ++i) now[points] += price(general.part[i].bm, general.part[i].bn, m, general.part[i].ncols);
    sum += now[points++];
    if (rows >= M) break;
  }
  for (int i = 0; i < general.n_parts; ++i) tallest = general.part[i].bm > tallest ? general.part[i].bm : tallest;
  float best = 0.97f * sum;
  GemmPlan p = general;
  for (const ShapeCost& s : kShapeCost) {
    if (s.bm > tallest || N % (s.bn / unit) != 0 || !has_shape(epi, s.bm, s.bn) || mispriced(s, M, N, ksplit)) continue;
    float total = 0.f;
    bool never_longer = true;
    for (int i = 0; i < points && never_longer; ++i) {
      const int rows = 1 + i * step;
      const float c = shape_cost(s, rows < M ? rows : M, N, unit, kt, ksplit);
      never_longer = c <= now[i];
      total += c;
    }
    if (!never_longer || total >= best) continue;
    best = total;
    p.n_parts = 1;
    p.part[0] = {s.bm, s.bn, 0, N, cdiv(M, s.bm) * (N / (s.bn / unit)) * ksplit};
  }
  return p;
}

// The launches of a layer's projection over rows_a rows and the rows_b rows that ride along: one launch when there are few rows in
// all (weight streaming sets the time: stream them once, not twice) or when the measured costs of the tile shapes say that it
// is no longer than two, in which each range has the shape that suits its height (a ragged total would otherwise pay a
// whole extra round of the tall tiles).  Rows are independent and the K order of an element does not depend on the shape.
RowsPlan plan_gemm_rows(int epi, int rows_a, int rows_b, int N, int K, int ksplit) {
  RowsPlan p = {1, {}};
  float one = 0.f, a_us = 0.f, b_us = 0.f;
  p.range[0] = plan_gemm_layer(epi, rows_a + rows_b, N, K, ksplit, &one);
  if (rows_b == 0 || rows_a + rows_b <= 512) return p;
  const GemmPlan a = plan_gemm_layer(epi, rows_a, N, K, ksplit, &a_us), b = plan_gemm_layer(epi, rows_b, N, K, ksplit, &b_us);
  if (one > a_us + b_us) {
    p.n_ranges = 2;
    p.range[0] = a;
    p.range[1] = b;
  }
  return p;
}

bool plan_has_kernels(int epi, const GemmPlan& p) {
  if (p.n_parts < 1) return false;
  for (int i = 0; i < p.n_parts; ++i) {
    const int bm = p.part[i].bm, bn = p.part[i].bn;
    if (epi == EPI_RESID ? bm != 256 || (bn != 128 && bn != 64) : !has_shape(epi, bm, bn)) return false;
  }
  return true;
}

hipError_t launch_gemm_plan(int epi, const GemmArgs& a0, const GemmPlan& p, hipStream_t st) {
  GemmArgs a = a0;
  if (a.ksplit < 1) a.ksplit = 1;
  if (p.n_parts < 1) return hipErrorInvalidValue;
  const TileShape t = {p.part[0].bm, p.part[0].bn};
  switch (epi) {
    case EPI_STORE:
      return launch_gemm_store(a, t, st);
    case EPI_QKV:
      return launch_gemm_qkv(a, t, st);
    case EPI_RESID:
      if (t.bn == 64) return launch_t<EPI_RESID, 64, 4>(a, cdiv(a.M, BM), a.N / 64, st);
      return launch_t<EPI_RESID, 128, 4>(a, cdiv(a.M, BM), a.N / 128, st);
    case EPI_PARTIAL:
      return launch_gemm_partial(a, t, st);
    case EPI_SWIGLU: {
      const size_t ldw = a.ldw ? a.ldw : a.K;
      for (int i = 0; i < p.n_parts; ++i) {
        GemmArgs g = a;
        g.N = p.part[i].ncols;
        g.W[0] = (const bf16_t*)a.W[0] + (size_t)p.part[i].col0 * ldw;
        g.W[1] = (const bf16_t*)a.W[1] + (size_t)p.part[i].col0 * ldw;
        g.C = (bf16_t*)a.C + p.part[i].col0;
        const hipError_t e = launch_gemm_swiglu(g, TileShape{p.part[i].bm, p.part[i].bn}, st);
        if (e != hipSuccess) return e;
      }
      return hipSuccess;
    }
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_mfma(int epi, const GemmArgs& a0, hipStream_t st) {
  GemmArgs a = a0;
  if (a.ksplit < 1) a.ksplit = 1;
  if (epi == EPI_LMHEAD) return launch_gemm_head(a, st);     // the shape is chosen on the device
  return launch_gemm_plan(epi, a, plan_gemm_mfma(epi, a.M, a.N, a.ksplit), st);
}

hipError_t launch_splitk_reduce(const float* P, int ksplit, const void* R, void* out, const void* gain, float eps,
                                void* normed, int M, int N, hipStream_t st, const int32_t* n_rows_dev,
                                const int32_t* out_rows, const int32_t* r_rows, const HeadRows* head) {
  // 1024 threads per row with few rows, while the row and its (chunk, lane) sums fit the 64 KB a launch gets by default
  const size_t sums = 64 * (size_t)((N + 255) / 256);
  const bool wide_fits = sizeof(float) * (N + sums) <= 64 * 1024;
  const int threads = (N >= 4096 && M <= 512 && (!normed || wide_fits)) ? 1024 : 256;
  const bf16_t *r = (const bf16_t*)R, *g = (const bf16_t*)gain;
  bf16_t *o = (bf16_t*)out, *n = (bf16_t*)normed;
  if (head)
    splitk_reduce_kernel<RED_HEAD><<<M, threads, sizeof(bf16_t) * (size_t)N, st>>>(P, ksplit, r, o, g, eps, n, M, N, n_rows_dev,
                                                                                    out_rows, r_rows, head->row_idx, head->count);
  else if (normed)
    splitk_reduce_kernel<RED_NORM><<<M, threads, sizeof(float) * (N + (threads > 256 ? sums : 0)), st>>>(
        P, ksplit, r, o, g, eps, n, M, N, n_rows_dev, out_rows, r_rows, nullptr, nullptr);
  else
    splitk_reduce_kernel<RED_PLAIN><<<M, threads, 0, st>>>(P, ksplit, r, o, nullptr, 0.f, nullptr, M, N, n_rows_dev, out_rows,
                                                           r_rows, nullptr, nullptr);
  return hipGetLastError();
}

}  // namespace spiffy
