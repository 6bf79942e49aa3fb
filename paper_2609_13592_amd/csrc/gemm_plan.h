#pragma once
// Which kernel a call runs on and how it is cut, from the sizes alone: host
// code without HIP, the launches (gemv.hip, gemm.h) and the route query share it.
#include <algorithm>
#include <cmath>
#include <cstdint>

namespace bst {
namespace gv {

constexpr int kDmaBlk = 1024;  // 8 rows x 128 bytes
constexpr int kDmaLds = 163840;  // LDS of a compute unit
// Most K slices a call splits a row group into.
constexpr int kMaxSlices = 8;
// Wavefronts of a workgroup (eight where the products weigh, four otherwise:
// 10240 x 8192 at 8 rows 29.4 us with four, 31.6 with eight; 28672 x 4096 at
// 256 rows 74 us with eight, 82 with four), and the stages of x and of W in
// its rings: 8..16 of both while two workgroups fit a compute unit (small
// units live off their depth), else four of x and up to seven of W, six where
// two workgroups fit then (64-row units at 64 rows: 2048 x 24064 at 42 44.1 us
// with seven and one workgroup), three and two of x where it takes 32 KiB a
// stage.
constexpr int gemm_waves(int bt, int rtl, int g) {
  if (g > 1) return 8;
  if (rtl == 5) return bt == 4 ? 4 : 8;
  return rtl >= 8 ? (bt >= 8 ? 8 : 4) : (bt >= 16 && rtl >= 4 ? 8 : 4);
}
constexpr int gemm_x_stages(int bt, int rows) {
  const int small = 80 / (2 * bt + 2 * rows);
  if (small >= 8) return small < 16 ? small : 16;
  return bt >= 16 ? (rows > 12 ? 2 : 3) : 4;
}
constexpr int gemm_w_stages(int bt, int rows) {
  const int xs = gemm_x_stages(bt, rows);
  if (xs >= 8) return xs;
  const int two = (kDmaLds / kDmaBlk / 2 - xs * 2 * bt) / (2 * rows);
  const int fit = two >= 6 ? two : (kDmaLds / kDmaBlk - xs * 2 * bt) / (2 * rows);
  return fit < 7 ? fit : 7;
}
// A host sub-unit (one row tile) loads W in spans of kSpan stages, 512 bytes of
// a row at a time: the link carries those faster than 128-byte reads (6144 x
// 4096 with one page of 24 on host, 8 rows: 45 us against 59; 57344 x 8192 with
// three of 448: 143 against 156).  Two spans in its ring; three and four took
// 1-9 % longer, the HBM units beside them most.
constexpr int kSpan = 4, kHostSpans = 2;
// Workgroups that a compute unit holds at once.
constexpr int gemm_occupancy(int bt, int rtl, int g) {
  const int rows = g * rtl;
  const int kib = gemm_x_stages(bt, rows) * 2 * bt + gemm_w_stages(bt, rows) * 2 * rows;
  const int lds = kDmaLds / kDmaBlk / kib, waves = 16 / gemm_waves(bt, rtl, g);
  return lds < waves ? lds : waves;
}
// The unit shapes: row tiles of a page, and pages.
struct GemmShape {
  int rtl, g;
};
constexpr GemmShape kGemmShapes[] = {{8, 1}, {8, 2}, {3, 4}, {5, 1}, {4, 1}, {2, 1}};
constexpr int kNumGemmShapes = sizeof kGemmShapes / sizeof *kGemmShapes;


// What a call needs to know to be planned.
struct PlanInput {
  int N, K, B, n_pages;
  int64_t most;           // rows that a page meets at most
  int n_cu;
  uint64_t ws_floats;     // of the context's workspace
  bool own_slices;        // the caller brings the buffer of the slices,
  uint64_t slice_floats;  // of this many floats
};

enum Kernel { kAuto = 0, kGemv = 1, kRows16 = 2, kGemm = 3 };

struct Route {
  int kernel;
  int shape;  // kGemm: index in kGemmShapes; kRows16: row tiles of a unit
  int S;      // K slices
};

// A route asked for instead of the planned one (kernel kAuto: none).
struct Forced {
  int kernel = kAuto, row_tiles = 0, pages = 0, S = 0;
};

// Batch tiles of 16 rows that the GEMM is built for.
inline int batch_tiles(int B) {
  const int t = (B + 15) / 16;
  return t <= 2 ? t : (t <= 4 ? 4 : (t <= 8 ? 8 : 16));
}

inline uint64_t floats_per_slice(const PlanInput& in) {
  return static_cast<uint64_t>(in.B) * (in.N + 2ull * (in.n_pages + 1));
}

// The slices that fit: of the context's workspace first, for its own calls and
// for a caller's buffer alike (so that both sum the same slices), then of that
// buffer.  The unit stays when a caller asks for fewer slices.
inline int fit_slices(const PlanInput& in, int S) {
  const uint64_t per = floats_per_slice(in);
  while (S > 1 && S * per > in.ws_floats) S /= 2;
  while (S > 1 && in.own_slices && S * per > in.slice_floats) S /= 2;
  return S;
}

// The 16-row kernel: one row tile a unit; two, which share x, above 8 rows on
// matrices of 2^25 elements or more (28672 x 4096 at 12: 54.5 -> 50.4 us;
// smaller ones need the workgroups of one: 6144 x 4096 19-27 % longer with
// two).  K is cut until there are two workgroups a compute unit, and while a
// slice is longer than 8192 columns (of 94 matrices of longer rows 11 % took 6 %
// longer without it than with the kernels before, 6 % with it), in slices of at
// least 512.
inline Route plan_rows16(const PlanInput& in) {
  const int rt = in.B > 8 && static_cast<int64_t>(in.N) * in.K >= (int64_t{1} << 25) ? 2 : 1;
  const int64_t units = in.n_pages * ((in.most + 16 * rt - 1) / (16 * rt));
  int S = 1;
  while (S < kMaxSlices && in.K / (2 * S) >= 512 &&
         (units * S < 2 * in.n_cu || in.K / S > 8192))
    S *= 2;
  return {kRows16, rt, fit_slices(in, S)};
}

// The estimates: a call's time in us but for what every kernel takes, fitted to
// the times of every unit and split of 2600 matrices at 4..256 batch rows (300..
// 60000 rows of 512..28800 columns drawn over their logarithm, and the layers of
// the 8B and 70B models).  The pick takes 0.6 % longer than the fastest in the
// mean (3 % up to 16 rows), 5 % at the 95th percentile (13 %).
//
// What a workgroup of the GEMM takes, with one batch tile and with more (W is
// the stream then, or W and x are): W's rate (TB/s) and the lines that ragged
// rows read more; the stages' rate (KiB a us and compute unit) and barrier; the
// least time of a stage, and the time that W's and x's ring cover; the least with
// five row tiles at up to two batch tiles, where three of eight wavefronts have
// none; beginning and end, and more where no other workgroup of the compute unit
// works meanwhile; the sums' launch (us) and traffic (us a MiB of slices), and
// the launch that joins cut rows.
struct GemmCost {
  double hbm, ragged, barrier, stage, w_ring, x_ring, stage5, begin, alone, split, slices, cut;
};
constexpr GemmCost kOneTile{7.3, 1.55, 0.045, 0.29, 0, 0, 0.55, 3.4, 1.5, 1.6, 4.2, 2.6};
constexpr GemmCost kMoreTiles{7.26, 1.18, 0.027, 0.27, 2.44, 1.37, 0.4, 2.43, 2.27, 2.1, 4.5, 1.9};

inline double sums_us(const PlanInput& in, int S, const GemmCost& c) {
  if (S > 1) return c.split + c.slices * S * 1e-6 * in.B * in.N;
  return in.n_pages > 1 && (int64_t{1} << 20) % in.K != 0 ? c.cut : 0;
}

// Units of `rows` rows of each of g pages that hold rows: one more than the
// compute units is a round more, so those of the last page are counted (28187 x
// 1584 at 144 rows, 128-row units: 256 of 258 places, 51.7 us; 66 with the
// 64-row units that seemed faster).
inline int64_t units_of(const PlanInput& in, int rows, int g) {
  if (g > 1) return (in.n_pages + g - 1) / g;
  const int64_t page = int64_t{1} << 20, total = static_cast<int64_t>(in.N) * in.K;
  const int64_t last = (total - 1) / in.K - (in.n_pages - 1) * page / in.K + 1;
  return (in.n_pages - 1) * ((in.most + rows - 1) / rows) + (last + rows - 1) / rows;
}

inline double rows16_us(const PlanInput& in, const Route& r) {
  const int64_t units = units_of(in, 16, 1);
  // three workgroups a compute unit; a wavefront takes chunks of 256 columns
  const double chunks = std::ceil(in.K / (4. * r.S) / 256);
  const double rounds = std::ceil(static_cast<double>(units) * r.S / (3 * in.n_cu));
  return std::max(2e-6 / 2.6 * in.N * in.K, rounds * (2.6 + 2.4 * chunks)) +
         sums_us(in, r.S, kOneTile);
}

inline double gemm_us(const PlanInput& in, int shape, int S) {
  const int BT = batch_tiles(in.B), rtl = kGemmShapes[shape].rtl, g = kGemmShapes[shape].g;
  const GemmCost& c = BT == 1 ? kOneTile : kMoreTiles;
  const int64_t units = units_of(in, 16 * rtl, g);
  const int occ = gemm_occupancy(BT, rtl, g), ring = gemm_w_stages(BT, g * rtl);
  const bool ragged = in.K % 64 != 0;
  const double wgs = static_cast<double>(units) * S, nst = (in.K / S + 63) / 64;
  const double rounds = std::ceil(wgs / (in.n_cu * occ));
  const double kib = 2 * g * rtl * (ragged ? 1.3 : 1) + 2 * BT;  // of a stage
  const double rate = BT == 1 ? 46 : (ring <= 3 ? 39 : (BT == 2 ? 47 : 51));
  const double stages = std::ceil(wgs / in.n_cu) * nst * (kib / rate + c.barrier);
  double stage = std::max({c.stage, c.w_ring / ring, c.x_ring / gemm_x_stages(BT, g * rtl)});
  if (BT <= 2 && rtl == 5) stage = std::max(stage, c.stage5);
  const double hbm = 2e-6 / c.hbm * (ragged ? c.ragged : 1) * in.N * in.K;
  return std::max({hbm, stages, rounds * nst * stage}) +
         rounds * (c.begin + (occ == 1 ? c.alone : 0)) + 0.65 + sums_us(in, S, c);
}

// The unit and the K slices with the least estimate.  Units without sums in
// blocks (see gemm.h) are left to matrices that need no more slices than theirs
// to fill the compute units, so that no row is summed in one longer chain than
// a smaller unit would.
inline Route plan_gemm(const PlanInput& in) {
  const int BT = batch_tiles(in.B);
  double best = 1e30;
  Route r{kGemm, -1, 1};
  for (int i = 0; i < kNumGemmShapes; ++i) {
    const int rtl = kGemmShapes[i].rtl, g = kGemmShapes[i].g;
    if (g > 1 && in.most > 16 * rtl) continue;
    for (int c = 1; c <= kMaxSlices; c *= 2) {
      if (c > 1 && (in.K / c < 512 || c * floats_per_slice(in) > in.ws_floats)) break;
      if (BT == 16 && g > 1 && c < kMaxSlices &&
          (static_cast<int64_t>(in.n_pages) * c < in.n_cu * 3 / 4 || in.K / c > 16384))
        continue;
      const double t = gemm_us(in, i, c);
      if (t < best) best = t, r.shape = i, r.S = c;
    }
  }
  r.S = fit_slices(in, r.S);
  return r;
}

// Up to 3 batch rows the GEMV (of 70 matrices of 2^26 elements or more at 2 and
// 3 rows 59 took 3 % longer or more on the matrix cores, by the GEMM's estimate:
// 49158 x 1976 at 3 40.8 -> 57.8 us, though 28672 x 4096 at 2 41.8 -> 38.2;
// smaller ones lose to the split sums' launch).  Up to 16 rows that are no
// multiple of a cache line take the 16-row kernel, which reads 512 bytes of a
// row at once where the GEMM reads 128 (7259 x 2848 at 8: 17.8 us against 20.1;
// 52515 x 2040 at 4: 47.7 against 60.2); of the others those that it is
// estimated to be faster on, which have few units (1278 x 784 at 10: 4.4 us
// against 7.8; 28672 x 4096 at 8: 48 against 42).
inline Route plan(const PlanInput& in) {
  if (in.B <= 3) return {kGemv, 0, 1};
  if (in.B > 16) return plan_gemm(in);
  const Route rows = plan_rows16(in);
  if (in.K % 64 != 0) return rows;
  const Route gemm = plan_gemm(in);
  return rows.shape == 1 && rows16_us(in, rows) < gemm_us(in, gemm.shape, gemm.S) ? rows : gemm;
}

// The route asked for, or one with kernel kAuto where the call does not fit it.
inline Route forced_route(const PlanInput& in, const Forced& f) {
  const Route none{kAuto, 0, 0};
  if (f.kernel == kGemv) return in.B <= 3 ? Route{kGemv, 0, 1} : none;
  if (f.S > 1 && (in.K / f.S < 512 || fit_slices(in, f.S) != f.S)) return none;
  if (f.kernel == kRows16) return in.B <= 16 ? Route{kRows16, f.row_tiles, f.S} : none;
  for (int i = 0; i < kNumGemmShapes; ++i) {
    const GemmShape u = kGemmShapes[i];
    if (u.rtl != f.row_tiles || u.g != f.pages) continue;
    if (u.g > 1 && in.most > 16 * u.rtl) return none;
    return {kGemm, i, f.S};
  }
  return none;
}

}  // namespace gv
}  // namespace bst
