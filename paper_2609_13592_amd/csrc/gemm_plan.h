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
// units live off their depth), else four of x and up to seven of W, three and
// two of x where it takes 32 KiB a stage.
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
  const int fit = (kDmaLds / kDmaBlk - xs * 2 * bt) / (2 * rows);
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
constexpr GemmShape kGemmShapes[] = {{8, 1}, {8, 2}, {3, 4}, {5, 1}, {4, 1}, {2, 1}, {1, 1}};
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

enum Kernel { kAuto = 0, kGemv = 1, kFewRowsKernel = 2, kGemm = 3 };

struct Route {
  int kernel;
  int shape;  // of kGemmShapes (kGemm)
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

// Picks the unit and the K slices by an estimate of the call's time in us, from
// times of every unit and split of 18 matrices at 8..200 batch rows; the pick
// is within 6 % of the fastest on most of them.  A compute unit passes about
// 45 KiB of stages a us (35 where W's ring has three stages or fewer), W is read at
// 6.8 TB/s at most, a workgroup takes at least `lat` us a stage (its ring over
// the loads' latency, and the barrier), and split sums cost a launch and their
// traffic.  16-row units are for few batch rows only: at more, x's traffic is
// the unit's.
inline Route plan_gemm(const PlanInput& in) {
  const int BT = batch_tiles(in.B);
  const double cu = in.n_cu;
  const uint64_t per = floats_per_slice(in);
  const double hbm = 2e-6 / 6.8 * in.N * in.K;  // us to read W
  double best = 1e30;
  Route r{kGemm, -1, 1};
  for (int i = 0; i < kNumGemmShapes; ++i) {
    const int rtl = kGemmShapes[i].rtl, g = kGemmShapes[i].g;
    const int64_t upp = (in.most + 16 * rtl - 1) / (16 * rtl);
    if ((g > 1 && upp != 1) || (rtl == 1 && BT > 2)) continue;
    const int64_t units = (in.n_pages + g - 1) / g * upp;
    const int occ = gemm_occupancy(BT, rtl, g);
    const double kb = 2 * g * rtl + 2 * BT;  // KiB of a stage
    const double lat = std::max(BT <= 2 && rtl == 5 ? 0.42 : 0.18, 1.5 / gemm_w_stages(BT, g * rtl));
    for (int c = 1; c <= kMaxSlices; c *= 2) {
      if (c > 1 && (in.K / c < 512 || c * per > in.ws_floats)) break;
      const double nst = (in.K / c + 63) / 64, wgs = static_cast<double>(units) * c;
      const double bytes = std::ceil(wgs / cu) * nst * kb / (gemm_w_stages(BT, g * rtl) > 3 ? 45 : 35);
      const double rounds = std::ceil(wgs / (cu * occ));
      const double sums = c > 1 ? 2 + 8e-6 / 4.5 * c * in.B * in.N : 0;
      const double t = std::max({hbm, bytes, rounds * nst * lat}) + rounds * 1.5 + sums;
      if (t < best) best = t, r.shape = i, r.S = c;
    }
  }
  while (r.S > 1 && in.own_slices && r.S * per > in.slice_floats) r.S /= 2;
  return r;
}

// Rows up to which the 16-row kernel takes the matrix-core calls of up to 16
// batch rows (both sides measured: see mfma_kernel).
constexpr int kFewRows = 1200;

inline Route plan_few_rows(const PlanInput& in) {
  // split K until there are two workgroups per CU, in slices of at least 512
  // columns whose partials fit the context's workspace or the caller's buffer
  const int64_t units = in.n_pages * ((in.most + 15) / 16);
  const uint64_t cap = in.own_slices ? in.slice_floats : in.ws_floats;
  Route r{kFewRowsKernel, 0, 1};
  while (r.S < kMaxSlices && units * r.S < 2 * in.n_cu && in.K / (2 * r.S) >= 512) r.S *= 2;
  while (r.S > 1 && r.S * floats_per_slice(in) > cap) r.S /= 2;
  return r;
}

// Whether a call runs on the matrix cores (the others on the GEMV): from four
// batch rows (28672 x 4096 at 4 / 6 rows: 38.1 / 38.1 us against 43.6 / 50.1;
// 4096 x 4096 at 6: 10.9 against 15.5; 5003 x 3080 at 4: 16.4 against 17.3).
// Of 70 drawn matrices of 2^26 elements or more at two and three rows 59 take 3 %
// longer on them or more (49158 x 1976 at 3: 57.8 us against 40.8; 22400 x 7040
// at 2: 81.9 and 57.9), a few less (28672 x 4096 at 2: 38.2 and 41.8).
inline bool matrix_cores(int B) { return B >= 4; }

inline Route plan(const PlanInput& in) {
  if (!matrix_cores(in.B)) return {kGemv, 0, 1};
  if (in.B <= 16 && in.N <= kFewRows) return plan_few_rows(in);
  return plan_gemm(in);
}

// The route asked for, or one with kernel kAuto where the call does not fit it.
inline Route forced_route(const PlanInput& in, const Forced& f) {
  const Route none{kAuto, 0, 0};
  const uint64_t cap = in.own_slices ? in.slice_floats : in.ws_floats;
  if (f.kernel == kGemv) return in.B <= 3 ? Route{kGemv, 0, 1} : none;
  if (f.S > 1 && (in.K / f.S < 512 || f.S * floats_per_slice(in) > cap)) return none;
  if (f.kernel == kFewRowsKernel) return in.B <= 16 ? Route{kFewRowsKernel, 0, f.S} : none;
  for (int i = 0; i < kNumGemmShapes; ++i) {
    const GemmShape u = kGemmShapes[i];
    if (u.rtl != f.row_tiles || u.g != f.pages) continue;
    if ((u.g > 1 && in.most > 16 * u.rtl) || (u.rtl == 1 && batch_tiles(in.B) > 2)) return none;
    return {kGemm, i, f.S};
  }
  return none;
}

}  // namespace gv
}  // namespace bst
