// What the GEMV (gemv.hip) and the matrix-core GEMM (gemm.h) share: the
// parameters of a call, page lookups, buffer resources, and the host side of
// a launch.
#pragma once
#include "gemm_plan.h"
#include "runtime.h"

namespace bst {
namespace gv {

constexpr int64_t kPageElems = static_cast<int64_t>(kPage / 2);

struct GemvParams {
  const char* const* page_table;
  const uint8_t* tiers;  // tier of every page
  const int32_t* hbm_pages;
  const int32_t* host_pages;
  // the same in closed form where the tensor's map is modulo placement:
  // page p is on host iff (p / lay_SP) % lay_M == lay_M - 1 (lay_M = 0: no
  // host page), each tier's pages sit in page order in one slab; lay_M < 0:
  // read the tables
  const char* hbm_base;
  const char* host_base;
  int lay_M;
  int lay_SP;
  int n_pages;
  int n_hbm_pages;
  int n_host_pages;
  int units_per_page;
  int host_workers;
  int address_order;
  int N;
  int K;
  const uint16_t* x;
  void* y;
  int y_bf16;
  int B;     // batch rows of x and y
  int join;  // 1: a cut row between two pages of one tier is summed by one unit
  int tail_first;  // 1: the last unit of every page is dispatched before the others
  int S;     // K slices per row group (matrix-core path; 1 = no split)
  int parts;    // partial sums of a row (blocks of all slices; matrix-core GEMM)
  int w_once;   // 1: no two column stages of W share a 128-byte line (streaming loads)
  int vec_out;  // 1: four consecutive outputs of a batch row may go out in one store
  float* ws;  // S > 1 (16-byte aligned): [S][B][N] partials, then [(n_pages + 1) * 2][S][B] of cut rows
  float* partial;  // [(n_pages + 1) boundaries][2 sides][kMaxGemvBatch]
  // host side only: a caller's buffer for the K slices (the layout of ws,
  // summed by the consumer instead of split_reduce) and its size in floats
  float* slices;
  int64_t slice_floats;
};

// Page lookups: the closed form of modulo placement where the tensor has it
// (no dependent load before a unit's first weight load), else the tables.
__device__ __forceinline__ const char* page_addr(const GemvParams& P, int p) {
  if (P.lay_M < 0) return P.page_table[p];
  if (P.lay_M == 0) return P.hbm_base + static_cast<int64_t>(p) * kPage;
  const int g = p / P.lay_SP, before = g / P.lay_M;  // host superpages before g's group
  if (g % P.lay_M == P.lay_M - 1)
    return P.host_base + (static_cast<int64_t>(before) * P.lay_SP + p % P.lay_SP) * kPage;
  return P.hbm_base + (static_cast<int64_t>(p) - static_cast<int64_t>(before) * P.lay_SP) *
                          kPage;
}
__device__ __forceinline__ uint8_t page_tier(const GemvParams& P, int p) {
  if (P.lay_M < 0) return P.tiers[p];
  return P.lay_M > 0 && (p / P.lay_SP) % P.lay_M == P.lay_M - 1 ? BOOST_TIER_HOST
                                                                 : BOOST_TIER_HBM;
}
// the i-th HBM page and the k-th host page in page order
__device__ __forceinline__ int hbm_page(const GemvParams& P, int i) {
  if (P.lay_M < 0) return P.hbm_pages[i];
  if (P.lay_M == 0) return i;
  const int per = (P.lay_M - 1) * P.lay_SP;  // HBM pages of a group of M superpages
  return (i / per) * P.lay_M * P.lay_SP + i % per;
}
__device__ __forceinline__ int host_page(const GemvParams& P, int k) {
  if (P.lay_M < 0) return P.host_pages[k];
  return (k / P.lay_SP) * P.lay_M * P.lay_SP + (P.lay_M - 1) * P.lay_SP + k % P.lay_SP;
}

// Round-to-nearest-even float -> bf16 bits (finite inputs; NaN kept quiet).
__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return 0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

__device__ __forceinline__ void store_y(const GemvParams& P, int b, int64_t row, float v) {
  const int64_t i = static_cast<int64_t>(b) * P.N + row;
  if (P.y_bf16)
    static_cast<uint16_t*>(P.y)[i] = to_bf16(v);
  else
    static_cast<float*>(P.y)[i] = v;
}

// Raw buffer resource over `bytes` bytes at `base` (CDNA: offsets at or past
// num_records read as zero, with no fault).  Word 3 selects 32-bit data.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base,
                                                            uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0,
                                           static_cast<int>(bytes), 0x00020000);
}

// Cache policy of weight loads: 2 = non-temporal (streamed once per token,
// no reuse to keep in L2).
#ifndef BOOST_W_AUX
#define BOOST_W_AUX 2
#endif
template <int AUX = 0>
__device__ __forceinline__ uint4 load16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  auto v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX);
  return *reinterpret_cast<uint4*>(&v);
}

// The same for a base and size the caller knows to be uniform over the
// wavefront: taken through readfirstlane, so the descriptor lives in scalar
// registers even where the compiler cannot prove the uniformity itself
// (otherwise every load through it becomes a loop over distinct descriptors).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc_uniform(const void* base,
                                                                    uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
  const uint32_t n = __builtin_amdgcn_readfirstlane(bytes);
  return make_rsrc(reinterpret_cast<const void*>((static_cast<uint64_t>(hi) << 32) | lo), n);
}

// Offsets at or above this are outside every resource used here (a page is
// 2 MiB, x at most 256 rows of 2^20 elements, 2^29 bytes), so the load returns
// zero.
constexpr uint32_t kOOB = 0x80000000u;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) double f64x4_t;

// Host side of a launch (gemv.hip).
// Rows of the matrix that the page with the most of them meets.
int64_t rows_met(const GemvParams& P, int n_pages);
// Persistent workgroups for host_units units on host pages.
int host_worker_count(const boost_ctx* ctx, int64_t host_units, bool matrix_core);
// The launch after the main one: the parts of rows cut by page boundaries, or
// with P.S > 1 the slices (left to the consumer where it brought a buffer).
int launch_sums(GemvParams& P, int n_pages, bool need_fixup, hipStream_t s);

// The matrix-core GEMM for BT batch tiles of 16 rows (gemm_*.hip).
template <int BT>
int launch_gemm(GemvParams& P, const Route& route, int n_pages, bool need_fixup,
                const boost_ctx* ctx, hipStream_t s);

}  // namespace gv
}  // namespace bst
