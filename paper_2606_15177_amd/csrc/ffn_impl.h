// Shared definitions of the two expert-FFN GEMM kernels.
#pragma once

#include "common.h"
#include "kernels.h"

namespace moe {

// out[row][n] = epilogue( sum_c x[row][c] * W(g, n, c) ) for every row of
// group g, with W(g, n, c) = w[g*group_stride + col_offset(c) + n*ldw] and
// col_offset(c) = c for a single K segment (kseg >= K) or
// (c / kseg)*seg_stride + c % kseg for K stacked over several experts.
// GATED kernels read two such matrices (w0 = gate, w1 = up) and write
// silu(gate) * up.  x rows have stride K and out rows stride N; row r of the
// grouped activation matrix is x[x_rows[r]] when x_rows != nullptr.
struct GemmArgs {
  const uint16_t* x;
  const int32_t* x_rows;
  int x_row_count;  // rows of x when x_rows is set
  const int32_t* offsets;  // [groups+1] device, or nullptr for one group of static_rows
  int static_rows;
  int groups;
  const uint16_t* w0;
  const uint16_t* w1;
  uint16_t* out;
  int K, N, kseg, ldw;
  size_t seg_stride, group_stride;
};

__device__ __forceinline__ size_t weight_col_offset(const GemmArgs& a, int c) {
  if (a.kseg >= a.K) return static_cast<size_t>(c);
  const int q = c / a.kseg;
  return static_cast<size_t>(q) * a.seg_stride + static_cast<size_t>(c - q * a.kseg);
}

// Immediate of s_waitcnt (gfx9 layout: vmcnt [3:0] and [15:14], expcnt [6:4],
// lgkmcnt [11:8]; a field at its maximum does not wait): at most n vector-
// memory operations in flight, the other counters not waited for.
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// Workgroup barrier that also fences the compiler: no instruction is moved
// across it, and memory accesses stay on their side (the hardware waits are
// the explicit s_waitcnt).
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// 64 lanes x 16 bytes from rs + off[lane] to lds + 16 * lane.
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t rs, unsigned char* lds, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)lds, 16, off, 0, 0, 0);
}

hipError_t launch_skinny(const Segments& seg, const GemmArgs& a, bool gated, hipStream_t st);
// Host-side size limits of the weight-streaming kernel (launch_skinny
// refuses arguments that fail this check).
bool skinny_ok(const GemmArgs& a);
// Its workgroups: 32 output columns of a group each (gated), or 64.
inline long long skinny_blocks(const Segments& seg, const GemmArgs& a, bool gated) {
  return static_cast<long long>(ceil_div(a.N, gated ? 32 : 64)) * seg.groups;
}
// The mid-sized kernel: seg with device offsets, sh (nullable) with static
// rows in the same launch; the caller has checked both (tiled_ok).
hipError_t launch_mid(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated, hipStream_t st);
// Whether a batch of at most kSkinnyMaxRows tokens takes it.
bool mid_streams(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated);
// Its launch: whether narrow items halve K, and its workgroups.
bool mid_splits_k(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated);
long long mid_blocks(const Segments& seg, const GemmArgs& a, const GemmArgs* sh, bool gated);
constexpr int kMidThreads = 4 * kWave;
constexpr long long kMidMaxBlocks = 0xffffffffll / kMidThreads;  // a grid dimension holds 2^32 - 1 threads

// K from which the kernels count a product as long (see the rules that use it).
constexpr int kLongK = 4096;

// Tokens of a decode batch at most (see mid_streams for its kernels).
constexpr int kSkinnyMaxRows = 64;

}  // namespace moe
