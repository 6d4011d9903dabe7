// Device-side building blocks for the gfx950 (CDNA4) kernels.
//
// MFMA lane layouts used throughout (wave64, v_mfma_f32_32x32x16_{bf16,f16}):
//   A (M x K = 32 x 16): lane l holds row l%32, k = 8*(l/32) .. +8
//   B (K x N = 16 x 32): lane l holds column l%32, k = 8*(l/32) .. +8
//   C/D (32 x 32 fp32):  lane l holds column l%32; register r holds row
//                        8*(r/4) + 4*(l/32) + (r%4)
// ds_read_b64_tr_b16 (LDS transpose read), per group of 16 lanes: lane i of
// the group receives element (i%4) of the 4 x 16-bit words read by source
// lane 4*e + i/4, for e = 0..3.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "records.hpp"

namespace cqsa {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));

typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
typedef __attribute__((address_space(3))) void* lds_ptr;
// Words read through the constant address space: a load at a wave-uniform
// address is then a scalar load (tables that no kernel writes).
typedef const __attribute__((address_space(4))) uint32_t const_u32;

// Input element tags.  kKeptSum: the largest sum of a lane's weights at which a
// tile keeps its row's shift; every weight is at most the sum and has to stay
// finite in the element type (fp16 ends at 65504, and 65520 rounds to infinity).
struct BF16 {
  typedef bf16x8 vec8;
  static constexpr float kKeptSum = 65536.f;
};
struct F16 {
  typedef f16x8 vec8;
  static constexpr float kKeptSum = 32768.f;
};

template <typename E>
__device__ __forceinline__ f32x16 mfma32(const typename E::vec8& a, const typename E::vec8& b,
                                         const f32x16& c);
template <>
__device__ __forceinline__ f32x16 mfma32<BF16>(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
template <>
__device__ __forceinline__ f32x16 mfma32<F16>(const f16x8& a, const f16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Convert 8 fp32 values to a packed 16-bit operand (round to nearest even).
template <typename E>
__device__ __forceinline__ typename E::vec8 pack8(const float* x);
template <>
__device__ __forceinline__ bf16x8 pack8<BF16>(const float* x) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (__bf16)x[i];
  return r;
}
template <>
__device__ __forceinline__ f16x8 pack8<F16>(const float* x) {
  f16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (_Float16)x[i];
  return r;
}

// Running sum of the 8 packed 16-bit values of an MFMA operand, as fp32:
// four dot products with (1, 1) (v_dot2c_f32_{bf16,f16}); the products are
// exact, so this adds exactly the rounded values the product consumes.
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(_Float16)))) _Float16 f16x2;
template <typename E>
__device__ __forceinline__ float sum8(const typename E::vec8& x, float acc);
template <>
__device__ __forceinline__ float sum8<BF16>(const bf16x8& x, float acc) {
  const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bf16x2 p = {x[2 * i], x[2 * i + 1]};
    acc = __builtin_amdgcn_fdot2_f32_bf16(p, one, acc, false);
  }
  return acc;
}
template <>
__device__ __forceinline__ float sum8<F16>(const f16x8& x, float acc) {
  const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f16x2 p = {x[2 * i], x[2 * i + 1]};
    acc = __builtin_amdgcn_fdot2(p, one, acc, false);
  }
  return acc;
}

template <typename V>
__device__ __forceinline__ V bitcast_u4(const u32x4& u) {
  return __builtin_bit_cast(V, u);
}

// Two LDS transpose reads forming one 8-element 16-bit MFMA operand.
template <typename E>
__device__ __forceinline__ typename E::vec8 lds_tr_pair(const char* __restrict__ p0, const char* __restrict__ p1) {
  i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p0);
  i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p1);
  u32x4 u;
  u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
  u[0] = a[0];
  u[1] = a[1];
  u[2] = b[0];
  u[3] = b[1];
  return __builtin_bit_cast(typename E::vec8, u);
}

// LDS row of a K/V tile: d padded up to 64, 128 or 256 elements, so that a
// row holds at least 8 swizzle slots and a 1 KB direct load covers whole rows.
// The padding chunks are loaded (the neighbouring row's bytes, or zero past
// the buffer range) and never read by a product.
template <int D>
constexpr int lds_row_elems() {
  return D <= 64 ? 64 : (D <= 128 ? 128 : 256);
}

// LDS layout of a tile of 16-bit rows (DP elements per row), one layout for
// the two ways the kernels read it: 16-byte row reads (ds_read_b128, lane =
// row, one chunk) and transpose reads (ds_read_b64_tr_b16, four rows by four
// chunks per 32 lanes).  The 64 banks hold 16 chunks of 16 bytes; per cycle
// they serve 16 lanes of a row read or 32 lanes of a transpose read, so both
// run free of conflicts when 16 consecutive rows put one chunk on 16
// different slots and four rows put chunks 4 b .. 4 b + 3 on 16 different
// slots.  Rows of 256 and 512 bytes: chunk c of row r sits in chunk
// c ^ 4 (r mod 4) (of its 16), and every group of 4 rows starts 16 bytes
// later than the rows alone would.  Rows of 128 bytes (two per bank line):
// chunk c sits in chunk c ^ (4 b1 + 2 b2), b1 and b2 the bits 1 and 2 of r,
// and every group of 8 rows starts 16 bytes later.  A tile arrives by direct
// loads of 1 KB (lane i's 16 bytes at + 16 i), whose bases carry the group's
// shift, so the padding costs nothing; and since only two or three bits of
// the chunk vary with the lane, a row's chunks need four per-lane offsets,
// the rest being instruction immediates.  Measured with a probe kernel:
// 4.2 cycles per row read and 2 per transpose read, against 8.1 and 4.1 for a
// swizzle of period 8.
template <int DP>
constexpr int lds_row_off(int r) {
  return DP == 64 ? (r >> 3) * 1040 + (r & 7) * 128
                  : DP == 128 ? (r >> 2) * 1040 + (r & 3) * 256 : (r >> 2) * 2064 + (r & 3) * 512;
}
// Bytes of a tile of `rows` rows (a multiple of 8).
template <int DP>
constexpr int lds_tile_bytes(int rows) {
  return lds_row_off<DP>(rows);
}
// First byte of the q-th 1 KB direct load of a tile (rows q * 1024 / (2 DP) ..).
template <int DP>
constexpr int lds_load_off(int q) {
  return DP == 256 ? (q >> 1) * 2064 + (q & 1) * 1024 : q * 1040;
}
// The chunk of the row that sits in chunk slot `slot` of row r (the swizzle is
// its own inverse), for the per-lane source addresses of the direct loads.
template <int DP>
__device__ __forceinline__ int lds_slot_chunk(int r, int slot) {
  return DP == 64 ? slot ^ (4 * ((r >> 1) & 1) + 2 * ((r >> 2) & 1)) : slot ^ (4 * (r & 3));
}
// Row read of chunk 2 ks + half of row r0 + r (r < 32 the lane's row, r0 a
// multiple of 32): lane part lds_row_lane(r, half, lds_row_var(ks)) plus the
// constant lds_row_imm(r0, ks).
template <int DP>
constexpr int lds_row_var(int ks) {
  return DP == 64 ? ks & 3 : (ks >> 1) & 3;
}
template <int DP>
__device__ __forceinline__ int lds_row_lane(int r, int half, int v) {
  return lds_row_off<DP>(r) + 16 * half +
         (DP == 64 ? 32 * (v ^ (2 * ((r >> 1) & 1) + ((r >> 2) & 1))) : 64 * (v ^ (r & 3)));
}
template <int DP>
constexpr int lds_row_imm(int r0, int ks) {
  return lds_row_off<DP>(r0) + (DP == 64 ? 0 : 32 * (ks & 1) + 256 * (ks >> 3));
}
// Transpose read of 32-column block g, the lane's 8 bytes of row r0 + r (r < 8
// the lane's row, r0 a multiple of 8): lane part lds_tr_lane(r, lane,
// lds_tr_var(g)) plus the constant lds_tr_imm(r0, g).
template <int DP>
constexpr int lds_tr_var(int g) {
  return DP == 64 ? g & 1 : g & 3;
}
template <int DP>
__device__ __forceinline__ int lds_tr_lane(int r, int lane, int v) {
  const int xl = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  return lds_row_off<DP>(r) + 8 * (lane & 1) +
         (DP == 64 ? 64 * (v ^ ((r >> 1) & 1)) + 16 * (xl ^ (2 * ((r >> 2) & 1))) : 64 * (v ^ (r & 3)) + 16 * xl);
}
template <int DP>
constexpr int lds_tr_imm(int r0, int g) {
  return lds_row_off<DP>(r0) + (DP == 64 ? 0 : 256 * (g >> 2));
}
// Keeps a per-lane offset in its register: without it the compiler splits the
// offset into parts and adds them again at every read.
__device__ __forceinline__ void keep_in_register(int& x) { asm volatile("" : "+v"(x)); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// a * b rounded to fp32 on its own: the opaque copy keeps the compiler from
// fusing the product into a following addition (an FMA rounds once), so a sum
// of such products is the same whichever code adds them.
__device__ __forceinline__ float mul_rounded(float a, float b) {
  float t = a * b;
  asm volatile("" : "+v"(t));
  return t;
}

// Value held by lane l^32 (the other half of the wave).
__device__ __forceinline__ float swap_halves(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v),
                                            __builtin_bit_cast(uint32_t, v), false, false);
  uint32_t lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  return __builtin_bit_cast(float, lane < 32 ? r[1] : r[0]);
}

// Raw buffer resource over `rows` rows of a [.., rows, H, d] tensor starting at
// `base` (row pitch `pitch_elems` 16-bit elements, `d` elements per row).  The
// range ends at the last element of row rows-1, so loads of later rows return
// zero (buffer range check) and every address is an SGPR base plus a 32-bit
// per-lane offset.  The last dword selects the raw (untyped) buffer format.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* base, int64_t rows,
                                                           int64_t pitch_bytes, int64_t row_bytes) {
  int64_t bytes = rows > 0 ? (rows - 1) * pitch_bytes + row_bytes : 0;
  if (bytes > 0x7fffffff) bytes = 0x7fffffff;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                           0x00020000);
}

// 16 bytes per lane from a buffer resource straight into LDS: lane i's bytes
// land at lds + 16 i (the wave fills 1 KB); out-of-range reads give zeros.
__device__ __forceinline__ void buf_load16_lds(__amdgpu_buffer_rsrc_t r, void* lds, uint32_t voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voff, 0,
                                           0, 0);
}

// Work-group barrier after this wave's own LDS reads and writes have
// completed (lgkmcnt(0)) that leaves LDS DMA loads (buffer_load ... lds,
// counted by vmcnt) in flight: the compiler's fences would wait for them.
// The caller waits (vmcnt) for the DMA loads the next phase reads.  The
// memory clobber keeps the compiler from moving memory accesses across it.
__device__ __forceinline__ void lds_barrier_dma_in_flight() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ int lane_id() {
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Group bits and global index of a task-local token (runs sorted by local start).
__device__ __forceinline__ uint32_t run_bits(const DevRun* runs, int n, int64_t local) {
  for (int i = 0; i < n; ++i)
    if (local < runs[i].local_start + runs[i].length) return runs[i].bits;
  return 0u;
}
__device__ __forceinline__ int64_t run_global(const DevRun* runs, int n, int64_t local) {
  for (int i = 0; i < n; ++i)
    if (local < runs[i].local_start + runs[i].length)
      return runs[i].global_start + (local - runs[i].local_start);
  return 0;
}

// Tensor row of local token r when the inputs are read in place: from the
// block row table when r's 64-token block lies in one run, else from the runs.
__device__ __forceinline__ int64_t in_place_row(const DevBlock* blks, const DevRun* runs, int n,
                                                int r) {
  const int32_t g = blks[r >> 6].row;
  return g != kNoRow ? int64_t(g) + (r & 63) : run_global(runs, n, r);
}

// Byte offset that every buffer load treats as out of range (resources span
// under 2^31 bytes): such lanes read zero.
constexpr uint32_t kOobOffset = 0x80000000u;

// Task of a work item in a launch over several tasks, whose work items are
// laid out task after task (ceil(L_j / rows) * per_row items for task j).
// Returns j and leaves the item's index within task j in `w`.  Lane i of every
// wave takes task i (a launch has at most 32), so the search is one load and a
// prefix sum over the lanes; a walk over the tasks was a chain of dependent
// loads at the head of every work group (forward of bf16 L = 1000, H = 4, d =
// 128 at depth 2: 134 -> 126 us; of L = 3000 at depth 1: 81.5 -> 80.2 us; long
// launches unchanged).
__device__ __forceinline__ int find_task(const DevTask* tasks, int ntask, int rows,
                                         int64_t per_row, int64_t& w) {
  if (ntask <= 1) return 0;
  static_assert(kMaxContrib <= 64, "one task per lane");
  const int lane = lane_id();
  int64_t n = 0;
  if (lane < ntask) n = ((tasks[lane].L_local + rows - 1) / rows) * per_row;
  int end = int(n);  // a launch has fewer than 2^31 work groups
#pragma unroll
  for (int k = 1; k < 64; k <<= 1) {
    const int up = __shfl_up(end, k);
    if (lane >= k) end += up;
  }
  // tasks that end at or before the item (the last lanes repeat the total)
  const uint64_t m = __builtin_amdgcn_ballot_w64(lane < ntask - 1 && int64_t(end) <= w);
  const int j = __builtin_popcountll(m);
  if (j > 0) w -= __builtin_amdgcn_readlane(end, j - 1);
  return j;
}

// Work-group id remapped so that consecutive work items land on the same XCD
// (the dispatcher deals work groups round-robin over the 8 XCDs, each with its
// own L2): work item w = xcd * per_xcd + slot.
__device__ __forceinline__ int64_t xcd_remap(int64_t id, int64_t n) {
  constexpr int64_t kXcd = 8;
  const int64_t per = n / kXcd, rem = n % kXcd;
  const int64_t xcd = id % kXcd, slot = id / kXcd;
  // the first `rem` XCDs own per+1 items
  const int64_t base = xcd * per + (xcd < rem ? xcd : rem);
  const int64_t cap = per + (xcd < rem ? 1 : 0);
  if (slot < cap) return base + slot;
  return id;  // unreachable when the grid has exactly n groups
}

}  // namespace cqsa
