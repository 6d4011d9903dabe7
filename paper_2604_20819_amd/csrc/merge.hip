// Recomposition (App. A.1): the max-shifted merge of Eq. "merge" of a launch
// group's task statistics (acc_i, m_i, l_i, lt_i) into the global
// accumulator, fused with the finalisation O = acc / lt, LSE = m + log l
// after the last group (l sums the fp32 weights, lt the rounded weights the
// inner kernel's P.V product consumed; both merge with the same factors).
//
// Gather form: every work group owns kCombinePairs consecutive (token, head)
// pairs of one elementary segment and one batch element.  A segment lies
// inside one run of each task that holds it, so each contribution is a
// contiguous slab of the task's statistics; the work group reads every
// contribution (and the running global state when an earlier group touched
// these tokens), merges in registers and writes each output once.  Work
// groups own disjoint tokens, so the merge needs no atomics and no ordering
// between tasks of the group.
//
// Statistics are in the log2 domain with integer-valued maxima (the inner
// kernels round running maxima up to integers), so every factor
// 2^(m_i - m') is an exact power of two.  A task row with no kept key carries
// m_i = -inf and l_i = lt_i = 0: a null contribution with factor 0.
#include "hip_common.hpp"
#include "kernels.hpp"

namespace cqsa {

// Segment of work group blk: the last one with blk0 <= blk (segment 0 starts at
// 0).  Each lane of a wave tests one segment, or, of more than 64, the first of
// every ceil(n / 64) and then those of the part found: one load up to 64
// segments (7 at depth 1 with c = 7, about 40 at depth 2), two up to 4096 (190
// at depth 3, 900 at depth 4), where a binary search is a chain of 3, 6, 8 and
// 10 dependent loads and a walk by 64 at depth 4 one of up to 15 (bf16 L =
// 16384, H = 1, d = 32, depth 4: the forward's 76 merges 1.41 ms by binary
// search, 1.11 by the walk, 1.06 now).
__device__ __forceinline__ int find_segment(const DevSeg* segs, int n_seg, int64_t blk) {
  const int lane = lane_id();
  int at = 0, n = n_seg;  // the segment is one of at .. at + n - 1
  while (n > 1) {
    const int step = (n + 63) >> 6;
    const bool in = lane * step < n;
    const uint64_t m = __builtin_amdgcn_ballot_w64(in && segs[in ? at + lane * step : 0].blk0 <= blk);
    const int k = m == 0ull ? 0 : 63 - __builtin_clzll(m);
    at += k * step;
    n = n - k * step < step ? n - k * step : step;
  }
  return __builtin_amdgcn_readfirstlane(at);
}

// Contributions read at once: their loads are issued together, so that a
// short merge waits for one memory latency per batch and not per
// contribution (a token lies in 3 tasks at depth 1 with c = 7).
constexpr int kMergeBatch = 4;

// Short merges are a chain of memory latencies (segment, contributions,
// statistics, rows), long ones run at HBM rate.  Statistics in batches against
// a binary search and one contribution at a time: f32 L = 1024, H = 1, d = 64
// 7.2 -> 5.6 us; bf16 L = 5000, H = 4, d = 96 at depth 2 19.8 -> 15.3 us; bf16
// L = 32768, H = 16, d = 128 226 -> 197 us for 1.09 GB (5.5 TB/s).
template <int D>
__global__ void __launch_bounds__(256) combine_kernel(const CombineArgs a) {
  constexpr int P = kCombinePairs;
  constexpr int F4 = D / 4;            // float4 per (token, head)
  constexpr int NF = P * F4 / 256;     // float4 per thread
  constexpr int U = kMergeBatch;
  static_assert(P * F4 % 256 == 0, "combine tiling");
  __shared__ float fac_s[kMaxContrib + 1][P];
  __shared__ float inv_s[P];

  const int tid = threadIdx.x;
  const int b = blockIdx.y;
  const int64_t blk = blockIdx.x;
  const DevSeg sg = a.segs[find_segment(a.segs, a.n_seg, blk)];
  const int H = a.H;
  const int64_t pair0 = (blk - sg.blk0) * P;        // first pair within the segment
  const int64_t npair64 = sg.len * H - pair0;
  const int npair = npair64 < P ? int(npair64) : P;
  const int nc = sg.n_c < kMaxContrib ? sg.n_c : kMaxContrib;  // the planner caps n_c
  const bool glob = sg.has_global != 0;
  const DevContrib* cons = a.contribs + sg.c_off;

  // merge factors of each pair (one thread per pair)
  if (tid < npair) {
    const int64_t pr = pair0 + tid;
    const int64_t r = pr / H;
    const int h = int(pr % H);
    const int64_t gi = (int64_t(b) * H + h) * a.L + sg.g0 + r;
    float mg = -INFINITY, lg = 0.f, ltg = 0.f;
    if (glob) {
      mg = a.m[gi];
      lg = a.l[gi];
      ltg = a.lt[gi];
    }
    auto stat = [&](int k) {
      const DevContrib c = cons[k];
      return c.j * a.st_stride + (int64_t(b) * H + h) * c.len + c.local_start + r;
    };
    float mk[U], lk[U], ltk[U];
    auto batch = [&](int k0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        mk[u] = -INFINITY;
        lk[u] = ltk[u] = 0.f;
        if (k0 + u < nc) {
          const int64_t si = stat(k0 + u);
          mk[u] = a.m_i[si];
          lk[u] = a.l_i[si];
          ltk[u] = a.lt_i[si];
        }
      }
    };
    float mx = mg;
    int k0 = (nc - 1) / U * U;  // the last batch first: the sums start with batch 0
    for (; k0 >= 0; k0 -= U) {
      batch(k0);
#pragma unroll
      for (int u = 0; u < U; ++u) mx = fmaxf(mx, mk[u]);
    }
    const float fg = mg == -INFINITY ? 0.f : fast_exp2(mg - mx);
    float lsum = lg * fg, ltsum = ltg * fg;
    fac_s[0][tid] = fg;
    for (k0 = 0; k0 < nc; k0 += U) {
      if (k0 > 0) batch(k0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (k0 + u >= nc) break;
        const float f = mk[u] == -INFINITY ? 0.f : fast_exp2(mk[u] - mx);
        lsum += lk[u] * f;
        ltsum += ltk[u] * f;
        fac_s[k0 + u + 1][tid] = f;
      }
    }
    if (a.final) {
      inv_s[tid] = 1.f / ltsum;
      a.m[gi] = (mx + __log2f(lsum)) * 0.69314718055994530942f;
    } else {
      inv_s[tid] = 1.f;
      a.m[gi] = mx;
      a.l[gi] = lsum;
      a.lt[gi] = ltsum;
    }
  }
  __syncthreads();

  // stream the (token, head) rows: contiguous in the global tensor and in
  // every contribution, 16 bytes per thread per pass (one contribution at a
  // time: with two or more of them in registers long merges slow down, 276
  // against 226 us at bf16 L = 32768, H = 16, d = 128)
  const int64_t row_g = (int64_t(b) * a.L + sg.g0) * H;  // pair index of token g0, head 0
  f32x4 acc[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int f = tid + 256 * i, p = f / F4;
    acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (glob && p < npair) {
      const f32x4 x = *(const f32x4*)(a.acc + (row_g + pair0 + p) * D + (f % F4) * 4);
      acc[i] = x * fac_s[0][p];
    }
  }
  for (int k = 0; k < nc; ++k) {
    const DevContrib c = cons[k];
    const float* src = a.acc_i + c.j * a.acc_stride +
                       ((int64_t(b) * c.len + c.local_start) * H + pair0) * D;
    f32x4 x[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const int f = tid + 256 * i, p = f / F4;
      x[i] = p < npair ? *(const f32x4*)(src + int64_t(p) * D + (f % F4) * 4)
                       : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const int p = (tid + 256 * i) / F4;
      if (p < npair) acc[i] += x[i] * fac_s[k + 1][p];
    }
  }
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int f = tid + 256 * i, p = f / F4;
    if (p < npair)
      *(f32x4*)(a.acc + (row_g + pair0 + p) * D + (f % F4) * 4) = acc[i] * inv_s[p];
  }
}

// Gradient recomposition of a launch group: every (token, head) row of dQ,
// dK and dV is the sum of the group's task-local rows that hold the token, in
// task order, added to the running value when an earlier group touched the
// token (task gradients add: each kept pair belongs to one task).  Work
// groups own kCombinePairs consecutive (token, head) pairs of one segment and
// batch element, as in the combine; the rows are contiguous in every buffer,
// 16 bytes per thread per pass.
// blockIdx.z is the gradient: with the three in turn, a short merge waited for
// each one's rows.  bf16 L = 3000, H = 4, d = 128: 29.8 -> 14.2 us; L = 5000,
// H = 4, d = 96 at depth 2: 61.5 -> 22.6 us; L = 32768, H = 16, d = 128: 617 ->
// 580 us for 3.22 GB (5.6 TB/s).
template <int D>
__global__ void __launch_bounds__(256) grad_merge_kernel(const GradMergeArgs a) {
  constexpr int P = kCombinePairs;
  constexpr int F4 = D / 4;
  constexpr int NF = P * F4 / 256;
  constexpr int UR = NF <= 4 ? kMergeBatch : NF <= 8 ? 2 : 1;  // rows of a batch that fit in registers
  static_assert(P * F4 % 256 == 0, "merge tiling");
  const int tid = threadIdx.x;
  const int b = blockIdx.y, t = blockIdx.z;
  const int64_t blk = blockIdx.x;
  const DevSeg sg = a.segs[find_segment(a.segs, a.n_seg, blk)];
  const int H = a.H;
  const int64_t pair0 = (blk - sg.blk0) * P;
  const int64_t npair64 = sg.len * H - pair0;
  const int npair = npair64 < P ? int(npair64) : P;
  const int nc = sg.n_c < kMaxContrib ? sg.n_c : kMaxContrib;
  const bool glob = sg.has_global != 0;
  const int64_t row_g = (int64_t(b) * a.L + sg.g0) * H + pair0;  // first pair's row
  float* dst = a.dst[t] + row_g * D;
  f32x4 acc[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int f = tid + 256 * i, p = f / F4;
    acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (glob && p < npair) acc[i] = *(const f32x4*)(dst + int64_t(p) * D + (f % F4) * 4);
  }
  for (int k0 = 0; k0 < nc; k0 += UR) {
    f32x4 x[UR][NF];
#pragma unroll
    for (int u = 0; u < UR; ++u) {
      if (k0 + u >= nc) break;
      const DevContrib c = a.contribs[sg.c_off + k0 + u];
      const float* src = a.src[t] + c.j * a.stride + ((int64_t(b) * c.len + c.local_start) * H + pair0) * D;
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        const int f = tid + 256 * i, p = f / F4;
        x[u][i] = p < npair ? *(const f32x4*)(src + int64_t(p) * D + (f % F4) * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int u = 0; u < UR; ++u) {
      if (k0 + u >= nc) break;
#pragma unroll
      for (int i = 0; i < NF; ++i) acc[i] += x[u][i];
    }
  }
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const int f = tid + 256 * i, p = f / F4;
    if (p < npair) *(f32x4*)(dst + int64_t(p) * D + (f % F4) * 4) = acc[i];
  }
}

// fp32 result rounded to a 16-bit output dtype (nearest even): 8 elements
// per thread, one 32-byte read and one 16-byte write.
template <typename T>
__global__ void __launch_bounds__(256) cast_out_kernel(const float* __restrict__ src,
                                                       T* __restrict__ dst, int64_t n) {
  const int64_t i = (int64_t(blockIdx.x) * 256 + threadIdx.x) * 8;
  if (i + 8 <= n) {
    const f32x4 x0 = *(const f32x4*)(src + i), x1 = *(const f32x4*)(src + i + 4);
    typedef __attribute__((__vector_size__(8 * sizeof(T)))) T t8;
    t8 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      y[e] = (T)x0[e];
      y[4 + e] = (T)x1[e];
    }
    *(t8*)(dst + i) = y;
  } else {
    for (int64_t k = i; k < n; ++k) dst[k] = (T)src[k];
  }
}

hipError_t launch_cast_out(const float* src, void* dst, int64_t n, cqsa_dtype dt, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 2047) / 2048;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  if (dt == CQSA_BF16)
    hipLaunchKernelGGL(cast_out_kernel<__bf16>, dim3(unsigned(blocks)), dim3(256), 0, s, src,
                       (__bf16*)dst, n);
  else if (dt == CQSA_F16)
    hipLaunchKernelGGL(cast_out_kernel<_Float16>, dim3(unsigned(blocks)), dim3(256), 0, s, src,
                       (_Float16*)dst, n);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_combine(const CombineArgs& a, int64_t blocks, hipStream_t s) {
  if (blocks <= 0 || a.B <= 0) return hipSuccess;
  if (a.n_seg < 1 || blocks > 0x7fffffff || a.B > 65535) return hipErrorInvalidValue;
  const dim3 grid(unsigned(blocks), unsigned(a.B));
  switch (a.d) {
    case 32: hipLaunchKernelGGL(combine_kernel<32>, grid, dim3(256), 0, s, a); break;
    case 64: hipLaunchKernelGGL(combine_kernel<64>, grid, dim3(256), 0, s, a); break;
    case 96: hipLaunchKernelGGL(combine_kernel<96>, grid, dim3(256), 0, s, a); break;
    case 128: hipLaunchKernelGGL(combine_kernel<128>, grid, dim3(256), 0, s, a); break;
    case 160: hipLaunchKernelGGL(combine_kernel<160>, grid, dim3(256), 0, s, a); break;
    case 192: hipLaunchKernelGGL(combine_kernel<192>, grid, dim3(256), 0, s, a); break;
    case 224: hipLaunchKernelGGL(combine_kernel<224>, grid, dim3(256), 0, s, a); break;
    case 256: hipLaunchKernelGGL(combine_kernel<256>, grid, dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace cqsa

namespace cqsa {

hipError_t launch_grad_merge(const GradMergeArgs& a, int64_t blocks, hipStream_t s) {
  if (blocks <= 0 || a.B <= 0) return hipSuccess;
  if (a.n_seg < 1 || blocks > 0x7fffffff || a.B > 65535) return hipErrorInvalidValue;
  const dim3 grid(unsigned(blocks), unsigned(a.B), 3);
  switch (a.d) {
    case 32: hipLaunchKernelGGL(grad_merge_kernel<32>, grid, dim3(256), 0, s, a); break;
    case 64: hipLaunchKernelGGL(grad_merge_kernel<64>, grid, dim3(256), 0, s, a); break;
    case 96: hipLaunchKernelGGL(grad_merge_kernel<96>, grid, dim3(256), 0, s, a); break;
    case 128: hipLaunchKernelGGL(grad_merge_kernel<128>, grid, dim3(256), 0, s, a); break;
    case 160: hipLaunchKernelGGL(grad_merge_kernel<160>, grid, dim3(256), 0, s, a); break;
    case 192: hipLaunchKernelGGL(grad_merge_kernel<192>, grid, dim3(256), 0, s, a); break;
    case 224: hipLaunchKernelGGL(grad_merge_kernel<224>, grid, dim3(256), 0, s, a); break;
    case 256: hipLaunchKernelGGL(grad_merge_kernel<256>, grid, dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

__global__ void __launch_bounds__(64) zero_u64_kernel(unsigned long long* p, int n) {
  const int i = threadIdx.x;
  if (i < n) p[i] = 0ull;
}

hipError_t launch_zero_u64(unsigned long long* p, int n, hipStream_t s) {
  if (n <= 0 || n > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace cqsa
