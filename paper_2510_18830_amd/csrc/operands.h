// fp16 copies of the attention operands, each times a power of two chosen from
// the tensor's max magnitude (V for the forward; Q, K, V and s dO for the
// backward).  The attention kernels stage every tile as a plain row copy, read
// row-wise or transposed from LDS, and fold the scales back in exactly.  Exact
// for |x| * mul in [2^-14, 65504]; smaller magnitudes round as fp16 subnormals.
//
// Both passes are bound by HBM at large sizes and by launches at small ones, so
// one launch serves every tensor of a call, its workgroups dealt to the tensors
// by their bytes.  The max pass leaves one word per workgroup and the
// conversion's workgroups reduce them again (at most kMaxParts words from L2):
// an atomic per workgroup on one word took 30-60 us at 4096 workgroups, more
// than the reading of a 134 MB tensor.
#pragma once

#include "common.h"

namespace msparse {

constexpr int kCvtThreads = 256;
constexpr int kMaxParts = 2048;     // workgroups of the max pass per tensor
constexpr int kCvtBlocks = 2048;    // workgroups of a conversion launch
constexpr int kCvtUnroll = 4;       // 16-byte loads in flight per thread

// A run of n8 chunks of 8 bf16 values, spread over `nblk` workgroups from
// blk0 on.  max pass: one word per workgroup to part.  conversion: dst =
// fp16(src * mul), mul from the nparts words of part, max |x| * mul in
// [2^(exp-1), 2^exp); *word receives the max.  nparts = 0: no pass ran, and the
// max is the one that an earlier call left in *word (kept) or, for a tensor
// without elements, 0.
struct OperandJob {
    const uint16_t* src;
    uint16_t* dst;
    uint32_t* part;
    uint32_t* word;
    int64_t n8;
    int32_t nparts;
    int32_t blk0, nblk;
    int32_t exp;
    int32_t kept;
};

// Workgroups for a job of `bytes` out of `total` when the launch may have
// `cap`: its share, and no more than leaves every thread one unrolled step.
inline int32_t job_blocks(double bytes, double total, int cap) {
    const double step = double(kCvtThreads) * kCvtUnroll * 16;
    const int64_t share = int64_t(cap * bytes / total) + 1, want = int64_t(bytes / step) + 1;
    return int32_t(share < want ? share : want);
}

__device__ __forceinline__ uint32_t block_max_u32(uint32_t m, uint32_t* sh) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, uint32_t(__shfl_xor(int(m), o)));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    m = 0;
#pragma unroll
    for (int w = 0; w < kCvtThreads / 64; ++w) m = max(m, sh[w]);
    return m;
}

// max |x| of workgroup `b` of the job's run, as fp32 bits (NaN compares above
// inf: the scale is then 1)
__device__ __forceinline__ void operand_max(const OperandJob& j, int b, uint32_t* sh) {
    const u32x4* src = reinterpret_cast<const u32x4*>(j.src);
    const int64_t stride = int64_t(j.nblk) * kCvtThreads;
    uint32_t m = 0;
    for (int64_t i0 = int64_t(b) * kCvtThreads + threadIdx.x; i0 < j.n8; i0 += kCvtUnroll * stride) {
        u32x4 x[kCvtUnroll];
#pragma unroll
        for (int u = 0; u < kCvtUnroll; ++u) {
            const int64_t i = i0 + u * stride;
            x[u] = src[i < j.n8 ? i : i0];
        }
#pragma unroll
        for (int u = 0; u < kCvtUnroll; ++u) {
            m = max(m, max(max(x[u].x & 0x7fffu, (x[u].x >> 16) & 0x7fffu), max(x[u].y & 0x7fffu, (x[u].y >> 16) & 0x7fffu)));
            m = max(m, max(max(x[u].z & 0x7fffu, (x[u].z >> 16) & 0x7fffu), max(x[u].w & 0x7fffu, (x[u].w >> 16) & 0x7fffu)));
        }
    }
    m = block_max_u32(m, sh);
    if (threadIdx.x == 0) j.part[b] = m << 16;   // bf16 magnitude bits -> fp32 bits
}

// the tensor's max, from the words of the max pass if there was one
__device__ __forceinline__ uint32_t operand_max_word(const OperandJob& j, uint32_t* sh) {
    if (j.nparts == 0) return j.kept ? *j.word : 0u;
    uint32_t m = 0;
    for (int i = threadIdx.x; i < j.nparts; i += kCvtThreads) m = max(m, j.part[i]);
    return block_max_u32(m, sh);
}

__device__ __forceinline__ void operand_convert(const OperandJob& j, int b, uint32_t* sh) {
    const uint32_t mx = operand_max_word(j, sh);
    if (b == 0 && j.nparts > 0 && threadIdx.x == 0) *j.word = mx;
    const float mul = j.exp == kOperandExp ? pow2_scale_to<kOperandExp>(&mx) : pow2_scale(&mx);
    const u32x4* src = reinterpret_cast<const u32x4*>(j.src);
    u32x4* dst = reinterpret_cast<u32x4*>(j.dst);
    const int64_t stride = int64_t(j.nblk) * kCvtThreads;
    for (int64_t i0 = int64_t(b) * kCvtThreads + threadIdx.x; i0 < j.n8; i0 += kCvtUnroll * stride) {
        u32x4 x[kCvtUnroll];
#pragma unroll
        for (int u = 0; u < kCvtUnroll; ++u) {
            const int64_t i = i0 + u * stride;
            x[u] = src[i < j.n8 ? i : i0];
        }
#pragma unroll
        for (int u = 0; u < kCvtUnroll; ++u) {
            const int64_t i = i0 + u * stride;
            u32x4 y;
            y.x = pack_f16x2(bf16_lo(x[u].x) * mul, bf16_hi(x[u].x) * mul);
            y.y = pack_f16x2(bf16_lo(x[u].y) * mul, bf16_hi(x[u].y) * mul);
            y.z = pack_f16x2(bf16_lo(x[u].z) * mul, bf16_hi(x[u].z) * mul);
            y.w = pack_f16x2(bf16_lo(x[u].w) * mul, bf16_hi(x[u].w) * mul);
            if (i < j.n8) dst[i] = y;
        }
    }
}

}  // namespace msparse
