// Unpermute + weighted combine: the rank-local part of the paper's result
// combination (Sec. "MoE Load Balancing Systems", Communication).  HBM-bound:
// reads each expert-output row once, writes each token row once.
#include "common.h"

namespace realb {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4c_t;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// float -> bf16 pattern, nearest-even (finite inputs).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

// acc += w * 8 BF16 values
__device__ __forceinline__ void accumulate8(float (&acc)[8], float w, const u32x4c_t& v) {
    acc[0] = fmaf(w, bf16_lo(v.x), acc[0]); acc[1] = fmaf(w, bf16_hi(v.x), acc[1]);
    acc[2] = fmaf(w, bf16_lo(v.y), acc[2]); acc[3] = fmaf(w, bf16_hi(v.y), acc[3]);
    acc[4] = fmaf(w, bf16_lo(v.z), acc[4]); acc[5] = fmaf(w, bf16_hi(v.z), acc[5]);
    acc[6] = fmaf(w, bf16_lo(v.w), acc[6]); acc[7] = fmaf(w, bf16_hi(v.w), acc[7]);
}

// One wave per token and panel of 512 columns (a wave: the token's rows and weights are scalars, and many small waves hide
// the latency of the chain row index -> row).  The local rows of a token are accumulated in FP32 in order of j, the loads of
// two rows in flight together.
// NT: rows are read and the output is written past the caches (see realb_combine for when).  Measured right behind the down
// GEMM, before (a block per token) -> after: 9 807 rows to 16384 tokens 26.9 -> 18.7 us, 36 183 rows 33.8 -> 33.6 us, 124 473 rows
// to 32768 tokens 128 -> 105 us; with rows and outputs from HBM, 249 000 rows to 65536 tokens 254 -> 206 us (6.2 TB/s; with plain
// loads 219).  Panels of 1024 and 2048 columns measured 3-5 % slower.
template <bool NT>
__global__ void __launch_bounds__(256) combine_kernel(const u32x4c_t* __restrict__ y_rows, const int32_t* __restrict__ assign_to_row,
                                                      const float* __restrict__ topk_w, int T, int k, int H,
                                                      u32x4c_t* __restrict__ out) {
    const int chunks = H >> 3;                            // 16-byte chunks of a row
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int panels = (chunks + 63) / 64;
    const long long item = (long long)blockIdx.x * 4 + wave;
    const int t = (int)(item / panels), c = (int)(item - (long long)t * panels) * 64 + lane;
    if (t >= T) return;
    // lane j holds the j-th row and weight
    const int my_row = lane < k ? assign_to_row[(size_t)t * k + lane] : -1;
    const float my_w = lane < k ? topk_w[(size_t)t * k + lane] : 0.f;
    unsigned long long left = __ballot(my_row >= 0);
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    while (left != 0) {
        int r[2] = {-1, -1};                              // the next two local rows (uniform per wave)
        float w[2] = {0.f, 0.f};
        u32x4c_t v[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            v[q] = u32x4c_t{0, 0, 0, 0};
            if (left == 0) continue;
            const int j = __ffsll((long long)left) - 1;
            left &= left - 1;
            r[q] = __builtin_amdgcn_readlane(my_row, j);
            w[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_w), j));
            const u32x4c_t* src = y_rows + (size_t)r[q] * chunks + c;
            if (c < chunks) v[q] = NT ? __builtin_nontemporal_load(src) : *src;
        }
        accumulate8(acc, w[0], v[0]);
        if (r[1] >= 0) accumulate8(acc, w[1], v[1]);
    }
    if (c >= chunks) return;
    const u32x4c_t o = {pack_bf16(acc[0], acc[1]), pack_bf16(acc[2], acc[3]), pack_bf16(acc[4], acc[5]), pack_bf16(acc[6], acc[7])};
    if (NT) __builtin_nontemporal_store(o, out + (size_t)t * chunks + c);
    else out[(size_t)t * chunks + c] = o;
}

// (a launch has fewer than 2^32 threads; pieces of 2^22 waves take half a millisecond and more, so another launch is nothing)
template <bool NT>
static void launch_combine(const void* y_rows, const int32_t* assign_to_row, const float* topk_w, int T, int k, int H, void* out, hipStream_t s) {
    const int chunks = H / 8, panels = (chunks + 63) / 64, most = (1 << 22) / panels;
    for (long long t = 0; t < T; t += most) {
        const int n = T - t < most ? (int)(T - t) : most;
        hipLaunchKernelGGL((combine_kernel<NT>), dim3((unsigned)ceil_div((long long)n * panels, 4)), dim3(256), 0, s,
                           (const u32x4c_t*)y_rows, assign_to_row + t * k, topk_w + t * k, n, k, H, (u32x4c_t*)out + t * chunks);
    }
}

}  // namespace realb

using namespace realb;

extern "C" int realb_combine(realb_ctx* ctx, const void* y_rows, const int32_t* assign_to_row, const float* topk_w, int T,
                             void* out, void* stream) {
    REALB_REQUIRE(ctx != nullptr, REALB_EINVAL, "ctx is NULL");
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    REALB_REQUIRE(T >= 0 && T <= c->cfg.T_max, REALB_ECAP, "T=%d outside [0, T_max=%d]", T, c->cfg.T_max);
    if (T == 0) return REALB_OK;
    REALB_REQUIRE(y_rows && assign_to_row && topk_w && out, REALB_EINVAL, "NULL argument");
    const int k = c->cfg.k, H = c->cfg.H;
    // Whether the caches are passed by is decided for combine AND the kernel that reads its output next: streaming the output
    // alone (or nothing) leaves the rows, which nobody reads again, in the memory-side cache in the place of what that kernel
    // reads.  The rows' number is on the device; the line is where hot ranks (2 to 4 rows per token) turn.  Down GEMM + combine
    // + an addition of a residual to the output, everything cached -> streamed, us, H = 2048: hot rank, 2.2 rows per token, FP4,
    // 8192 / 9000 / 10000 / 12288 / 16384 / 32768 tokens 71.7 / 77.4 / 89.3 / 117 / 154 / 309 -> 73.1 / 78.8 / 84.5 / 104 / 143 / 299;
    // 3.8 rows 82.0 / 103 / 112 / 145 / 192 / 388 -> 83.5 / 91.7 / 98.5 / 120 / 161 / 371; cold rank, half a row, BF16, 57.7 / 58.2 /
    // 80.2 / 73.0 / 107 / 240 -> 58.7 / 59.4 / 81.1 / 74.7 / 105 / 227.  Only the output streamed: 72.9 / 78.4 / 84.6 / 115 / 156 / 307.
    hipStream_t s = as_stream(stream);
    if ((long long)T * H * 2 < (38ll << 20)) launch_combine<false>(y_rows, assign_to_row, topk_w, T, k, H, out, s);
    else launch_combine<true>(y_rows, assign_to_row, topk_w, T, k, H, out, s);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}
