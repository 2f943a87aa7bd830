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
// NT_STORE: the output is written past the caches; for outputs that would not stay there for their reader, which are also
// those long enough for the write-back of dirty lines at the kernel's end to cost.  NT_LOAD: so are the rows read, for rows
// that the memory-side cache (256 MB) cannot have kept.  Measured right behind the down GEMM, before (a block per token) ->
// after: 9 807 rows to 16384 tokens 26.9 -> 18.7 us, 36 183 rows 33.8 -> 33.6 us, 124 473 rows to 32768 tokens 128 -> 105 us;
// with rows and outputs from HBM, 249 000 rows to 65536 tokens 254 -> 206 us (6.2 TB/s; with plain loads 219).  Panels of
// 1024 and 2048 columns measured 3-5 % slower.
template <bool NT_LOAD, bool NT_STORE>
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
            if (c < chunks) v[q] = NT_LOAD ? __builtin_nontemporal_load(src) : *src;
        }
        accumulate8(acc, w[0], v[0]);
        if (r[1] >= 0) accumulate8(acc, w[1], v[1]);
    }
    if (c >= chunks) return;
    const u32x4c_t o = {pack_bf16(acc[0], acc[1]), pack_bf16(acc[2], acc[3]), pack_bf16(acc[4], acc[5]), pack_bf16(acc[6], acc[7])};
    if (NT_STORE) __builtin_nontemporal_store(o, out + (size_t)t * chunks + c);
    else out[(size_t)t * chunks + c] = o;
}

// (a launch has fewer than 2^32 threads; pieces of 2^22 waves take half a millisecond and more, so another launch is nothing)
template <bool NT_LOAD, bool NT_STORE>
static void launch_combine(const void* y_rows, const int32_t* assign_to_row, const float* topk_w, int T, int k, int H, void* out, hipStream_t s) {
    const int chunks = H / 8, panels = (chunks + 63) / 64, most = (1 << 22) / panels;
    for (int t = 0; t < T; t += most) {
        const int n = T - t < most ? T - t : most;
        hipLaunchKernelGGL((combine_kernel<NT_LOAD, NT_STORE>), dim3((unsigned)ceil_div((long long)n * panels, 4)), dim3(256), 0, s,
                           (const u32x4c_t*)y_rows, assign_to_row + (size_t)t * k, topk_w + (size_t)t * k, n, k, H,
                           (u32x4c_t*)out + (size_t)t * chunks);
        if (T - t <= most) break;                         // (t + most may not fit)
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
    // the rows' number is on the device; a rank that is worth an FP4 path has about two per token
    const long long out_bytes = (long long)T * H * 2;
    hipStream_t s = as_stream(stream);
    if (out_bytes < (32ll << 20)) launch_combine<false, false>(y_rows, assign_to_row, topk_w, T, k, H, out, s);
    else if (out_bytes < (96ll << 20)) launch_combine<false, true>(y_rows, assign_to_row, topk_w, T, k, H, out, s);
    else launch_combine<true, true>(y_rows, assign_to_row, topk_w, T, k, H, out, s);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}
