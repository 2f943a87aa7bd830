// Encoding work that rides along in another kernel's launch, and the precision rule as device code evaluates it.
//
// A layer call is a chain of short, latency-bound kernels (routing, permutation indices) followed by the GEMMs; the FP4
// path also has to stream weights and activations through the encoder, which is bound by HBM.  Launched on a second stream,
// the encoder costs two cross-stream waits of 6-10 us each; appended to the launches of the latency-bound kernels, as blocks
// behind theirs, it fills the same idle memory system without one.  Forced FP4, four sets of weights in turn, the weights' encoder
// in a launch of its own in front of a layer call that finds them encoded -> riding along: 512 tokens of the tiny layer
// 28.5 -> 23.9 us, 512 / 4096 / 16384 tokens of the Kimi-VL shape 64.6 / 116.8 / 267.8 -> 63.2 / 116.6 / 264.9 us, of the Qwen3-VL
// shape 68.6 / 126.5 / 291.6 -> 65.8 / 124.4 / 290.3 us.  (One set of weights again and again, which the memory-side cache then
// holds: alone 4-7 us faster at 16384 tokens.)
#pragma once
#include "common.h"
#include "mxfp4_device.h"

namespace realb {

// ---- the precision decision of one rank (paper Sec. "Real-time Modality-aware LB Scheduling"); ratios are never formed
struct PolicyRule {
    double C, M_dec_congested, M_dec_calm, tau;   // M after this layer's AIMD update, for either outcome of the congestion test
    double total;                                 // T*k
    int D;
};
__host__ __device__ inline bool policy_congested(long long max_load, int D, double tau, double total) {
    return (double)(max_load * D) > tau * total;
}
__host__ __device__ inline bool policy_fp4(int load, int vis, int D, double C, double M_dec, double total) {
    const bool hot = (double)((long long)load * D) > C * total;
    const bool vision_heavy = (double)vis > M_dec * (double)load;
    return hot && vision_heavy && load > 0;
}

// What a kernel needs to know the layer's precision: fixed by the host, or decided from the routing statistics, which every
// wave evaluates for itself (D <= 64 loads) -- so no kernel waits for the host and none has to publish the decision.
struct PrecisionSource {
    int fixed;                                    // REALB_BF16 / REALB_FP4, or -1: decide
    int rank;
    const int32_t* rank_load;
    const int32_t* rank_vis;
    PolicyRule rule;
};
__device__ __forceinline__ bool precision_is_fp4(const PrecisionSource& p) {
    if (p.fixed >= 0) return p.fixed == REALB_FP4;
    const int lane = threadIdx.x & 63;
    const int load = lane < p.rule.D ? p.rank_load[lane] : 0;
    const int vis = p.rank_vis[p.rank];
    int m = load;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) m = max(m, __shfl_xor(m, d));
    m = __builtin_amdgcn_readfirstlane(m);
    const int mine = __builtin_amdgcn_readlane(load, p.rank);
    const double M = policy_congested(m, p.rule.D, p.rule.tau, p.rule.total) ? p.rule.M_dec_congested : p.rule.M_dec_calm;
    return policy_fp4(mine, vis, p.rule.D, p.rule.C, M, p.rule.total);
}

// The same before rank_load / rank_vis are there, from per-block partial counts [n_part, 2*D] (a whole block of NT threads
// calls it; tot: 2*D ints of LDS).
template <int NT>
__device__ __forceinline__ bool precision_from_parts(const PrecisionSource& p, const int32_t* __restrict__ rank_part, int n_part, int32_t* tot) {
    if (p.fixed >= 0) return p.fixed == REALB_FP4;
    const int C2 = 2 * p.rule.D;                              // <= 128
    if ((int)threadIdx.x < C2) tot[threadIdx.x] = 0;
    __syncthreads();
    int sum = 0;
    const int cols = C2 <= 16 ? 16 : C2 <= 32 ? 32 : C2 <= 64 ? 64 : 128, c = threadIdx.x % cols;
    if (c < C2) {
        const int step = NT / cols;
        for (int b = threadIdx.x / cols; b < n_part; b += 16 * step) {
            int v[16];                                        // 16 independent loads in flight
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = b + i * step < n_part ? rank_part[(size_t)(b + i * step) * C2 + c] : 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += v[i];
        }
        atomicAdd(&tot[c], sum);
    }
    __syncthreads();
    int m = 0;
    for (int d = 0; d < p.rule.D; ++d) m = max(m, tot[d]);
    const double M = policy_congested(m, p.rule.D, p.rule.tau, p.rule.total) ? p.rule.M_dec_congested : p.rule.M_dec_calm;
    return policy_fp4(tot[p.rank], tot[p.rule.D + p.rank], p.rule.D, p.rule.C, M, p.rule.total);
}

// ---- weights: a tensor is a flat sequence of 32-element blocks (rows are multiples of 128 long and contiguous)
struct QuantTensor {
    const u32x4_t* src;      // BF16 values, 16-byte chunks
    uint32_t* q;             // codes, one dword per chunk
    uint8_t* s;              // scales, K-step tiled
    long long n_chunks;
    int cpr;                 // chunks per row = K / 8
    float inv_cpr;
};
struct QuantJob { QuantTensor t[2]; unsigned blocks0, blocks; };   // blocks0: blocks of t[0]; blocks: of both

// Block `block` (NT threads) of a job.  A quad of lanes encodes one block of 32: each lane loads 16 B (8 values), the quad
// shares the maximum, each lane stores 4 B of codes and the quad's first lane stores the scale byte at its K-step-tiled
// position.  UNROLL independent loads per lane keep enough bytes in flight.  One job covers up to two tensors (the rank's
// W13 and W2): the first `blocks0` blocks take tensor 0, the rest tensor 1.
template <int NT, int UNROLL>
__device__ __forceinline__ void quantize_block(const QuantJob& job, unsigned block) {
    const bool second = block >= job.blocks0;                                     // uniform per block
    const QuantTensor& t = job.t[second ? 1 : 0];
    const u32x4_t* __restrict__ src = t.src;
    uint32_t* __restrict__ q = t.q;
    uint8_t* __restrict__ s = t.s;
    const long long n_chunks = t.n_chunks;
    const int cpr = t.cpr;
    const long long block_base = ((long long)(block - (second ? job.blocks0 : 0u)) * UNROLL) * NT;
    const int KD = cpr >> 4;                                  // K-steps per row (128 elements = 16 chunks)
    const unsigned row_b = (unsigned)block_base / (unsigned)cpr;             // one division per thread; n_chunks < 2^31
    const int in_row0 = (int)((unsigned)block_base - row_b * (unsigned)cpr);
    u32x4_t v[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const long long c = block_base + (long long)u * NT + threadIdx.x;
        v[u] = c < n_chunks ? __builtin_nontemporal_load(src + c) : u32x4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const long long c = block_base + (long long)u * NT + threadIdx.x;
        uint32_t byte;
        const uint32_t codes = encode_block_quad(v[u], &byte);    // whole quads are in or out of range together
        if (c < n_chunks) {
            __builtin_nontemporal_store(codes, q + c);
            if ((threadIdx.x & 3) == 0) {
                const int in_row = in_row0 + u * NT + threadIdx.x;                   // < cpr + NT * UNROLL < 2^16
                const int dr = (int)(((float)in_row + 0.5f) * t.inv_cpr);            // exact: in_row < 2^16
                s[scale_byte_offset(row_b + dr, (in_row - dr * cpr) >> 2, KD)] = (uint8_t)byte;
            }
        }
    }
}

// ---- activations: the tokens with a local expert, one encoded row per token (row index = token index)
struct TokenJob {
    const u32x4_t* x;
    const int32_t* topk_ids;
    uint32_t* q;
    uint8_t* s;
    int T, k, chunks;        // chunks = H / 8
    int lo, n_local;         // local experts
    unsigned blocks;
};

constexpr unsigned kTokenBlocksMax = 1u << 20;
// Block `block` (NT threads): a wave takes one token, 2048 elements in one go.  One token per wave, not several in turn:
// what hides the latency of the chain ids -> row -> store is the number of waves (16384 tokens, 75 MB: 35 -> 24 us for the
// launch that carries them together with W2); beyond kTokenBlocksMax blocks (4M tokens and more) they take turns, so that a
// launch stays below 2^32 threads.
template <int NT>
__device__ __forceinline__ void encode_tokens_block(const TokenJob& job, unsigned block) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int t = (int)block * (NT / 64) + wave; t < job.T; t += (int)job.blocks * (NT / 64)) {
        const int e = lane < job.k ? job.topk_ids[(size_t)t * job.k + lane] - job.lo : -1;
        if (__ballot(e >= 0 && e < job.n_local) == 0ull) continue;                 // no local expert: nobody reads this row
        const u32x4_t* src = job.x + (size_t)t * job.chunks;
        for (int c0 = 0; c0 < job.chunks; c0 += 256) {
            u32x4_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * 64 + lane;
                v[u] = c < job.chunks ? src[c] : u32x4_t{0, 0, 0, 0};
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * 64 + lane;
                uint32_t byte;
                const uint32_t codes = encode_block_quad(v[u], &byte);
                // the four scales of a 128-element K-step are one dword of the tiled tensor: lane 16m stores the dword
                // packed from lanes 16m, 16m+4, 16m+8, 16m+12 (chunks is a multiple of 16)
                const uint32_t word = byte | ((uint32_t)__shfl_down((int)byte, 4) << 8) | ((uint32_t)__shfl_down((int)byte, 8) << 16) |
                                      ((uint32_t)__shfl_down((int)byte, 12) << 24);
                if (c < job.chunks) {
                    job.q[(size_t)t * job.chunks + c] = codes;
                    if ((lane & 15) == 0) *reinterpret_cast<uint32_t*>(job.s + scale_byte_offset(t, c >> 2, job.chunks >> 4)) = word;
                }
            }
        }
    }
}

// ---- what rides along in one launch, behind the launch's own blocks
struct SideJobs {
    PrecisionSource when;     // nothing is done if this says BF16
    TokenJob x;
    QuantJob w;
    __host__ __device__ unsigned blocks() const { return x.blocks + w.blocks; }
};
#ifndef REALB_QUANT_UNROLL
#define REALB_QUANT_UNROLL 4
#endif
// TOKENS = false: launches that never carry activations (fewer registers)
template <int NT, bool TOKENS = true>
__device__ __forceinline__ void do_side_job(const SideJobs& jobs, unsigned block) {
    if (TOKENS && block < jobs.x.blocks) encode_tokens_block<NT>(jobs.x, block);
    else quantize_block<NT, REALB_QUANT_UNROLL>(jobs.w, block - jobs.x.blocks);
}
template <int NT, bool TOKENS = true>
__device__ __forceinline__ void run_side_jobs(const SideJobs& jobs, unsigned block) {
    if (precision_is_fp4(jobs.when)) do_side_job<NT, TOKENS>(jobs, block);
}

// Side jobs in a launch of their own; their blocks have kSideThreads threads.
constexpr int kSideThreads = 256;
int launch_side_jobs(const SideJobs& jobs, hipStream_t stream);

// Adds a tensor [rows, K] to a job whose launch has blocks of NT threads (a job holds at most two).
int add_quant_tensor(QuantJob* job, const void* src, long long rows, int K, uint8_t* q, uint8_t* s, int NT);

}  // namespace realb
