// On-the-fly BF16 -> MXFP4 weight transformation (paper Sec. "Overhead-Aware
// Pipeline Orchestration", Overlapping Pipeline): a pure HBM stream, 2 B read
// and 17/32 B written per element.  Scale bytes go to their K-step-tiled positions.
#include "encode_device.h"

namespace realb {

template <int NT>
__global__ void __launch_bounds__(NT) quantize_flat_kernel(const QuantJob job) { quantize_block<NT, REALB_QUANT_UNROLL>(job, blockIdx.x); }

template <int NT>
__global__ void __launch_bounds__(NT) side_jobs_kernel(const SideJobs jobs) { run_side_jobs<NT>(jobs, blockIdx.x); }

int launch_side_jobs(const SideJobs& jobs, hipStream_t stream) {
    if (jobs.blocks() == 0) return REALB_OK;
    hipLaunchKernelGGL(side_jobs_kernel<kSideThreads>, dim3(jobs.blocks()), dim3(kSideThreads), 0, stream, jobs);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}

int add_quant_tensor(QuantJob* job, const void* src, long long rows, int K, uint8_t* q, uint8_t* s, int NT) {
    const long long per_block = (long long)NT * REALB_QUANT_UNROLL;
    const long long n_chunks = rows * (K / 8);
    REALB_REQUIRE(n_chunks < (1ll << 31), REALB_ECAP, "tensor too large for one launch");
    const unsigned blocks = (unsigned)((n_chunks + per_block - 1) / per_block);
    QuantTensor& t = job->t[job->blocks > 0 ? 1 : 0];
    t = QuantTensor{(const u32x4_t*)src, (uint32_t*)q, s, n_chunks, K / 8, 1.0f / (float)(K / 8)};
    if (job->blocks == 0) job->blocks0 = blocks;
    job->blocks += blocks;
    return REALB_OK;
}

// Encodes one tensor [rows0, K0], or two when rows1 > 0, in a single launch (the second tensor's stream starts while the
// first one's last blocks drain instead of behind a kernel boundary).
int launch_quantize_flat(const void* src0, long long rows0, int K0, uint8_t* q0, uint8_t* s0,
                         const void* src1, long long rows1, int K1, uint8_t* q1, uint8_t* s1, hipStream_t stream) {
    constexpr int NT = 256;
    QuantJob job{};
    int rc = add_quant_tensor(&job, src0, rows0, K0, q0, s0, NT);
    if (rc == REALB_OK && rows1 > 0) rc = add_quant_tensor(&job, src1, rows1, K1, q1, s1, NT);
    if (rc != REALB_OK) return rc;
    if (job.blocks == 0) return REALB_OK;
    hipLaunchKernelGGL(quantize_flat_kernel<NT>, dim3(job.blocks), dim3(NT), 0, stream, job);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}

}  // namespace realb

using namespace realb;

extern "C" {

int realb_quantize_rows_fp4(const void* x, long long rows, int K, uint8_t* q, uint8_t* s, void* stream) {
    REALB_REQUIRE(rows >= 0 && K > 0 && K % 128 == 0 && K <= 65536, REALB_ESHAPE, "rows=%lld K=%d: K must be a positive multiple of 128", rows, K);
    if (rows == 0) return REALB_OK;
    REALB_REQUIRE(x && q && s, REALB_EINVAL, "NULL argument");
    return launch_quantize_flat(x, rows, K, q, s, nullptr, 0, 0, nullptr, nullptr, as_stream(stream));
}

int realb_quantize_experts_fp4(realb_ctx* ctx, const void* w13, const void* w2, int n_local, uint8_t* w13_q,
                               uint8_t* w13_s, uint8_t* w2_q, uint8_t* w2_s, void* stream) {
    REALB_REQUIRE(ctx && w13 && w2 && w13_q && w13_s && w2_q && w2_s, REALB_EINVAL, "NULL argument");
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    REALB_REQUIRE(n_local >= 0 && n_local <= c->n_local, REALB_ECAP, "n_local=%d exceeds the context's %d", n_local, c->n_local);
    return launch_quantize_flat(w13, (long long)n_local * 2 * c->cfg.I, c->cfg.H, w13_q, w13_s,
                                w2, (long long)n_local * c->cfg.H, c->cfg.I, w2_q, w2_s, as_stream(stream));
}

}  // extern "C"
