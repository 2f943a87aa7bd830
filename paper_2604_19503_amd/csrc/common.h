// Internal declarations shared by the library's translation units (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdarg.h>
#include "../../include/realb.h"

namespace realb {

constexpr int kWave = 64;
constexpr int kPermChunk = 256;    // assignments ranked by one wave in permute
// Chunks that one block of the permutation's count and rank kernels handles, a wave each (the workspace holds one per-expert
// sum per group).
constexpr int kPermGroup = 4;
constexpr int kPermThreads = 64 * kPermGroup;      // block size of those kernels
constexpr int kTopkThreads = 1024;     // block size of the routing kernel
constexpr int kRouteBlocksMax = 512;   // most blocks the routing kernel is launched with (two per CU on 256 CUs)

struct Ctx {
    realb_config cfg;
    int n_local;
    int device;
    int num_cus;
    double M;
    // device workspace
    int32_t* wave_cnt;     // [n_local, n_chunks]  per-chunk local-expert counts of the permutation (one allocation with group_cnt)
    int32_t* group_cnt;    // [n_local, n_groups]  the same summed over groups of kPermGroup chunks
    int n_chunks_max;
    int32_t* hist_part;    // [kRouteBlocksMax, 2*E]  per-block partial histograms of route_stats
    // pinned host staging for the policy's inputs
    int32_t* stats_host;   // [2*D]: rank loads, rank vision loads
    unsigned long long* stats_words;   // [2*D], host-coherent: the same, written by the layer call's reduce blocks or for
                                       // realb_select_precision, each word tagged with the call's sequence number
                                       // (see hist_reduce_body)
    unsigned long long* start_word;    // behind them: c->start_seq once the gate/up GEMM of a prefetching call has started
    int start_seq;
    int stats_seq;         // sequence number of the last set of statistics words (never 0)
    hipStream_t side;      // side stream for the cross-layer prefetch
    hipEvent_t ev_fork;    // orders a rank call's prefetch behind the work before its GEMMs
    hipEvent_t ev_prefetch;   // end of the last cross-layer prefetch on the side stream
    bool prefetch_pending;    // ev_prefetch has been recorded and not yet been waited for by a caller's stream
    unsigned prefetches;      // prefetches issued so far
    int gemm_shape;           // tile shape of the step-by-step GEMMs, GemmParams::tile_mode (realb_set_gemm_tile_shape)
    int gemm_reserve;         // compute units the grouped GEMMs' persistent grids leave free (set around a prefetching call)
    // optional per-stage timing of the layer calls (realb_stage_timing): events recorded on the caller's stream
    bool stage_timing;
    bool stage_valid;      // a whole layer call has recorded all boundaries since timing was switched on
    hipEvent_t stage_ev[REALB_N_STAGES + 1];
};

void set_error(const char* fmt, ...);
// Waits until the reduce block launched on `s` has written the statistics tagged `seq` to stats_words, then evaluates the policy.
int select_precision_pinned(Ctx* c, int T, int force, int32_t* prec_host, double* ib_global_host, double* M_after_host,
                            int seq, hipStream_t s);
bool gate_up_gather_supported(const Ctx* c, int T, bool fp4);
struct SideJobs;           // encode_device.h
struct PrecisionSource;
PrecisionSource precision_source(const Ctx* c, int T, int force, int rank, const int32_t* rank_load, const int32_t* rank_vis);
// The layer call's two GEMMs, in the precision `prec` says or will say (gate/up: rows fetched through row_to_assign).
int launch_layer_gate_up(Ctx* c, const PrecisionSource& prec, const realb_layer_io* io, bool announce, hipStream_t s);
int launch_layer_down(Ctx* c, const PrecisionSource& prec, const realb_layer_io* io, hipStream_t s);
int next_stats_seq(Ctx* c);      // sequence number of the next set of statistics words
// Waits until the gate/up GEMM that was launched with start_seq has started.
int wait_for_gemm_start(Ctx* c, hipStream_t s);
int permute_indices(Ctx* c, const int32_t* topk_ids, int T, int rank, long long max_rows, int32_t* expert_offsets,
                    int32_t* row_to_assign, int32_t* assign_to_row, const SideJobs& beside_count, const SideJobs& beside_rank, hipStream_t s);
int route_topk_only(Ctx* c, const float* logits, const uint8_t* is_vision, int T, int32_t* topk_ids, float* topk_w, const SideJobs& jobs,
                    int* per_block, int32_t** rank_part, hipStream_t s);
bool route_small(Ctx* c, const realb_layer_io* io, int stats_seq, hipStream_t s);
int route_and_index(Ctx* c, const realb_layer_io* io, int stats_seq, const SideJobs& beside_topk, const SideJobs& beside_finish, hipStream_t s);
int permute_gather(Ctx* c, const void* x, const int32_t* assign_to_row, int T, int prec, void* x_perm, uint8_t* x_q,
                   uint8_t* x_s, hipStream_t s);
// BF16 -> MXFP4 encoder on one matrix [rows0, K0], or two when rows1 > 0, in a single launch.
int launch_quantize_flat(const void* src0, long long rows0, int K0, uint8_t* q0, uint8_t* s0,
                         const void* src1, long long rows1, int K1, uint8_t* q1, uint8_t* s1, hipStream_t stream);
int hip_fail(hipError_t e, const char* what);
// Address (on the current device) of the file-scope scratch array of realb_route_stats_static and the device's CU
// count; looked up once per device and cached.  Either output may be NULL.
int static_scratch_lookup(int32_t** ptr, int* num_cus);

#define REALB_HIP(call)                                                        \
    do {                                                                       \
        hipError_t e__ = (call);                                               \
        if (e__ != hipSuccess) return ::realb::hip_fail(e__, #call);           \
    } while (0)

#define REALB_REQUIRE(cond, code, ...)                                         \
    do {                                                                       \
        if (!(cond)) { ::realb::set_error(__VA_ARGS__); return (code); }       \
    } while (0)

// Stage boundary i of a layer call (no-op unless stage timing is on).
inline void stage_mark(Ctx* c, hipStream_t s, int i) {
    if (c->stage_timing) (void)hipEventRecord(c->stage_ev[i], s);
}

// Inclusive prefix sum over the 64 lanes with DPP only: four shifts inside each row of 16 lanes, then the
// last lane of row 0 / row 2 is added to the following row, then lane 31 to the upper half.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);     // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);     // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);     // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);     // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);     // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);     // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_inclusive_scan(v), 63); }

// 64 assignments, a lane each; v: the assignment's local expert, anything outside [0, n_local) if it has none.  own: the lanes
// whose expert is this lane's (if this lane has one); of_lane: the lanes whose expert has this lane's number (lanes below
// n_local).  One ballot for the local ones and one per bit of the expert's number: 4 for 8 local experts, 7 for 64, where one
// per expert would be 8 and 64.
struct SameExpert { unsigned long long own, of_lane; };
__device__ __forceinline__ SameExpert same_expert(int v, int n_local, int lane) {
    const unsigned long long any = __ballot((unsigned)v < (unsigned)n_local);
    SameExpert s{any, any};
    for (int b = 0; (1 << b) < n_local; ++b) {
        const unsigned long long set = __ballot((v >> b) & 1);
        s.own &= (v >> b) & 1 ? set : ~set;
        s.of_lane &= (lane >> b) & 1 ? set : ~set;
    }
    return s;
}

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }
inline int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }

}  // namespace realb
