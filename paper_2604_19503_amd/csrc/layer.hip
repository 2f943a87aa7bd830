// The rank layer end to end: the paper's four-stage pipeline (Sec. "System
// Overview") with the weight transformation overlapped with other work
// (Sec. "Overhead-Aware Pipeline Orchestration"): the encoders ride along in the
// launches of the routing and permutation kernels, which are bound by latency
// and leave the memory system idle, or, for the NEXT layer's weights, run on the
// context's side stream beside this layer's GEMMs.
//
// A layer call does not wait for the host between its kernels: where the precision is not known up front (forced, or the
// LB gate closed), the encoders and GEMMs evaluate the policy on the device from the routing statistics.  The host waits
// for the statistics last, with everything enqueued, and then evaluates the same rule for its results.
#include "encode_device.h"

using namespace realb;

// Checks of a layer call's arguments that do not depend on the precision; made before anything is enqueued.
static int validate_io(const Ctx* c, const realb_layer_io* io) {
    REALB_REQUIRE(io->T >= 0 && io->T <= c->cfg.T_max, REALB_ECAP, "T=%d outside [0, T_max=%d]", io->T, c->cfg.T_max);
    REALB_REQUIRE(io->rank >= 0 && io->rank < c->cfg.D, REALB_EINVAL, "rank=%d outside [0,%d)", io->rank, c->cfg.D);
    REALB_REQUIRE(io->max_rows >= (long long)io->T * (c->cfg.k < c->n_local ? c->cfg.k : c->n_local), REALB_EINVAL,
                  "max_rows=%lld is below the worst case", io->max_rows);
    REALB_REQUIRE(io->overlap >= 0 && io->overlap <= 4, REALB_EINVAL, "bad overlap value %d", io->overlap);
    REALB_REQUIRE(io->expert_offsets && io->h_mid && io->y_rows && io->w2 && io->w13, REALB_EINVAL, "NULL argument");
    REALB_REQUIRE(io->T == 0 || (io->x && io->topk_ids && io->topk_w && io->row_to_assign && io->assign_to_row && io->out), REALB_EINVAL,
                  "NULL argument");
    if (io->next_w13 != nullptr || io->next_w2 != nullptr) {      // cross-layer prefetch requested
        REALB_REQUIRE(io->next_w13 && io->next_w2 && io->next_w13_q && io->next_w13_s && io->next_w2_q && io->next_w2_s, REALB_EINVAL,
                      "cross-layer prefetch needs next_w13, next_w2 and all four next_* buffers");
        REALB_REQUIRE(io->next_w13_q != io->w13_q && io->next_w13_s != io->w13_s && io->next_w2_q != io->w2_q && io->next_w2_s != io->w2_s,
                      REALB_EINVAL, "the prefetch buffers must differ from this layer's FP4 weight buffers");
        REALB_REQUIRE(io->reserve_cus >= 0 && io->reserve_cus < c->num_cus, REALB_EINVAL, "reserve_cus=%d outside [0, %d)", io->reserve_cus, c->num_cus);
    }
    return REALB_OK;
}

static bool fp4_buffers(const realb_layer_io* io) {
    return io->w13_q && io->w13_s && io->w2_q && io->w2_s && io->x_q && io->x_s && io->h_s;
}

// Parts of the encoding work of a layer call, as side jobs for launches with blocks of `threads` threads.
static int add_w13(const Ctx* c, const realb_layer_io* io, int threads, SideJobs* jobs) {
    return add_quant_tensor(&jobs->w, io->w13, (long long)c->n_local * 2 * c->cfg.I, c->cfg.H, io->w13_q, io->w13_s, threads);
}
static int add_w2(const Ctx* c, const realb_layer_io* io, int threads, SideJobs* jobs) {
    return add_quant_tensor(&jobs->w, io->w2, (long long)c->n_local * c->cfg.H, c->cfg.I, io->w2_q, io->w2_s, threads);
}
static void add_tokens(const Ctx* c, const realb_layer_io* io, int threads, SideJobs* jobs) {
    const unsigned blocks = (unsigned)ceil_div(io->T, threads / 64);
    jobs->x = TokenJob{(const u32x4_t*)io->x, io->topk_ids, (uint32_t*)io->x_q, io->x_s, io->T, c->cfg.k, c->cfg.H / 8,
                       io->rank * c->n_local, c->n_local, blocks < kTokenBlocksMax ? blocks : kTokenBlocksMax};
}

// Makes `s` wait for the pending cross-layer prefetch.  may_query: an event that has completed is not waited for -- a wait
// costs the stream microseconds even then, and by the time a layer call's statistics have arrived the previous call's
// prefetch has ended.  Only the layer call, which waits for the host anyway, may ask so: the rank call and
// realb_prefetch_join can be recorded into a graph, where querying an event breaks the recording.
static int join_prefetch(Ctx* c, hipStream_t s, bool may_query) {
    if (!c->prefetch_pending) return REALB_OK;
    const hipError_t q = may_query ? hipEventQuery(c->ev_prefetch) : hipErrorNotReady;
    if (q != hipSuccess) {
        if (may_query) (void)hipGetLastError();           // (not-ready is no error of this call)
        REALB_HIP(hipStreamWaitEvent(s, c->ev_prefetch, 0));
    }
    c->prefetch_pending = false;
    return REALB_OK;
}

// A call that encodes its own weights comes behind a pending prefetch, which may be writing the same buffers.  The prefetch
// stays pending: the call that consumes it may be on another stream.  (In a stream that is being recorded into a graph an event
// from outside cannot be waited for; what a graph's replays find in flight is for the caller to join.)  may_query, as above: a
// prefetch that has ended is pending no more -- else every call after a pipeline that nobody continued would wait for it again.
static int order_behind_prefetch(Ctx* c, hipStream_t s, bool may_query) {
    if (!c->prefetch_pending) return REALB_OK;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    REALB_HIP(hipStreamIsCapturing(s, &capture));
    if (capture != hipStreamCaptureStatusNone) return REALB_OK;
    if (may_query) {
        if (hipEventQuery(c->ev_prefetch) == hipSuccess) {
            c->prefetch_pending = false;
            return REALB_OK;
        }
        (void)hipGetLastError();                          // (not-ready is no error of this call)
    }
    REALB_HIP(hipStreamWaitEvent(s, c->ev_prefetch, 0));
    return REALB_OK;
}

// The next layer's weights, on the side stream.  The caller has made sure that the buffers' readers (the previous call's
// GEMMs) are done or waited for.
static int issue_prefetch(Ctx* c, const realb_layer_io* io) {
    const int rc = launch_quantize_flat(io->next_w13, (long long)c->n_local * 2 * c->cfg.I, c->cfg.H, io->next_w13_q, io->next_w13_s,
                                        io->next_w2, (long long)c->n_local * c->cfg.H, c->cfg.I, io->next_w2_q, io->next_w2_s, c->side);
    ++c->prefetches;
    REALB_HIP(hipEventRecord(c->ev_prefetch, c->side));
    c->prefetch_pending = true;
    return rc;
}

// gate/up, down and combine of a layer call whose activations (and weights, FP4) are in place.
// prefetch: what starts the next layer's encoder -- ON_START: the host, when it sees the gate/up GEMM start; ON_EVENT: an
// event in front of that GEMM (for calls that do not wait for the GPU).
enum class Prefetch { NONE, ON_START, ON_EVENT };
static int gemms_and_combine(realb_ctx* ctx, realb_layer_io* io, const PrecisionSource& prec, Prefetch prefetch, void* stream) {
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    hipStream_t s = as_stream(stream);
    struct ReserveReset { Ctx* c; ~ReserveReset() { c->gemm_reserve = 0; } } reserve_reset{c};
    if (prefetch != Prefetch::NONE) {
        c->gemm_reserve = io->reserve_cus;
        c->start_seq = c->start_seq >= 0x7FFFFFFF ? 1 : c->start_seq + 1;
    }
    if (prefetch == Prefetch::ON_EVENT) REALB_HIP(hipEventRecord(c->ev_fork, s));
    stage_mark(c, s, 4);
    int rc = launch_layer_gate_up(c, prec, io, prefetch == Prefetch::ON_START, s);
    if (rc != REALB_OK) return rc;
    stage_mark(c, s, 5);
    if (prefetch == Prefetch::ON_EVENT) {
        REALB_HIP(hipStreamWaitEvent(c->side, c->ev_fork, 0));
        rc = issue_prefetch(c, io);
        if (rc != REALB_OK) return rc;
    }
    rc = launch_layer_down(c, prec, io, s);
    if (rc != REALB_OK) return rc;
    stage_mark(c, s, 6);
    rc = realb_combine(ctx, io->y_rows, io->assign_to_row, io->topk_w, io->T, io->out, stream);
    if (rc != REALB_OK) return rc;
    stage_mark(c, s, 7);
    c->stage_valid = c->stage_timing;
    if (prefetch != Prefetch::ON_START) return REALB_OK;
    // The next layer's encoder is launched when the gate/up GEMM has started (a word that its first block writes): earlier it
    // would compete with this layer's own encoding for the memory the GEMM leaves idle, and an event to order the two would
    // cost the caller's stream microseconds.
    rc = wait_for_gemm_start(c, s);
    return rc != REALB_OK ? rc : issue_prefetch(c, io);
}

// permute .. combine in a precision the host knows; indices_done: the permutation's index kernels are already on the stream.
static int rank_forward_steps(realb_ctx* ctx, realb_layer_io* io, int prec, void* stream, bool indices_done) {
    REALB_REQUIRE(ctx && io, REALB_EINVAL, "NULL argument");
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    REALB_REQUIRE(prec == REALB_BF16 || prec == REALB_FP4, REALB_EINVAL, "bad precision %d", prec);
    hipStream_t s = as_stream(stream);
    // everything that can be refused is checked before anything is enqueued
    int rc = validate_io(c, io);
    if (rc != REALB_OK) return rc;
    const bool fp4 = prec == REALB_FP4;
    if (fp4) REALB_REQUIRE(fp4_buffers(io), REALB_EINVAL, "NULL FP4 buffer");
    const bool prefetch = io->next_w13 != nullptr;
    const bool encode_weights = fp4 && io->overlap != 2 && io->overlap != 4;
    const bool gather = gate_up_gather_supported(c, io->T, fp4);
    if (io->overlap == 4 || prefetch) {                   // weights encoded by the previous call's prefetch, or its buffers reused
        rc = join_prefetch(c, s, false);
        if (rc != REALB_OK) return rc;
    } else if (encode_weights) {
        rc = order_behind_prefetch(c, s, false);
        if (rc != REALB_OK) return rc;
    }
    // FP4: the encoding rides along with the index kernels -- W13 beside the counting, tokens and W2 beside the ranking
    static_assert(kPermThreads == kSideThreads, "the side jobs of either launch");
    PrecisionSource known{};
    known.fixed = prec;
    SideJobs first{}, second{};
    first.when = second.when = known;
    if (encode_weights) {
        rc = add_w13(c, io, kSideThreads, &first);
        if (rc == REALB_OK) rc = add_w2(c, io, kSideThreads, &second);
        if (rc != REALB_OK) return rc;
    }
    if (fp4 && gather) add_tokens(c, io, kSideThreads, &second);
    if (!indices_done) {
        stage_mark(c, s, 0);
        stage_mark(c, s, 1);
        rc = permute_indices(c, io->topk_ids, io->T, io->rank, io->max_rows, io->expert_offsets, io->row_to_assign,
                             io->assign_to_row, first, second, s);
        stage_mark(c, s, 2);
    } else {
        rc = launch_side_jobs(first, s);
        if (rc == REALB_OK) rc = launch_side_jobs(second, s);
    }
    if (rc != REALB_OK) return rc;
    stage_mark(c, s, 3);
    if (gather) return gemms_and_combine(ctx, io, known, prefetch ? Prefetch::ON_EVENT : Prefetch::NONE, stream);
    // rows the gate/up GEMM cannot fetch through row_to_assign: the permuted copy, then the plain GEMMs
    rc = permute_gather(c, io->x, io->assign_to_row, io->T, prec, io->x_perm, io->x_q, io->x_s, s);
    if (rc != REALB_OK) return rc;
    stage_mark(c, s, 4);
    if (fp4)
        rc = realb_grouped_moe_ffn(ctx, prec, io->expert_offsets, c->n_local, io->max_rows, io->x_q, io->x_s, io->w13_q,
                                   io->w13_s, io->w2_q, io->w2_s, io->h_mid, io->h_s, io->y_rows, stream);
    else
        rc = realb_grouped_moe_ffn(ctx, prec, io->expert_offsets, c->n_local, io->max_rows, io->x_perm, nullptr, io->w13,
                                   nullptr, io->w2, nullptr, io->h_mid, nullptr, io->y_rows, stream);
    if (rc != REALB_OK) return rc;
    stage_mark(c, s, 5);                                 // (the two GEMMs went out in one call: their time is reported under [4])
    if (prefetch) {                                      // its buffers' last readers come before this point of the stream
        REALB_HIP(hipEventRecord(c->ev_fork, s));
        REALB_HIP(hipStreamWaitEvent(c->side, c->ev_fork, 0));
        rc = issue_prefetch(c, io);
        if (rc != REALB_OK) return rc;
    }
    stage_mark(c, s, 6);
    rc = realb_combine(ctx, io->y_rows, io->assign_to_row, io->topk_w, io->T, io->out, stream);
    if (rc != REALB_OK) return rc;
    stage_mark(c, s, 7);
    c->stage_valid = c->stage_timing;
    return REALB_OK;
}

// Runs the steps of a call; if one of them fails after the call has issued its prefetch, the caller's stream is still made to
// wait for it, so that the caller may free or reuse the buffers after its stream has drained, whatever the call returned.  An
// earlier call's prefetch is left to the call that will consume it: that may be on another stream than a call that is refused.
template <typename F>
static int joined_on_error(realb_ctx* ctx, void* stream, const F& steps) {
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    const unsigned issued_before = c ? c->prefetches : 0;
    const int rc = steps();
    if (rc != REALB_OK && c && c->prefetches != issued_before && c->prefetch_pending &&
        hipStreamWaitEvent(as_stream(stream), c->ev_prefetch, 0) == hipSuccess)
        c->prefetch_pending = false;
    return rc;
}

extern "C" int realb_rank_forward(realb_ctx* ctx, realb_layer_io* io, int prec, void* stream) {
    return joined_on_error(ctx, stream, [&] { return rank_forward_steps(ctx, io, prec, stream, false); });
}

static int layer_forward_steps(realb_ctx* ctx, realb_layer_io* io, void* stream) {
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    hipStream_t s = as_stream(stream);
    // Everything that can be refused is checked before anything is enqueued.
    int rc = validate_io(c, io);
    if (rc != REALB_OK) return rc;
    REALB_REQUIRE(io->force == REALB_FORCE_NONE || io->force == REALB_BF16 || io->force == REALB_FP4, REALB_EINVAL,
                  "bad force value %d", io->force);
    REALB_REQUIRE(io->expert_cnt && io->expert_vis && io->rank_load && io->rank_vis, REALB_EINVAL, "NULL argument");
    REALB_REQUIRE(io->T == 0 || (io->logits && io->is_vision), REALB_EINVAL, "NULL argument");
    if (io->force == REALB_FP4) REALB_REQUIRE(fp4_buffers(io), REALB_EINVAL, "NULL FP4 buffer");
    if (io->overlap == 3 && io->force != REALB_BF16)
        REALB_REQUIRE(io->w13_q && io->w13_s && io->w2_q && io->w2_s, REALB_EINVAL, "NULL FP4 weight buffer");
    const PrecisionSource prec = precision_source(c, io->T, io->force, io->rank, io->rank_load, io->rank_vis);
    const bool can_fp4 = prec.fixed != REALB_BF16, can_bf16 = prec.fixed != REALB_FP4;
    const bool prefetch = io->next_w13 != nullptr;
    // The whole layer goes out before the statistics are known, unless the GEMMs need a permuted copy of the rows (its form
    // depends on the precision) or the FP4 buffers are there only if the caller knows that the decision will be BF16.
    const bool ahead = (!can_fp4 || (fp4_buffers(io) && gate_up_gather_supported(c, io->T, true))) &&
                       (!can_bf16 || gate_up_gather_supported(c, io->T, false));
    // Side jobs: W13 beside the routing kernel if it is certain to be used, or speculated on (overlap = 3); the rest in the
    // next launch, which can evaluate the policy.
    SideJobs beside_topk{}, beside_finish{};
    if (ahead && can_fp4) {
        beside_topk.when.fixed = REALB_FP4;
        beside_finish.when = prec;
        add_tokens(c, io, kSideThreads, &beside_finish);
        if (io->overlap != 2 && io->overlap != 4) {
            rc = order_behind_prefetch(c, s, true);
            if (rc != REALB_OK) return rc;
            if (prec.fixed == REALB_FP4 || io->overlap == 3) rc = add_w13(c, io, kTopkThreads, &beside_topk);
            else rc = add_w13(c, io, kSideThreads, &beside_finish);
            if (rc == REALB_OK) rc = add_w2(c, io, kSideThreads, &beside_finish);
            if (rc != REALB_OK) return rc;
        }
    }
    stage_mark(c, s, 0);
    // The statistics reach pinned host memory with the histogram reduce, tagged with this call's sequence number.
    const int seq = next_stats_seq(c);
    rc = route_and_index(c, io, seq, beside_topk, beside_finish, s);
    if (rc != REALB_OK) return rc;
    stage_mark(c, s, 1);
    stage_mark(c, s, 2);
    auto wait_for_statistics = [&]() {
        return select_precision_pinned(c, io->T, io->force, io->prec_host, &io->ib_global, &io->M_after, seq, s);
    };
    if (!ahead) {
        rc = wait_for_statistics();
        if (rc != REALB_OK) return rc;
        return rank_forward_steps(ctx, io, io->prec_host[io->rank], stream, true);
    }
    stage_mark(c, s, 3);
    if (io->overlap != 4 && !prefetch) {
        rc = gemms_and_combine(ctx, io, prec, Prefetch::NONE, stream);
        const int rc2 = wait_for_statistics();
        return rc != REALB_OK ? rc : rc2;
    }
    // A prefetching pipeline launches its GEMMs once the statistics are there (the ranking kernel runs meanwhile): by then
    // everything the previous call enqueued has run, so the prefetch that filled this call's weights has ended and the
    // buffers of the next one have no reader left -- neither needs an event on the caller's stream.
    rc = wait_for_statistics();
    if (rc == REALB_OK) rc = join_prefetch(c, s, true);
    if (rc != REALB_OK) return rc;
    PrecisionSource known = prec;
    known.fixed = io->prec_host[io->rank];
    return gemms_and_combine(ctx, io, known, prefetch ? Prefetch::ON_START : Prefetch::NONE, stream);
}

extern "C" int realb_layer_forward(realb_ctx* ctx, realb_layer_io* io, void* stream) {
    REALB_REQUIRE(ctx && io, REALB_EINVAL, "NULL argument");
    return joined_on_error(ctx, stream, [&] { return layer_forward_steps(ctx, io, stream); });
}

extern "C" int realb_prefetch_join(realb_ctx* ctx, void* stream) {
    REALB_REQUIRE(ctx != nullptr, REALB_EINVAL, "ctx is NULL");
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    return join_prefetch(c, as_stream(stream), false);
}
