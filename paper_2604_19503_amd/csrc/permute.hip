// Token permutation / dispatch packing for one rank: a deterministic, stable
// counting sort of the rank's (token, expert) assignments by local expert,
// then a row gather that either copies BF16 rows or encodes them to MXFP4.
// Stands in for the all-to-all dispatch of the paper's pipeline (Sec.
// "Overhead-Aware Pipeline Orchestration"); the weight encoder overlaps it.
#include "encode_device.h"
#include "hist_reduce.h"

namespace realb {

constexpr int kIters = kPermChunk / 64;   // 64 assignments per wave iteration
// Chunks (= waves) per block of the count and rank kernels.  They are bound by latency, and a wave's chain of instructions
// takes the longer the more waves share its SIMD: blocks of 4 waves, one per SIMD.  8192 tokens, 65 536 assignments, 16 local
// experts: ranking 10.4 us with blocks of 16 waves, 7.5 us with 4; with a ballot per bit of the expert's number (same_expert)
// 6.0 us; counting 6.6 -> 4.1 us.  Blocks of 4 against 16 waves, both with those ballots: FP4 rank calls, whose encoders run
// beside these kernels, 62.5 against 65.7 us (512 tokens, 8 local experts), 109.0 / 111.8 (3001, 16) and 147.9 / 150.2 (8192, 64);
// realb_permute with 64 local experts, where every wave adds up 16 experts' group counts, 21.1 / 19.7 us at 85 chunks, 24.4 /
// 24.8 at 256 and 34.4 / 31.3 at 512 -- and 50.4, 56.4 and 63.2 us with 16 waves and a ballot per expert.

// The local expert (or -1) of each of the 4 x 64 assignments a = t*k + j of a wave's chunk.
__device__ __forceinline__ void load_chunk(int (&le)[kIters], const int32_t* __restrict__ topk_ids, int chunk, int n_chunks, int A,
                                           int lo, int lane) {
#pragma unroll
    for (int i = 0; i < kIters; ++i) {
        const int a = chunk * kPermChunk + i * 64 + lane;
        le[i] = (chunk < n_chunks && a < A) ? topk_ids[a] - lo : -1;
    }
}

// Phase 1 (a block = one group of kPermGroup chunks, one wave per chunk): each wave counts, per local expert, the
// assignments of its chunk of kPermChunk consecutive flat indices (lane e holds expert e's count); the block adds
// them up per expert.  wave_cnt is expert-major [n_local, n_chunks], group_cnt [n_local, n_groups].
// gsum: 64 ints of LDS.
__device__ __forceinline__ void perm_count_body(int* gsum, int group, const int32_t* __restrict__ topk_ids, int A, int lo, int n_local,
                                                int n_chunks, int n_groups, int32_t* __restrict__ wave_cnt,
                                                int32_t* __restrict__ group_cnt) {
    const int lane = threadIdx.x & 63;
    const int chunk = group * kPermGroup + (threadIdx.x >> 6);
    int le[kIters];
    load_chunk(le, topk_ids, chunk, n_chunks, A, lo, lane);
    if (threadIdx.x < 64) gsum[threadIdx.x] = 0;
    __syncthreads();
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < kIters; ++i)
        cnt += __popcll(same_expert(le[i], n_local, lane).of_lane);
    if (chunk < n_chunks && lane < n_local) {
        wave_cnt[(size_t)lane * n_chunks + chunk] = cnt;
        atomicAdd(&gsum[lane], cnt);
    }
    __syncthreads();
    if ((int)threadIdx.x < n_local) group_cnt[(size_t)threadIdx.x * n_groups + group] = gsum[threadIdx.x];
}

__global__ void __launch_bounds__(kPermThreads) perm_count_kernel(const int32_t* __restrict__ topk_ids, int A, int lo, int n_local,
                                                            int n_chunks, int n_groups, int32_t* __restrict__ wave_cnt,
                                                            int32_t* __restrict__ group_cnt, const SideJobs jobs) {
    __shared__ int gsum[64];
    if ((int)blockIdx.x >= n_groups) return run_side_jobs<kPermThreads>(jobs, blockIdx.x - n_groups);
    perm_count_body(gsum, blockIdx.x, topk_ids, A, lo, n_local, n_chunks, n_groups, wave_cnt, group_cnt);
}

// Phase 2 (same blocks): every block first works out, from the group sums, each expert's total (whose exclusive scan
// over the experts is expert_offsets; block 0 stores it) and the number of its assignments in earlier groups -- wave w
// adds up expert w's column of group_cnt, 64 groups per step -- so no separate scan kernel sits between the two
// phases.  Then each wave walks its chunk again and gives every local assignment its row:
// expert_offsets[e] + (assignments of e in earlier groups) + (in earlier chunks of the group) + (rank inside the chunk).
__global__ void __launch_bounds__(kPermThreads) perm_rank_kernel(const int32_t* __restrict__ topk_ids, int A, int lo, int n_local,
                                                                 int n_chunks, int n_groups, const int32_t* __restrict__ wave_cnt,
                                                                 const int32_t* __restrict__ group_cnt,
                                                                 int32_t* __restrict__ expert_offsets,
                                                                 int32_t* __restrict__ row_to_assign, int32_t* __restrict__ assign_to_row,
                                                                 const SideJobs jobs) {
    __shared__ int before[64], total[64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int group = blockIdx.x, n_front = max(n_groups, 1);
    if (group >= n_front) return run_side_jobs<kPermThreads>(jobs, blockIdx.x - n_front);
    const int chunk = group * kPermGroup + wave;
    int le[kIters];
    load_chunk(le, topk_ids, chunk, n_chunks, A, lo, lane);
    // this lane's expert: its assignments in the earlier chunks of this group
    int within = 0;
    if (lane < n_local) {
        int v[kPermGroup];
#pragma unroll
        for (int q = 0; q < kPermGroup; ++q)                          // (q < wave: that chunk exists whenever this wave's does)
            v[q] = (q < wave && group * kPermGroup + q < n_chunks) ? wave_cnt[(size_t)lane * n_chunks + group * kPermGroup + q] : 0;
#pragma unroll
        for (int q = 0; q < kPermGroup; ++q) within += v[q];
    }
    for (int e = wave; e < n_local; e += kPermGroup) {
        int b = 0, t = 0;
        for (int q = lane; q < n_groups; q += 64) {
            const int v = group_cnt[(size_t)e * n_groups + q];
            t += v;
            if (q < group) b += v;
        }
        b = wave_sum(b);
        t = wave_sum(t);
        if (lane == 0) { before[e] = b; total[e] = t; }
    }
    __syncthreads();
    const int tot = lane < n_local ? total[lane] : 0;
    const int incl = wave_inclusive_scan(tot);
    if (group == 0 && wave == 0) {
        if (lane < n_local) expert_offsets[lane] = incl - tot;
        if (lane == n_local - 1) expert_offsets[n_local] = incl;
    }
    if (chunk >= n_chunks) return;
    int running = (lane < n_local) ? incl - tot + before[lane] + within : 0;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < kIters; ++i) {
        const int a = chunk * kPermChunk + i * 64 + lane;
        const SameExpert same = same_expert(le[i], n_local, lane);
        const bool local = (unsigned)le[i] < (unsigned)n_local;
        const int base = __shfl(running, local ? le[i] : 0);
        const int row = local ? base + __popcll(same.own & lt_mask) : -1;
        running += __popcll(same.of_lane);
        if (a < A) {
            assign_to_row[a] = row;
            if (row >= 0) row_to_assign[row] = a;
        }
    }
}

// The layer call's index kernel.  There the routing kernel has just written, for each of its blocks of per_block consecutive
// tokens, a histogram over all experts -- which is what the count kernel would count again.  So one launch finishes the
// routing: the first D blocks add up the partial histograms, one EP rank each, and hand the statistics to the host; block
// D + b ranks the assignments of routing block b (expert_offsets and its own base from the partial histograms of all blocks
// and of the blocks before it); the blocks behind those run the side jobs, whose precision they evaluate from the per-rank
// partial counts, since the reduced ones are being written beside them.
// Bound by latency: two dependent memory round trips, and a few ballots per 64 assignments, twice.
constexpr int kFinishThreads = 256, kFinishWaves = kFinishThreads / 64, kFinishRegs = 8;
struct FinishArgs {
    const int32_t* hist_part;
    const int32_t* rank_part;
    int n_part, per_block, E, D;
    int32_t *expert_cnt, *expert_vis, *rank_load, *rank_vis;
    unsigned long long* stats_words;
    int stats_seq;
    const int32_t* topk_ids;
    int A, k, lo, n_local;
    int32_t *expert_offsets, *row_to_assign, *assign_to_row;
    unsigned side_blocks;        // blocks launched for the side jobs: they share the jobs' own blocks out among themselves
};

__global__ void __launch_bounds__(kFinishThreads) route_finish_kernel(const FinishArgs p, const SideJobs jobs) {
    extern __shared__ int32_t dyn[];                  // 2*E/D ints (reduce blocks), 2*D ints (side blocks)
    __shared__ int before[64], total[64], wcnt[kFinishWaves][64];
    const int front = p.D + max(p.n_part, 1);
    if ((int)blockIdx.x < p.D)
        return hist_reduce_body(dyn, p.hist_part, p.n_part, p.E, p.D, blockIdx.x, p.expert_cnt, p.expert_vis, p.rank_load, p.rank_vis,
                                p.stats_words, p.stats_seq);
    if ((int)blockIdx.x >= front) {
        if (!precision_from_parts<kFinishThreads>(jobs.when, p.rank_part, p.n_part, dyn)) return;
        for (unsigned b = blockIdx.x - front; b < jobs.blocks(); b += p.side_blocks) do_side_job<kFinishThreads>(jobs, b);
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.x - p.D, n_local = p.n_local;
    // this wave's share of the block's assignments: `iters` pieces of 64
    const int a_lo = b * p.per_block * p.k, n = min(p.per_block * p.k, p.A - a_lo);
    const int iters = (n + 64 * kFinishWaves - 1) / (64 * kFinishWaves);
    const int w_lo = wave * iters * 64;
    auto local_expert = [&](int i) __attribute__((always_inline)) {
        const int q = w_lo + i * 64 + lane;
        return q < n ? p.topk_ids[a_lo + q] - p.lo : -1;
    };
    int le[kFinishRegs];
#pragma unroll
    for (int i = 0; i < kFinishRegs; ++i) le[i] = i < iters ? local_expert(i) : -1;
    // expert totals and the counts of earlier blocks: thread (r, e) walks the partials r, r + R, ..
    if (threadIdx.x < 64) before[threadIdx.x] = total[threadIdx.x] = 0;
    __syncthreads();
    {
        const int cols = n_local <= 8 ? 8 : n_local <= 16 ? 16 : n_local <= 32 ? 32 : 64, e = threadIdx.x % cols;
        if (e < n_local) {
            int bsum = 0, tsum = 0;
            const int step = kFinishThreads / cols;
            for (int q = threadIdx.x / cols; q < p.n_part; q += 8 * step) {
                int v[8];                                     // 8 independent loads in flight
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = q + i * step < p.n_part ? p.hist_part[(size_t)(q + i * step) * 2 * p.E + p.lo + e] : 0;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    tsum += v[i];
                    bsum += q + i * step < b ? v[i] : 0;
                }
            }
            atomicAdd(&total[e], tsum);
            atomicAdd(&before[e], bsum);
        }
    }
    int cnt = 0;
    for (int i = 0; i < iters; ++i) {
        int v = -1;
        if (iters <= kFinishRegs) {
#pragma unroll
            for (int r = 0; r < kFinishRegs; ++r) v = r == i ? le[r] : v;
        } else v = local_expert(i);
        cnt += __popcll(same_expert(v, n_local, lane).of_lane);
    }
    wcnt[wave][lane] = cnt;
    __syncthreads();
    const int tot = lane < n_local ? total[lane] : 0;
    const int incl = wave_inclusive_scan(tot);
    if (b == 0 && wave == 0) {
        if (lane < n_local) p.expert_offsets[lane] = incl - tot;
        if (lane == n_local - 1) p.expert_offsets[n_local] = incl;
    }
    int running = lane < n_local ? incl - tot + before[lane] : 0;
    for (int w = 0; w < wave; ++w) running += wcnt[w][lane];
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    for (int i = 0; i < iters; ++i) {
        int v = -1;
        if (iters <= kFinishRegs) {
#pragma unroll
            for (int r = 0; r < kFinishRegs; ++r) v = r == i ? le[r] : v;
        } else v = local_expert(i);
        const SameExpert same = same_expert(v, n_local, lane);
        const bool local = (unsigned)v < (unsigned)n_local;
        const int base = __shfl(running, local ? v : 0);
        const int row = local ? base + __popcll(same.own & lt_mask) : -1;
        running += __popcll(same.of_lane);
        const int q = w_lo + i * 64 + lane;
        if (q < n) {
            p.assign_to_row[a_lo + q] = row;
            if (row >= 0) p.row_to_assign[row] = a_lo + q;
        }
    }
}

// Phase 4: one wave per TOKEN, grid-strided: a token routed to several local experts
// is read (and, on the FP4 path, encoded) once and written to each of its rows.
// H/8 chunks of 16 B per row; FP4: quads of lanes share one 32-element block.
template <bool FP4, int CPL>   // CPL = 16-byte chunks per lane = H / 512 rounded up
__global__ void __launch_bounds__(256) perm_gather_kernel(const u32x4_t* __restrict__ x, const int32_t* __restrict__ assign_to_row,
                                                          int T, int k, int H, u32x4_t* __restrict__ x_perm,
                                                          uint32_t* __restrict__ x_q, uint8_t* __restrict__ x_s) {
    const int lane = threadIdx.x & 63;
    const int chunks = H >> 3;                             // 16-B chunks per row, multiple of 16
    // A block takes a contiguous range of tokens: the rows of one 32-row group of an expert come from
    // tokens close together, so their scale words (which share 128-byte lines in the tiled scale tensor)
    // are written through the same L2 and leave it as whole lines.
    // Blocks b, b+8, .. share an XCD: each XCD takes one contiguous eighth of the tokens, its blocks
    // contiguous pieces of it.
    // (BF16 rows are whole lines anyway; there the strided assignment of tokens to blocks measured faster.)
    const int per_xcd = (T + 7) >> 3, nb = max((int)gridDim.x >> 3, 1);
    const int x_lo = (int)(blockIdx.x & 7) * per_xcd, x_hi = min(T, x_lo + per_xcd);
    const int per_block = (per_xcd + nb - 1) / nb;
    const int t_lo = FP4 ? x_lo + (int)(blockIdx.x >> 3) * per_block + (int)(threadIdx.x >> 6)
                         : (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    const int t_end = FP4 ? min(x_hi, x_lo + ((int)(blockIdx.x >> 3) + 1) * per_block) : T;
    const int t_step = FP4 ? (int)(blockDim.x >> 6) : (int)(gridDim.x * (blockDim.x >> 6));
    for (int t = t_lo; t < t_end; t += t_step) {
        const int my_row = lane < k ? assign_to_row[(size_t)t * k + lane] : -1;
        if (__ballot(my_row >= 0) == 0ull) continue;       // no local expert for this token
        const u32x4_t* src = x + (size_t)t * chunks;
        u32x4_t v[CPL];
#pragma unroll
        for (int u = 0; u < CPL; ++u) {
            const int c = u * 64 + lane;
            v[u] = c < chunks ? src[c] : u32x4_t{0, 0, 0, 0};
        }
        uint32_t codes[CPL], byte[CPL], word[CPL];
        if (FP4) {
#pragma unroll
            for (int u = 0; u < CPL; ++u) {
                codes[u] = encode_block_quad(v[u], &byte[u]);
                word[u] = byte[u] | ((uint32_t)__shfl_down((int)byte[u], 4) << 8) | ((uint32_t)__shfl_down((int)byte[u], 8) << 16) |
                          ((uint32_t)__shfl_down((int)byte[u], 12) << 24);
            }
        }
        for (int j = 0; j < k; ++j) {
            const int r = __builtin_amdgcn_readlane(my_row, j);
            if (r < 0) continue;
#pragma unroll
            for (int u = 0; u < CPL; ++u) {
                const int c = u * 64 + lane;
                if (c < chunks) {
                    if (FP4) {
                        x_q[(size_t)r * chunks + c] = codes[u];
                        // the four scales of a 128-element K-step are one dword of the tiled tensor: lane 16m
                        // stores the dword packed from lanes 16m, 16m+4, 16m+8, 16m+12 (chunks is a multiple of 16)
                        if ((lane & 15) == 0)
                            *reinterpret_cast<uint32_t*>(x_s + scale_byte_offset(r, c >> 2, chunks >> 4)) = word[u];
                    } else {
                        x_perm[(size_t)r * chunks + c] = v[u];
                    }
                }
            }
        }
    }
}

template <bool FP4>
static void launch_gather(int blocks, hipStream_t s, const void* x, const int32_t* a2r, int T, int k, int H, void* x_perm,
                          uint8_t* x_q, uint8_t* x_s) {
    const int cpl = (H / 8 + 63) / 64;
#define REALB_GATHER(CPL)                                                                                              \
    hipLaunchKernelGGL((perm_gather_kernel<FP4, CPL>), dim3(blocks), dim3(256), 0, s, (const u32x4_t*)x, a2r, T, k, H, \
                       (u32x4_t*)x_perm, (uint32_t*)x_q, x_s)
    if (cpl <= 1) REALB_GATHER(1);
    else if (cpl <= 2) REALB_GATHER(2);
    else if (cpl <= 4) REALB_GATHER(4);
    else if (cpl <= 8) REALB_GATHER(8);
    else REALB_GATHER(16);
#undef REALB_GATHER
}

}  // namespace realb

using namespace realb;

namespace realb {

static int check_permute(const Ctx* c, const int32_t* topk_ids, int T, int rank, long long max_rows, const int32_t* expert_offsets,
                         const int32_t* row_to_assign, const int32_t* assign_to_row) {
    REALB_REQUIRE(c && expert_offsets, REALB_EINVAL, "NULL argument");
    REALB_REQUIRE(T >= 0 && T <= c->cfg.T_max, REALB_ECAP, "T=%d outside [0, T_max=%d]", T, c->cfg.T_max);
    REALB_REQUIRE(rank >= 0 && rank < c->cfg.D, REALB_EINVAL, "rank=%d outside [0,%d)", rank, c->cfg.D);
    const int k = c->cfg.k, n_local = c->n_local;
    const long long worst = (long long)T * (k < n_local ? k : n_local);
    REALB_REQUIRE(max_rows >= worst, REALB_EINVAL, "max_rows=%lld is below the worst case %lld", max_rows, worst);
    REALB_REQUIRE(T == 0 || (topk_ids && row_to_assign && assign_to_row), REALB_EINVAL, "NULL argument");
    return REALB_OK;
}

// The index half of realb_permute (count / rank); the side jobs' blocks have kPermThreads threads.
int permute_indices(Ctx* c, const int32_t* topk_ids, int T, int rank, long long max_rows, int32_t* expert_offsets,
                    int32_t* row_to_assign, int32_t* assign_to_row, const SideJobs& beside_count, const SideJobs& beside_rank, hipStream_t s) {
    const int rc = check_permute(c, topk_ids, T, rank, max_rows, expert_offsets, row_to_assign, assign_to_row);
    if (rc != REALB_OK) return rc;
    const int n_local = c->n_local, lo = rank * n_local;
    const long long A = (long long)T * c->cfg.k;
    const int n_chunks = ceil_div(A, kPermChunk);
    const int n_groups = ceil_div(n_chunks, kPermGroup);
    if (n_groups + beside_count.blocks() > 0)
        hipLaunchKernelGGL(perm_count_kernel, dim3(n_groups + beside_count.blocks()), dim3(kPermThreads), 0, s, topk_ids, (int)A, lo, n_local,
                           n_chunks, n_groups, c->wave_cnt, c->group_cnt, beside_count);
    hipLaunchKernelGGL(perm_rank_kernel, dim3((n_groups > 0 ? n_groups : 1) + beside_rank.blocks()), dim3(kPermThreads), 0, s, topk_ids,
                       (int)A, lo, n_local, n_chunks, n_groups, c->wave_cnt, c->group_cnt, expert_offsets, row_to_assign,
                       assign_to_row, beside_rank);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}

// Routing and the permutation's indices as the layer call issues them: top-k + histograms, then route_finish_kernel, whose
// reduce blocks write the statistics, tagged with stats_seq, to pinned memory.  Both launches carry side jobs (blocks of
// kTopkThreads and kSideThreads threads).
int route_and_index(Ctx* c, const realb_layer_io* io, int stats_seq, const SideJobs& beside_topk, const SideJobs& beside_finish, hipStream_t s) {
    REALB_REQUIRE(io->expert_cnt && io->expert_vis && io->rank_load && io->rank_vis, REALB_EINVAL, "NULL argument");
    const int rc = check_permute(c, io->topk_ids, io->T, io->rank, io->max_rows, io->expert_offsets, io->row_to_assign, io->assign_to_row);
    if (rc != REALB_OK) return rc;
    if (beside_topk.blocks() + beside_finish.blocks() == 0 && route_small(c, io, stats_seq, s)) {
        REALB_HIP(hipGetLastError());
        return REALB_OK;
    }
    FinishArgs p{};
    int32_t* rank_part = nullptr;
    const int n_part = route_topk_only(c, io->logits, io->is_vision, io->T, io->topk_ids, io->topk_w, beside_topk, &p.per_block, &rank_part, s);
    if (n_part < 0) return n_part;
    const int E = c->cfg.E, D = c->cfg.D;
    p.hist_part = c->hist_part; p.rank_part = rank_part; p.n_part = n_part; p.E = E; p.D = D;
    p.expert_cnt = io->expert_cnt; p.expert_vis = io->expert_vis; p.rank_load = io->rank_load; p.rank_vis = io->rank_vis;
    p.stats_words = c->stats_words; p.stats_seq = stats_seq;
    p.topk_ids = io->topk_ids; p.A = io->T * c->cfg.k; p.k = c->cfg.k; p.lo = io->rank * c->n_local; p.n_local = c->n_local;
    p.expert_offsets = io->expert_offsets; p.row_to_assign = io->row_to_assign; p.assign_to_row = io->assign_to_row;
    // blocks that evaluate the policy (a microsecond each) are few enough to be resident at once and take several jobs
    const unsigned jobs = beside_finish.blocks(), resident = 8u * (unsigned)c->num_cus;
    p.side_blocks = beside_finish.when.fixed >= 0 || jobs < resident ? jobs : resident;
    hipLaunchKernelGGL(route_finish_kernel, dim3(D + (n_part > 0 ? n_part : 1) + p.side_blocks), dim3(kFinishThreads),
                       2 * (size_t)(c->n_local > D ? c->n_local : D) * sizeof(int32_t), s, p, beside_finish);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}

int permute_gather(Ctx* c, const void* x, const int32_t* assign_to_row, int T, int prec, void* x_perm, uint8_t* x_q,
                   uint8_t* x_s, hipStream_t s) {
    REALB_REQUIRE(c != nullptr, REALB_EINVAL, "NULL argument");
    REALB_REQUIRE(prec == REALB_BF16 || prec == REALB_FP4, REALB_EINVAL, "bad precision %d", prec);
    REALB_REQUIRE(T >= 0 && T <= c->cfg.T_max, REALB_ECAP, "T=%d outside [0, T_max=%d]", T, c->cfg.T_max);
    if (T == 0) return REALB_OK;
    REALB_REQUIRE(x && assign_to_row, REALB_EINVAL, "NULL argument");
    REALB_REQUIRE(prec == REALB_BF16 ? x_perm != nullptr : (x_q && x_s), REALB_EINVAL, "NULL row buffer");
    const int k = c->cfg.k, H = c->cfg.H;
    const int blocks = 8 * (T < 32 ? 1 : (T / 32 < 512 ? T / 32 : 512));      // a multiple of 8 (XCDs), 4 waves each
    if (prec == REALB_FP4) launch_gather<true>(blocks, s, x, assign_to_row, T, k, H, nullptr, x_q, x_s);
    else launch_gather<false>(blocks, s, x, assign_to_row, T, k, H, x_perm, nullptr, nullptr);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}

}  // namespace realb

extern "C" int realb_permute(realb_ctx* ctx, const void* x, const int32_t* topk_ids, int T, int rank, int prec,
                             long long max_rows, int32_t* expert_offsets, int32_t* row_to_assign, int32_t* assign_to_row,
                             void* x_perm, uint8_t* x_q, uint8_t* x_s, void* stream) {
    REALB_REQUIRE(ctx != nullptr, REALB_EINVAL, "NULL argument");
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    REALB_REQUIRE(prec == REALB_BF16 || prec == REALB_FP4, REALB_EINVAL, "bad precision %d", prec);
    REALB_REQUIRE(T <= 0 || (x && (prec == REALB_BF16 ? x_perm != nullptr : (x_q && x_s))), REALB_EINVAL, "NULL row buffer");
    int rc = permute_indices(c, topk_ids, T, rank, max_rows, expert_offsets, row_to_assign, assign_to_row, SideJobs{}, SideJobs{}, as_stream(stream));
    if (rc != REALB_OK) return rc;
    return permute_gather(c, x, assign_to_row, T, prec, x_perm, x_q, x_s, as_stream(stream));
}
