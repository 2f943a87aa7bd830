// Stage 4, balanced MoE execution (paper Sec. "System Overview"): the SwiGLU
// expert FFN of one rank as two grouped GEMMs, in the precision the scheduler
// picked -- BF16 operands on v_mfma_f32_32x32x16_bf16 (tiles of 192 and more rows:
// v_mfma_f32_16x16x32_bf16), or MXFP4 operands (W4A4)
// on the block-scaled v_mfma_scale_f32_32x32x64_f8f6f4.
//
// Both precisions share their tiles, which are byte-identical: a K-step is 64 bytes
// of every operand row in the register-staged kernel (32 BF16 or 128 FP4 values) and
// 128 in the direct-to-LDS one, made of MFMA K-slices of 32 bytes (16 x 16 MFMAs: 64),
// and a lane's fragment is 16 contiguous bytes of one row (8 BF16 values, or the 32
// FP4 values of exactly one MX block, whose E8M0 scale is therefore one byte per lane).
// The K-loop is one code for both, but for the BF16 tiles of 192 and 256 rows.
//
// The MFMA runs "transposed": the weight rows are its A operand and the
// activation rows its B operand, so a lane ends up with one activation row and
// 16 weight rows (16 x 16 MFMAs: two rows and 8 weight rows of either, which the
// epilogue exchanges between lanes to the same).  The weight rows of a 32-row tile
// are stored in LDS in a permuted order chosen so that those 16 are CONSECUTIVE
// output columns (columns 16*half .. 16*half+15 of the tile, half = lane/32).  The
// epilogues therefore need no LDS and no barrier:
//   gate/up : a wave holds the gate and the up tile of the same 32 columns, so
//             SwiGLU is element-wise in registers; h is rounded to BF16 and a
//             lane stores 32 contiguous bytes, or -- FP4 path -- shares the
//             block maximum with lane^32 (the other 16 columns of the MX block),
//             encodes its 16 values and stores 8 contiguous code bytes.
//   down    : a lane stores 32 contiguous bytes of its output row per tile.
// Tiles never straddle experts; row tails are clamped on load and masked on
// store.  expert_offsets is read on the device, so no host round trip.
#include "ffn_device.h"
#include "encode_device.h"
#include <type_traits>

namespace realb {

constexpr int BM = 256;              // activation rows per block
constexpr int KSTEP_BYTES = 64;      // bytes of each operand row per K-step

// Tile geometry: the block has 2 x WGN waves (rows x columns); a wave owns 128 activation rows
// x WN*32 weight rows, i.e. 4 x WN MFMA tiles of 32x32.
//
// LDS stage layout: a 64-byte row segment is split into its four 16-byte parts p = 2*slice + half
// (the unit one lane feeds to one MFMA), and each part has its own sub-array indexed by row:
// [p][row][16 B].  A wave's fragment read (32 consecutive rows, fixed p) is then 512 contiguous
// bytes, and the 32-byte pad between sub-arrays spreads the four parts a lane quad writes over
// different banks.
template <int WN, int WGN>
struct Geo {
    static constexpr int NT = 128 * WGN;                // threads per block
    static constexpr int BNW = 32 * WN * WGN;           // weight rows per block
    static constexpr int GC = BNW / 2;                  // gate/up: h columns per block
    static constexpr int SUB_A = BM * 16 + 32;
    static constexpr int SUB_B = BNW * 16 + 32;
    static constexpr int REGION_A = 4 * SUB_A;
    static constexpr int STAGE = 4 * SUB_A + 4 * SUB_B;
    static constexpr int JA = BM * 4 / NT;              // 16-byte global loads per thread per K-step, activations
    static constexpr int JB = BNW * 4 / NT;             //                                           , weights
};

// Tile index -> (expert, row tile, column tile); column tiles are the fast index.
__device__ __forceinline__ TileInfo decode_tile(const GemmParams& p, int tile, int cols_per_tile) {
    int mi = tile / p.n_tiles_n;
    const int nt = tile - mi * p.n_tiles_n;
    int e = 0, seg_lo = 0, seg_hi = 0;
    for (; e < p.n_local; ++e) {
        seg_lo = p.offs[e];
        seg_hi = p.offs[e + 1];
        const int te = (seg_hi - seg_lo + BM - 1) / BM;
        if (mi < te) break;
        mi -= te;
    }
    return TileInfo{e, seg_lo + mi * BM, seg_hi, nt * cols_per_tile};
}

// Epilogue of a wave's MT row tiles.
template <bool FP4, bool GATEUP, int MT, int WN, bool NT>
__device__ __forceinline__ void epilogue(const GemmParams& p, v16f_t (&acc)[MT][WN], int row0, int rows_valid, int n0,
                                         int wm, int wn, int li, int half) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
        epilogue_mt<FP4, GATEUP, WN, NT>(p, acc[mt], wm * (32 * MT) + mt * 32, row0, rows_valid, n0, wn, li, half);
}

template <int TA>
__device__ __forceinline__ int tiles_of(int lo, int hi) { return hi > lo ? (hi - lo + TA - 1) / TA : 0; }

// Persistent blocks of an XCD that take tiles: the fewest that finish the XCD's per_xcd tiles in as many rounds as all the
// launched ones would; the others exit at once.  A partly filled last round takes as long as a full one, so the idle
// blocks gain nothing -- and compute units left entirely free make the working ones faster (config 2, 1595 and 1160
// tiles: 29 instead of 32 blocks per XCD, both GEMMs 3.8 % faster; fewer active CUs share the power budget and the
// memory system), besides leaving room for whatever runs beside the GEMM.  FP4 only: the BF16 GEMMs move four times the
// bytes, their partly filled last round IS shorter (fewer blocks share the bandwidth), and they measured 1.2 % slower so.
__device__ __forceinline__ int working_slots(int per_xcd, int launched) {
    if (per_xcd <= 0) return 0;
    const int rounds = (per_xcd + launched - 1) / launched;
    return (per_xcd + rounds - 1) / rounds;
}

// Blocks b, b+8, b+16, .. share an XCD (and its L2), so each XCD takes a contiguous range of tiles
// (consecutive row tiles over all column tiles).  BF16: persistent blocks, one per residency slot,
// walk their XCD's range with a stride, and while a tile's epilogue runs the first K-step of the
// block's next tile is already in flight.  FP4: one tile per block (grid = worst-case tile count).
template <bool FP4, bool GATEUP, int WN, int WGN, int MINB>
__global__ void __launch_bounds__(128 * WGN, MINB) ffn_gemm_kernel(const GemmParams p) {
    using G = Geo<WN, WGN>;
    constexpr int NT = G::NT;
    constexpr int COLS = GATEUP ? G::GC : G::BNW;
    constexpr bool PERSIST = !FP4;    // the FP4 body has no registers to spare for a tile carried across the epilogue
    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WGN, wn = wave % WGN;
    const int li = lane & 31, half = lane >> 5;

    int total_m = 0;
    for (int e = 0; e < p.n_local; ++e) total_m += (p.offs[e + 1] - p.offs[e] + BM - 1) / BM;
    const int total = total_m * p.n_tiles_n;
    const int per_xcd = (total + 7) >> 3;
    const int nslots = FP4 ? working_slots(per_xcd, (int)(gridDim.x >> 3)) : (int)(gridDim.x >> 3);
    if ((int)(blockIdx.x >> 3) >= nslots) return;
    const int tile_hi = min(total, ((int)(blockIdx.x & 7) + 1) * per_xcd);
    int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= tile_hi) return;
    const bool nt_out = stream_output<FP4>(p);

    const int I_up = p.w_rows >> 1;                       // gate/up: offset of the up rows
    const size_t rowbytes = FP4 ? (size_t)(p.K >> 1) : (size_t)p.K * 2;
    const int nks = (int)(rowbytes / KSTEP_BYTES);
    const int kd = p.K >> 7;                              // FP4: K-steps = scale dwords per row
    const uint32_t* As32 = reinterpret_cast<const uint32_t*>(p.As);
    const uint32_t* Ws32 = reinterpret_cast<const uint32_t*>(p.Ws);

    // ---- tile-independent: LDS destinations of this thread's 16-byte chunks (4 per 64-byte row
    //      segment) and the fragment / scale addresses of this lane
    const int part = tid & 3;
    int a_dst[G::JA], b_dst[G::JB];
#pragma unroll
    for (int j = 0; j < G::JA; ++j) a_dst[j] = part * G::SUB_A + ((tid >> 2) + (NT / 4) * j) * 16;
#pragma unroll
    for (int j = 0; j < G::JB; ++j) b_dst[j] = G::REGION_A + part * G::SUB_B + w_slot((tid >> 2) + (NT / 4) * j) * 16;
    int b_rows[WN];                                       // first weight-tile row of each of this wave's column tiles
#pragma unroll
    for (int t = 0; t < WN; ++t) {
        if constexpr (GATEUP) b_rows[t] = (t < WN / 2 ? 0 : G::GC) + wn * (WN / 2) * 32 + (t % (WN / 2)) * 32;
        else b_rows[t] = wn * WN * 32 + t * 32;
    }
    const int a_frag = half * G::SUB_A + (wm * 128 + li) * 16;                 // + mt*512 + slice*2*SUB_A
    int b_frag[WN];
#pragma unroll
    for (int t = 0; t < WN; ++t) b_frag[t] = G::REGION_A + half * G::SUB_B + (b_rows[t] + li) * 16;   // + slice*2*SUB_B
    const int sshift = half * 8;

    // ---- per-tile prefetch state: source pointers and the first K-step
    const uint8_t* a_src[G::JA];
    const uint8_t* b_src[G::JB];
    u32x4_t ga[G::JA], gb[G::JB];
    // FP4: dword index (K-step 0) of this lane's scale words in the K-step-tiled scale tensors; a
    // wave's 32 rows at one K-step are one contiguous 128-byte line (two when the rows straddle
    // a group of 32), so the scales go from memory to the MFMA operand registers directly.
    int sa_off[4], sb_off[WN];
    uint32_t sa_nx[4], sb_nx[WN];                         // scale words of the next K-step
    TileInfo ti = decode_tile(p, tile, COLS);
    int kp = 0;                                           // the K-step (64 bytes) that the next loads fetch
    auto next_k = [&]() { kp = kp + 1 == nks ? 0 : kp + 1; };

    auto prefetch_tile = [&](const TileInfo& t) {
        kp = 2 * k_start<FP4, GATEUP>(t.n0, (nks + 1) >> 1);
#pragma unroll
        for (int j = 0; j < G::JA; ++j) {
            const int gr = min(t.row0 + (tid >> 2) + (NT / 4) * j, t.seg_hi - 1);
            a_src[j] = p.A + (size_t)gr * rowbytes + part * 16;
        }
#pragma unroll
        for (int j = 0; j < G::JB; ++j) {
            const int br = (tid >> 2) + (NT / 4) * j;
            b_src[j] = p.W + ((size_t)t.e * p.w_rows + w_tile_row<GATEUP, G::GC>(br, t.n0, I_up)) * rowbytes + part * 16;
        }
#pragma unroll
        for (int j = 0; j < G::JA; ++j) ga[j] = *reinterpret_cast<const u32x4_t*>(a_src[j] + (size_t)kp * KSTEP_BYTES);
#pragma unroll
        for (int j = 0; j < G::JB; ++j) gb[j] = *reinterpret_cast<const u32x4_t*>(b_src[j] + (size_t)kp * KSTEP_BYTES);
        if constexpr (FP4) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const int row = min(t.row0 + wm * 128 + mt * 32 + li, t.seg_hi - 1);
                sa_off[mt] = ((row >> 5) * kd) * 32 + (row & 31);
                sa_nx[mt] = As32[sa_off[mt] + kp * 32];
            }
#pragma unroll
            for (int c = 0; c < WN; ++c) {
                const int wrow = t.e * p.w_rows + w_tile_row<GATEUP, G::GC>(b_rows[c] + w_row_of_lane(li), t.n0, I_up);
                sb_off[c] = ((wrow >> 5) * kd) * 32 + (wrow & 31);
                sb_nx[c] = Ws32[sb_off[c] + kp * 32];
            }
        }
        next_k();
    };
    prefetch_tile(ti);

    while (true) {
        // ---- scales and the prefetched first K-step go to LDS, K-step 1 starts
#pragma unroll
        for (int j = 0; j < G::JA; ++j) *reinterpret_cast<u32x4_t*>(smem + a_dst[j]) = ga[j];
#pragma unroll
        for (int j = 0; j < G::JB; ++j) *reinterpret_cast<u32x4_t*>(smem + b_dst[j]) = gb[j];
        if (nks > 1) {
#pragma unroll
            for (int j = 0; j < G::JA; ++j) ga[j] = *reinterpret_cast<const u32x4_t*>(a_src[j] + (size_t)kp * KSTEP_BYTES);
#pragma unroll
            for (int j = 0; j < G::JB; ++j) gb[j] = *reinterpret_cast<const u32x4_t*>(b_src[j] + (size_t)kp * KSTEP_BYTES);
        }
        __syncthreads();

        v16f_t acc[4][WN];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

        // ---- main loop: LDS holds K-step ks (double buffered), registers hold K-step ks+1,
        //      whose global loads were issued a whole iteration earlier.
        for (int ks = 0; ks < nks; ++ks) {
            const uint8_t* st = smem + (ks & 1) * G::STAGE;
            int sa[4] = {0, 0, 0, 0}, sb[WN];
#pragma unroll
            for (int t = 0; t < WN; ++t) sb[t] = 0;
            if constexpr (FP4) {
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) sa[mt] = (int)(sa_nx[mt] >> sshift);
#pragma unroll
                for (int t = 0; t < WN; ++t) sb[t] = (int)(sb_nx[t] >> sshift);
                if (ks + 1 < nks) {
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) sa_nx[mt] = As32[sa_off[mt] + kp * 32];
#pragma unroll
                    for (int t = 0; t < WN; ++t) sb_nx[t] = Ws32[sb_off[t] + kp * 32];
                }
            }
            next_k();
            u32x4_t fa0[4], fb0[WN], fa1[4], fb1[WN];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) fa0[mt] = *reinterpret_cast<const u32x4_t*>(st + a_frag + mt * 512);
#pragma unroll
            for (int t = 0; t < WN; ++t) fb0[t] = *reinterpret_cast<const u32x4_t*>(st + b_frag[t]);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) fa1[mt] = *reinterpret_cast<const u32x4_t*>(st + 2 * G::SUB_A + a_frag + mt * 512);
#pragma unroll
            for (int t = 0; t < WN; ++t) fb1[t] = *reinterpret_cast<const u32x4_t*>(st + 2 * G::SUB_B + b_frag[t]);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)                   // K-slice 0: scale bytes 0/1 of the K-step's dword
#pragma unroll
                for (int t = 0; t < WN; ++t) mma<FP4, 0>(acc[mt][t], fb0[t], fa0[mt], sb[t], sa[mt]);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)                   // K-slice 1: scale bytes 2/3
#pragma unroll
                for (int t = 0; t < WN; ++t) mma<FP4, 2>(acc[mt][t], fb1[t], fa1[mt], sb[t], sa[mt]);
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 1 < nks) {
                uint8_t* nx = smem + ((ks + 1) & 1) * G::STAGE;
#pragma unroll
                for (int j = 0; j < G::JA; ++j) *reinterpret_cast<u32x4_t*>(nx + a_dst[j]) = ga[j];
#pragma unroll
                for (int j = 0; j < G::JB; ++j) *reinterpret_cast<u32x4_t*>(nx + b_dst[j]) = gb[j];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 2 < nks) {
#pragma unroll
                for (int j = 0; j < G::JA; ++j) ga[j] = *reinterpret_cast<const u32x4_t*>(a_src[j] + (size_t)kp * KSTEP_BYTES);
#pragma unroll
                for (int j = 0; j < G::JB; ++j) gb[j] = *reinterpret_cast<const u32x4_t*>(b_src[j] + (size_t)kp * KSTEP_BYTES);
            }
            __syncthreads();
        }

        // ---- the block's next tile: get its first K-step moving before the epilogue
        const TileInfo cur = ti;
        const bool more = PERSIST && tile + nslots < tile_hi;
        if (more) {
            tile += nslots;
            ti = decode_tile(p, tile, COLS);
            prefetch_tile(ti);
        }

        // ---- epilogue, straight from registers
        if (nt_out) epilogue<FP4, GATEUP, 4, WN, true>(p, acc, cur.row0, cur.seg_hi - cur.row0, cur.n0, wm, wn, li, half);
        else epilogue<FP4, GATEUP, 4, WN, false>(p, acc, cur.row0, cur.seg_hi - cur.row0, cur.n0, wm, wn, li, half);
        if (!more) break;
    }
}

// ---------------------------------------------------------------------------------------------
// Tile kernel with direct-to-LDS loads (the default): 256 x 256 tiles for long expert segments, smaller shapes for short
// ones and for what is left behind the last whole round of tiles.
//
// What bounds the 256 x 256 tiles on this chip is the path from L2 into the CU, not the MFMA rate (BF16 tiles of 192 and 256
// rows, whose waves take turns so that transfers and MFMAs overlap: the power limit): a CU takes in about one 1-KB vector-memory
// instruction per 18-26 cycles, and the vector L1 fetches whole 128-byte lines.  So this kernel
//   - fetches 128 bytes of every operand row per K-step (a full line: 256 FP4 or 64 BF16 values,
//     four MFMA K-slices), which halves the L2->L1 traffic of 64-byte steps;
//   - uses a 256 x 256 block tile (8 waves of 128 x 64), the largest whose two 64-KB stages fit the
//     160 KB of LDS, to minimise bytes fetched per MFMA;
//   - loads with global_load_lds_dwordx4 (memory -> LDS without passing through registers): a wave
//     instruction carries 8 rows x 128 B and lands as 1 KB of contiguous LDS.  Inside a 128-byte LDS
//     row the eight 16-byte parts are XOR-swizzled by (row>>1)&7 (done on the global address of
//     each lane, since the LDS side of the transfer is fixed), which makes the 32-row x 16-byte
//     fragment reads bank-conflict free;
//   - spreads the transfer instructions between MFMAs (a wave blocks while the memory pipeline accepts
//     an instruction, and eight waves issuing at once stall all MFMA issue) and keeps the producer a
//     whole K-step ahead, so that no transfer is waited for;
//   - is persistent: a block walks its XCD's tile range and its producer runs across tile boundaries
//     (the expert table sits in registers, so switching tiles touches no memory); only the
//     register-only epilogue sits between two tiles' MFMA streams;
//   - FP4: stages the E8M0 scales through LDS as well (global_load_lds_dword, 32 rows x 2 dwords
//     per instruction), because one vector-memory instruction per lane-dword costs as much issue
//     time as a 1-KB one.
//
// Short segments (decode steps, small prefills, ranks without load) are bound by something else: a batch of 24 tokens on a
// Kimi-VL-shaped rank has 88 tiles of 256 weight rows, a CU of which keeps one K-step (64 KB) in flight, and reading the
// 92 MB of W13 is a matter of bytes in flight.  So:
//   - 128- and 64-row tiles have three LDS stages (48 or 40 KB each), and the barrier of a K-step waits only for the next
//     step's transfers (s_waitcnt vmcnt(n), n > 0), leaving those of the step behind it in flight;
//   - 64 x 128 and (BF16) 64 x 64 tiles double the number of blocks once or twice and have six or nine stages (five or
//     eight steps in flight); four or two waves multiply, eight move data.
// Measured, BF16, weights from HBM, gate/up + down us, 256-row tiles -> these: 24 tokens (61 rows) 49.9 + 27.8 -> 19.6 + 11.6;
// 192 tokens 50.9 + 28.2 -> 22.5 + 13.2; 1 token 19 + 14 with 64 x 256 tiles -> 13.3 + 10.2; 1000 tokens (2169 rows) 56.5 + 30.7 -> 37 + 23.
// With four sets of weights in turn, under the profiler: 1 token 14.6 + 10.6, 24 tokens 24.0 + 12.3 (170 MB read, 138 of them weights
// and the rest K-steps that the producer fetches behind a block's last tile: 3.8 TB/s of what is needed), 1000 tokens 37.9 + 26.1.
// A split of the contraction over the waves of a block with operands straight in registers (no LDS) measured 34 + 18 at 24 tokens and
// was dropped.
// The accumulation order along K is the same for every shape and that of the other kernel, so results are bit-identical: a
// row's result does not depend on the batch it is in.
constexpr int KB = 128;                    // bytes of each operand row per K-step
// Geometry of a block tile: 64*MT activation rows x TW weight rows, 8 waves.  TW = 256: a 2 x 4 grid of waves of 32*MT x 64
// each.  TW = 128 and 64 (MT = 1 only): waves 0..3 (0..1) are that grid's first two columns (first column), the others only
// move data.
template <int MT, int TW>
struct TileGeo {
    static_assert(TW == 256 || ((TW == 128 || TW == 64) && MT == 1), "tile shapes");
    static constexpr int TA = 64 * MT;                 // activation rows of the block tile
    static constexpr int WN = TW / 64;                 // waves along the weight rows
    static constexpr int NS = MT >= 3 ? 2 : TW == 256 ? 3 : TW == 128 ? 6 : 9;   // LDS stages: 2 x 64 or 56 KB, 3 x 48 or 40 KB, 6 x 24 KB, 9 x 16 KB
    static constexpr int OPS_A = MT;                   // 8-row transfers per wave and K-step: activations
    static constexpr int OPS_W = TW / 64;              //                                    : weights
    static constexpr int W_ROWS = TW / 8;              // weight rows a wave moves
    static constexpr int REGION_W = TA * KB;           // weight rows follow the activation rows
    static constexpr int STAGE = (TA + TW) * KB;
    static constexpr int SC_BASE = NS * STAGE;         // FP4: scale staging, per stage [TA + TW rows][2 dwords]
    static constexpr int SC_STAGE = (TA + TW) * 8;
    static constexpr int SC_W = TA * 8;
    static constexpr int TOK_BASE = SC_BASE + NS * SC_STAGE;  // gathering kernel: row_to_assign entries of a tile, two buffers x 8 waves x 64 ints
    static constexpr int TOK_BUF = 8 * 64 * 4;
    static constexpr int LDS_BYTES = TOK_BASE + 2 * TOK_BUF;
};

// BF16 tiles of 192 and 256 rows: 16 x 16 MFMA tiles and a K-loop in which the two waves of a SIMD take turns at the matrix cores.
template <bool FP4, int MT>
constexpr bool kTurns = !FP4 && MT >= 3;

// All tiles of height TA = 64*MT of the row segments [off_lo, off_hi) (lane e: expert e's).  Every wave of the block calls it.
// GATHER (gate/up only): the activation rows are fetched straight from a token-indexed matrix (x itself,
// or the tokens' FP4 codes and scales) through row_to_assign, so no permuted copy has to be written.
template <bool FP4, bool GATEUP, bool GATHER, int MT, int TW>
__device__ __forceinline__ void tile_phase(const GemmParams& p, uint8_t* smem, const int off_lo, const int off_hi, const bool nt_out) {
    using G = TileGeo<MT, TW>;
    constexpr int TA = G::TA;
    constexpr int COLS = GATEUP ? TW / 2 : TW;             // output columns per block
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = TW == 256 ? wave >> 2 : (wave / G::WN) & 1, wn = wave & (G::WN - 1);
    const bool multiplies = TW == 256 || wave < 2 * G::WN;
    const int n_tiles_n = GATEUP ? p.n_out / COLS : (p.n_out + COLS - 1) / COLS;
    const int li = lane & 31, half = lane >> 5;

    // Order of an expert's tiles.  An XCD takes a contiguous range of them, and what its blocks share they fetch once: with column
    // tiles first the activations, with row tiles first the weights.  Row tiles first for BF16 tiles of up to 192 rows, of which an
    // expert has few.  Column tiles first against this, layer calls: 384 tokens 50.8 -> 46.0 us, 200 46.6 -> 44.7 (the 64-column
    // shapes), 500 tokens of the Qwen3-VL shape 51.6 -> 49.6 with cached weights; with weights from HBM 200 tokens 52.0 -> 50.7, 1000
    // 71.7 -> 71.0 (gate/up reads 168 -> 120 MB from behind the L2 in 38.9 -> 38.4 us: the K-step binds it, not memory); 8 to
    // 100 tokens, 2000 and 5003: within 1 % either way.
    // Column tiles first for 256-row tiles (row tiles first, FP4 down GEMM of 249 000 rows: 304 -> 409 us) and FP4 (0.7 % faster).
    constexpr bool ROWS_FIRST = !FP4 && MT < 4;
    // The expert table is in registers: lane e holds expert e's row segment and the inclusive prefix of row-tile counts (lanes from the
    // last expert on repeat the total), so that decoding a tile index is a multiplication, a ballot and three lane reads (row tiles first: a
    // fourth and, for experts of several row tiles, a division).  In LDS it was three dependent reads, for which every wave of the
    // block stood still at each tile: see advance().
    const int cum = wave_inclusive_scan(tiles_of<TA>(off_lo, off_hi));
    const int total = __builtin_amdgcn_readlane(cum, 63) * n_tiles_n;
    __syncthreads();                                          // (a second phase: the first one's readers of the stages are done)
    constexpr int WIDTH = TW == 256 ? 0 : TW == 128 ? 1 : 2;
    const uint32_t nt_magic = p.col_magic[WIDTH];
    const int nt_shift = p.col_shift[WIDTH];
    auto decode = [&](int t) __attribute__((always_inline)) {
        const int mi = div_by_magic(t, nt_magic, nt_shift), nt = t - mi * n_tiles_n;
        const int e = __popcll(__ballot(cum <= mi));              // experts that end at or before row tile mi
        const int lo = __builtin_amdgcn_readlane(off_lo, e), hi = __builtin_amdgcn_readlane(off_hi, e);
        const int first = e == 0 ? 0 : __builtin_amdgcn_readlane(cum, e - 1);
        if constexpr (ROWS_FIRST) {
            const int rows = __builtin_amdgcn_readlane(cum, e) - first, local = t - first * n_tiles_n;
            int col = local;
            if (rows > 1) col = local / rows;                 // (decode steps: one row tile per expert, no second division)
            return TileInfo{e, lo + (local - col * rows) * TA, hi, col * COLS};
        }
        return TileInfo{e, lo + (mi - first) * TA, hi, nt * COLS};
    };
    const int per_xcd = (total + 7) >> 3;
    const int nslots = FP4 ? working_slots(per_xcd, (int)(gridDim.x >> 3)) : (int)(gridDim.x >> 3);
    if ((int)(blockIdx.x >> 3) >= nslots) return;
    const int tile_hi = min(total, ((int)(blockIdx.x & 7) + 1) * per_xcd);
    int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= tile_hi) return;

    const int I_up = p.w_rows >> 1;
    const uint32_t rowbytes = FP4 ? (uint32_t)(p.K >> 1) : (uint32_t)p.K * 2;
    const int nks = (int)((rowbytes + KB - 1) / KB);
    // last K-step holds 64 bytes per row: FP4 rows only (K is a multiple of 128 values, so a BF16 row is whole K-steps)
    const bool tail_half = FP4 && (rowbytes % KB) != 0;
    const int kd = p.K >> 7;                              // FP4: scale dwords per row

    // ---- consumer side: fragment offsets inside a stage
    constexpr bool TURNS = kTurns<FP4, MT>;
    const int sw = (li >> 1) & 7;
    const int f_off0 = li * KB + ((half ^ sw) << 4);       // slice s reads part 2s+half: offset f_off0 ^ (s << 5)
    const int a_base = wm * (32 * MT) * KB;
    int b_pos[2];                                         // first LDS weight position of the wave's two column tiles
    if constexpr (GATEUP) { b_pos[0] = wn * 32; b_pos[1] = TW / 2 + wn * 32; }
    else { b_pos[0] = wn * 64; b_pos[1] = wn * 64 + 32; }

    // ---- producer side: this wave moves activation rows 8*MT*wave .. 8*MT*(wave+1)-1 and weight positions
    //      W_ROWS*wave .. W_ROWS*(wave+1)-1, 8 rows per instruction, and the scale dwords of 32 rows of each operand (the
    //      128-row tile has four such groups of activation rows: waves 4..7 repeat those of waves 0..3, so that every
    //      wave has the same number of transfers in flight).  Addresses are a per-tile scalar base plus a 32-bit
    //      per-lane offset.
    const int prow = lane >> 3;                           // row inside an 8-row instruction
    // 16-byte part a lane fetches in instruction j: (lane&7) ^ key, key = (R>>1)&7 = (4*(j&1) + (lane>>4)) & 7
    // for LDS row R = 8*j + prow (mod 16) of the j-th 8-row group of the tile.
    auto part16 = [&](int q) __attribute__((always_inline)) { return (uint32_t)(((lane & 7) ^ ((q * 4 + (lane >> 4)) & 7)) << 4); };
    auto part_w = [&](int j) __attribute__((always_inline)) { return (wave * G::OPS_W + j) & 1; };
    auto part_a = [&](int j) __attribute__((always_inline)) { return (wave * MT + j) & 1; };   // activations: 8-row group wave*MT + j
    // Weights: LDS position R holds weight-tile row (R & ~31) | w_row_of_lane(R & 31), which for
    // R & 31 = 8*j + prow is 16*((prow>>2)&1) + 4*j + (prow&3): instruction j is 4*j rows below
    // instruction 0, a scalar offset.  Per lane only the two part offsets differ (by parity of j).
    // (TURNS: w_row_of_slot16, that is 16*(j&1) + 4*(j>>1) + 8*(prow>>2) + (prow&3).)
    auto w_below = [&](int j) __attribute__((always_inline)) { return TURNS ? 16 * (j & 1) + 4 * (j >> 1) : 4 * j; };
    uint32_t b_voff[2];
    {
        // (a wave's first 8-row group is the g-th of a 32-row group, g = wave * OPS_W mod 4)
        const int br0 = TURNS ? wave * 32 + w_row_of_slot16(prow)
                              : (wave * G::OPS_W >> 2) * 32 + (wave * G::OPS_W & 3) * 4 + (((prow >> 2) & 1) << 4) + (prow & 3);
#pragma unroll
        for (int q = 0; q < 2; ++q) b_voff[q] = (uint32_t)w_tile_row<GATEUP, TW / 2>(br0, 0, I_up) * rowbytes + part16(q);
    }
    int a_last = 0;                                       // scalar: last existing row of the tile being fetched
    uint32_t a_goff[GATHER ? G::OPS_A : 1];               // GATHER: byte offset of this lane's source row, per instruction
    const int wgrp = TW == 256 ? wave : wave & (TW / 32 - 1);              // the group of 32 weight rows whose scales this wave moves
    const int srow = wgrp * 32 + (lane >> 1), swhich = lane & 1;
    const int sgrp = MT == 3 ? (wave < 6 ? wave : wave - 6) : wave & (2 * MT - 1);      // the group of 32 activation rows whose scales this wave moves
    int sa_idx = 0, sb_idx = 0;                           // FP4: dword index of this lane's scale word, K-step 0
    const uint8_t* a_tile = nullptr;                      // scalar: first activation row / weight row of the tile being fetched
    const uint8_t* b_tile = nullptr;

    TileInfo ti = decode(tile);
    // GATHER: the row_to_assign entries of a tile's rows are brought into LDS one tile ahead (a wave fetches the
    // entries of its own rows with one direct-to-LDS transfer and later reads back only what it fetched), so
    // that switching tiles never waits for global memory: a register load at the switch would stall the producer
    // for a full memory latency, behind every transfer in flight.
    int tokbuf = 0;
    auto fetch_tokens = [&](const TileInfo& t, int buf) __attribute__((always_inline)) {
        if constexpr (GATHER) {
            const int row0 = __builtin_amdgcn_readfirstlane(t.row0), rows = __builtin_amdgcn_readfirstlane(t.seg_hi - t.row0);
            // entries 0 .. 8*MT-1: the wave's rows; MT < 4: behind them the 32 rows of its scale group (MT = 4: the same rows)
            const int want = MT == 4 ? wave * 32 + (lane & 31) : lane < 8 * MT ? wave * (8 * MT) + lane : sgrp * 32 + ((lane - 8 * MT) & 31);
            const int r = row0 + min(want, rows - 1);                             // rows past the segment: its last row again
            lds_dma4(reinterpret_cast<const uint32_t*>(p.row_src) + r, smem + G::TOK_BASE + buf * G::TOK_BUF + wave * 256);
        }
    };
    auto setup_src = [&](const TileInfo& t) __attribute__((always_inline)) {
        const int row0 = __builtin_amdgcn_readfirstlane(t.row0), rows = __builtin_amdgcn_readfirstlane(t.seg_hi - t.row0);
        const int e = __builtin_amdgcn_readfirstlane(t.e), n0 = __builtin_amdgcn_readfirstlane(t.n0);
        a_tile = GATHER ? p.A : p.A + (size_t)row0 * rowbytes;
        // down GEMM with n_out an odd multiple of 128: the last column tile is half a tile; the waves that would fetch
        // weight rows behind it fetch the half that exists again, and the epilogue skips those columns
        const int wshift = !GATEUP && TW == 256 && n0 + TW > p.n_out && wave >= 4 ? TW / 2 : 0;
        b_tile = p.W + ((size_t)e * p.w_rows + n0 - wshift) * rowbytes;
        a_last = rows - 1;
        const int* toks = reinterpret_cast<const int*>(smem + G::TOK_BASE + tokbuf * G::TOK_BUF) + wave * 64;   // this tile's entries (GATHER)
        if constexpr (GATHER) {
#pragma unroll
            for (int j = 0; j < G::OPS_A; ++j)
                a_goff[j] = (uint32_t)div_by_magic(toks[j * 8 + prow], p.src_magic, p.src_shift) * rowbytes + part16(part_a(j));
        }
        if constexpr (FP4) {
            int gr = row0 + min(sgrp * 32 + (lane >> 1), rows - 1);
            if constexpr (GATHER) gr = div_by_magic(toks[(MT == 4 ? 0 : 8 * MT) + (lane >> 1)], p.src_magic, p.src_shift);   // the token that holds this row's codes and scales
            sa_idx = ((gr >> 5) * kd) * 32 + (gr & 31);
            const int br = (srow & ~31) | w_row_of_lane(srow & 31);
            const int wr = e * p.w_rows + w_tile_row<GATEUP, TW / 2>(br, n0 - wshift, I_up);
            sb_idx = ((wr >> 5) * kd) * 32 + (wr & 31);
        }
    };
    // One producer instruction of K-step k into stage `dstg`: op 0/1 = scales (FP4), 2..5 = activations, 6..9 = weights.
    auto issue = [&](int op, int k, int dstg) __attribute__((always_inline)) {
        if (op < 2) {
            if constexpr (FP4) {
                const int ko = min(2 * k + swhich, kd - 1) * 32;
                uint8_t* l = smem + G::SC_BASE + dstg * G::SC_STAGE;
                if (op == 0) lds_dma4(reinterpret_cast<const uint32_t*>(p.As) + (uint32_t)(sa_idx + ko), l + sgrp * 256);
                else lds_dma4(reinterpret_cast<const uint32_t*>(p.Ws) + (uint32_t)(sb_idx + ko), l + G::SC_W + wgrp * 256);
            }
        } else {
            const int j = (op - 2) & 3;
            const bool halfstep = tail_half && k == nks - 1;
            // half step: lanes of parts 4..7 fetch parts 0..3 again (the row has only 64 bytes left)
            const int q = op < 6 ? part_a(j) : part_w(j);
            const uint32_t koff = (uint32_t)(k * KB) - (halfstep ? (uint32_t)(((lane << 4) ^ (q << 6)) & 64) : 0u);
            uint8_t* l = smem + dstg * G::STAGE;
            if (op < 6) {
                uint32_t v;
                l += (wave * G::OPS_A + j) * 1024;
                if constexpr (GATHER) v = a_goff[j];
                else v = (uint32_t)min(wave * (8 * MT) + j * 8 + prow, a_last) * rowbytes + part16(part_a(j));   // rows past the segment: its last row again
                lds_dma16(a_tile + (v + koff), l);
            } else {
                lds_dma16(b_tile + (size_t)w_below(j) * rowbytes + (b_voff[q] + koff), l + G::REGION_W + (wave * G::OPS_W + j) * 1024);
            }
        }
    };

    // ---- producer position: the K-step it fetches next (pk of tile ptile).  Past the block's last tile
    //      it keeps refetching that tile's steps, which nobody reads but the block waits for: with the 64 x 128 tiles of K = 2048
    //      5 steps for 32, with the 64 x 64 tiles of K = 1408 8 for 22 (24 tokens: 107 + 63 MB read for 92 + 46 MB of weights).
    constexpr bool STARTS = kHasStarts<FP4, GATEUP>;          // (without them the counters pn and ck, which then equal pk and ks, are not kept)
    int ptile = tile, pn = 0, pk = k_start<FP4, GATEUP>(ti.n0, nks);      // pn: K-steps of the tile issued before this one
    auto advance = [&]() __attribute__((always_inline)) {
        pk = pk + 1 == nks ? 0 : pk + 1;
        if constexpr (STARTS) pn = pn + 1 == nks ? 0 : pn + 1;
        if ((STARTS ? pn : pk) == 0) {
            if (ptile + nslots < tile_hi) {
                ptile += nslots;
                if constexpr (GATHER) tokbuf ^= 1;                     // fetched while the previous tile was being produced
                const TileInfo next = decode(ptile);
                setup_src(next);
                if constexpr (STARTS) pk = k_start<FP4, GATEUP>(next.n0, nks);
                if constexpr (GATHER) {
                    if (ptile + nslots < tile_hi) fetch_tokens(decode(ptile + nslots), tokbuf ^ 1);
                }
            }
        }
    };
    if constexpr (GATHER) {
        fetch_tokens(ti, 0);
        if (tile + nslots < tile_hi) fetch_tokens(decode(tile + nslots), 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    setup_src(ti);
    auto issue_step = [&](int k, int dstg) __attribute__((always_inline)) {
#pragma unroll
        for (int op = 0; op < 10; ++op)
            if (op < 2 + G::OPS_A || (op >= 6 && op < 6 + G::OPS_W)) issue(op, k, dstg);
    };
    // Fill the stages, then wait for the first step only: draining them all here would leave the memory system idle for a
    // latency.  (Where the producer crosses a tile boundary already here, the gather entries it then reads must have landed.)
    constexpr int OPS = G::OPS_A + G::OPS_W + (FP4 ? 2 : 0);             // transfers per wave and step
    auto step_forward = [&]() __attribute__((always_inline)) {
        if (GATHER && nks < G::NS) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        advance();
    };
    issue_step(pk, 0);
#pragma unroll
    for (int q = 1; q < G::NS - 1; ++q) { step_forward(); issue_step(pk, q); }
    step_forward();
    // transfers from .. to-1 of a step (no scales), activations first
    auto issue_some = [&](int from, int to, int k, int dstg) __attribute__((always_inline)) {
#pragma unroll
        for (int i = from; i < to; ++i) issue(i < G::OPS_A ? 2 + i : 6 + i - G::OPS_A, k, dstg);
    };
    constexpr int EARLY = 4;                                             // TURNS: transfers of a step that go out in the step that frees its stage
    if constexpr (TURNS) {
        issue_some(0, EARLY, pk, G::NS - 1);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((G::NS - 2) * OPS + EARLY) : "memory");
    } else if constexpr (TW < 256) {
        issue_step(pk, G::NS - 1);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((G::NS - 1) * OPS) : "memory");
    } else {
#pragma unroll
        for (int j = 0; j < G::OPS_A; ++j) issue(2 + j, pk, G::NS - 1);  // first half of the step that fills the last stage (see below)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((G::NS - 2) * OPS + G::OPS_A) : "memory");
    }

    // One flat loop over the (tile, K-step) pairs of this block, with a single copy of the K-step code:
    // the steps of a tile follow each other without a seam, and the producer runs ahead across tile
    // boundaries.  Inside a step the block barrier sits after the third K-slice: by then every wave
    // holds its fourth slice in registers, so the stage is free, and behind the barrier
    //   - the first fragments and the scales of the NEXT step are read while the fourth slice
    //     multiplies (no LDS latency is exposed at the start of a step), and
    //   - the producer starts on the step AFTER the next one: its activation rows go out between the
    //     MFMAs of the fourth slice, its weight rows and scales between those of the next step's first
    //     slice, so every transfer has a whole step to land before the barrier that publishes it.
    int stg = 0, left = G::NS - 1;                        // stage of the current step, stage of the step before it
    int ks = 0, ck = k_start<FP4, GATEUP>(ti.n0, nks);          // steps of the tile multiplied so far, K-step being multiplied
    v16f_t acc[TURNS ? 1 : MT][2];                        // 32 x 32 tiles
    v4f_t acc16[TURNS ? MT : 1][2][4];                    // TURNS: 16 x 16 tiles, in pairs of row tiles
    auto clear = [&]() __attribute__((always_inline)) {
        if constexpr (TURNS) {
#pragma unroll
            for (int i = 0; i < 2 * MT; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc16[i / 2][i % 2][j] = v4f_t{0.f, 0.f, 0.f, 0.f};
        } else {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        }
    };
    clear();
    int cur_row0 = ti.row0, cur_rows = ti.seg_hi - ti.row0, cur_n0 = ti.n0;

    auto store16_tiles = [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            epilogue16<GATEUP, decltype(nt)::value>(p, acc16[mt], wm * (32 * MT) + mt * 32, cur_row0, cur_rows, cur_n0, wn, lane);
    };
    auto store_tile = [&]() __attribute__((always_inline)) {
        if (!multiplies || (!GATEUP && cur_n0 + wn * 64 >= p.n_out)) {}   // columns behind the output's end
        else if constexpr (TURNS) {
            if (nt_out) store16_tiles(std::true_type{});
            else store16_tiles(std::false_type{});
        }
        else if (nt_out) epilogue<FP4, GATEUP, MT, 2, true>(p, acc, cur_row0, cur_rows, cur_n0, wm, wn, li, half);
        else epilogue<FP4, GATEUP, MT, 2, false>(p, acc, cur_row0, cur_rows, cur_n0, wm, wn, li, half);
    };
    // Accumulators back to zero, the block's next tile; false if there is none.
    auto next_tile = [&]() __attribute__((always_inline)) {
        tile += nslots;
        if (tile >= tile_hi) return false;
        clear();
        ti = decode(tile);
        cur_row0 = ti.row0; cur_rows = ti.seg_hi - ti.row0; cur_n0 = ti.n0;
        ks = 0;
        if constexpr (STARTS) ck = k_start<FP4, GATEUP>(ti.n0, nks);
        return true;
    };

    if constexpr (TW < 256) {
        // One multiplying wave per SIMD, and a K-slice is two MFMAs (64 cycles), less than the latency of an LDS read: reading
        // a slice ahead would expose that latency four times per step (24 tokens, down GEMM: 12.8 against 11.6 us).  Here a wave reads all of the next step's fragments
        // right behind the barrier that publishes it, into the other register set, and multiplies this step meanwhile.
        u32x4_t xa[2][4], xb[2][4][2];
        u32x2_t xra[2], xrb[2][2];
        auto read_step = [&](int set, int stage) __attribute__((always_inline)) {
            if (!multiplies) return;
            const uint8_t* st = smem + stage * G::STAGE;
            if constexpr (FP4) {
                const uint8_t* sc = smem + G::SC_BASE + stage * G::SC_STAGE;
                xra[set] = *reinterpret_cast<const u32x2_t*>(sc + (wm * 32 + li) * 8);
#pragma unroll
                for (int t = 0; t < 2; ++t) xrb[set][t] = *reinterpret_cast<const u32x2_t*>(sc + G::SC_W + (b_pos[t] + li) * 8);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                xa[set][q] = *reinterpret_cast<const u32x4_t*>(st + a_base + (f_off0 ^ (q << 5)));
#pragma unroll
                for (int t = 0; t < 2; ++t) xb[set][q][t] = *reinterpret_cast<const u32x4_t*>(st + G::REGION_W + b_pos[t] * KB + (f_off0 ^ (q << 5)));
            }
        };
        read_step(0, 0);
        auto step = [&](int set) __attribute__((always_inline)) {
            const bool last = ks == nks - 1;
            const bool full = !(tail_half && (STARTS ? ck : ks) == nks - 1);
            // the next step has landed, this wave's reads of the current stage are done: its transfers may be replaced
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((G::NS - 2) * OPS) : "memory");
            left = stg;
            stg = stg + 1 == G::NS ? 0 : stg + 1;
            advance();
            read_step(set ^ 1, stg);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (multiplies && (q < 2 || full)) {
                    const int wa = FP4 ? (int)((q < 2 ? xra[set].x : xra[set].y) >> (half * 8)) : 0;
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int wb = FP4 ? (int)((q < 2 ? xrb[set][t].x : xrb[set][t].y) >> (half * 8)) : 0;
                        if (q & 1) mma<FP4, 2>(acc[0][t], xb[set][q][t], xa[set][q], wb, wa);
                        else mma<FP4, 0>(acc[0][t], xb[set][q][t], xa[set][q], wb, wa);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (q == 0) {
#pragma unroll
                    for (int op = FP4 ? 0 : 2; op < 3; ++op) issue(op, pk, left);
                } else if (q - 1 < G::OPS_W) {
                    issue(6 + q - 1, pk, left);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            ++ks;
            if constexpr (STARTS) ck = ck + 1 == nks ? 0 : ck + 1;
            if (!last) return true;
            store_tile();
            return next_tile();
        };
        while (step(0) && step(1)) {}
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no transfer may still be writing this block's LDS when it ends
        return;
    }

    if constexpr (TURNS) {
        // The two waves of a SIMD take turns: waves 0..3 (rows wm = 0, one per SIMD) multiply while waves 4..7 read fragments and issue
        // transfers, then the other way round, a barrier at each change; waves 4..7 are one change behind.  In the loop below,
        // where all waves do the same at the same time, a wave that multiplies also blocks on its transfers (a CU takes one per 18-25
        // cycles), and the step lasts as long as its MFMAs and half of its transfers one behind the other: 2900 cycles for 2048
        // of MFMA.  Here a step is four turns per wave, each half the rows of a K-slice of 64 bytes: 16 MFMAs of 16 cycles (192 rows: 12).
        //   section 0: fragments of slice 0 (weights, lower rows, upper rows), transfers   turn 0: slice 0, lower rows
        //   section 1: fragments of slice 1 (weights, lower rows), transfers                turn 1: slice 0, upper rows
        //   section 2: fragments of slice 1 (upper rows): the stage is read                 turn 2: slice 1, lower rows
        //   section 3: transfers of the step after the next into that stage; the next step  turn 3: slice 1, upper rows
        //              has landed
        // Whole K-steps only (a BF16 row is a multiple of 128 bytes).  Measured with the 16 x 16 MFMA, 36 000 rows: gate/up K = 2048 345 -> 317
        // us, down K = 1408 191 -> 177; 249 000 rows: K = 2048 1259 -> 1185, K = 768 807 -> 735 (with 32 x 32 MFMAs 340, 187, 1246, 757).  With
        // operands of zeros, that is at the full clock, 297 -> 262: the rest is the power limit.  Sections that read one slice further
        // ahead, transfers spread over 2, 3 or 4 sections, one turn per slice, and no turns but separate barriers for "read" and "landed": within 2 %, or slower.
        constexpr int RS = MT;                             // 16-row tiles of a turn
        constexpr int LGKM = 0xC07F;                       // s_waitcnt of the LDS counter alone (bits 8..11; no scalar load is in flight in the loop)
        const int l16 = lane & 15, g = lane >> 4;
        const int f_off = l16 * KB + ((g ^ (l16 >> 1)) << 4);            // slice s, part 4s + g: f_off ^ (s << 6)
        u32x4_t xa[2][RS], xw[2][4];                       // [lower, upper rows], [slice]
        auto fence = [&]() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
        auto barrier = [&]() __attribute__((always_inline)) { fence(); asm volatile("s_barrier" ::: "memory"); fence(); };
        auto read_rows = [&](const uint8_t* st, int s, int h) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < RS; ++i) xa[h][i] = *reinterpret_cast<const u32x4_t*>(st + a_base + (h * RS + i) * 16 * KB + (f_off ^ (s << 6)));
        };
        auto read_weights = [&](const uint8_t* st, int s) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 4; ++t) xw[s][t] = *reinterpret_cast<const u32x4_t*>(st + G::REGION_W + b_pos[t >> 1] * KB + (t & 1) * 16 * KB + (f_off ^ (s << 6)));
        };
        auto turn = [&](int s, int h) __attribute__((always_inline)) {
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < RS; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t) mma16(acc16[(h * RS + i) / 2][(h * RS + i) % 2][t], xw[s][t], xa[h][i]);
#pragma unroll
            for (int i = 0; i < RS; ++i)                   // (the MFMAs stay in this turn instead of moving to where their results are used)
#pragma unroll
                for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(acc16[(h * RS + i) / 2][(h * RS + i) % 2][t]));
            __builtin_amdgcn_s_setprio(0);
        };
        __builtin_amdgcn_s_waitcnt(LGKM);
        if (wm) barrier();
        while (true) {
            const bool last = ks == nks - 1;
            const uint8_t* st = smem + stg * G::STAGE;
            read_weights(st, 0);
            read_rows(st, 0, 0);
            fence();
            issue_some(EARLY, EARLY + 2, pk, left);
            fence();
            read_rows(st, 0, 1);
            fence();
            __builtin_amdgcn_s_waitcnt(LGKM | RS << 8);    // all but the upper rows
            barrier();
            turn(0, 0);
            barrier();
            read_weights(st, 1);
            read_rows(st, 1, 0);
            fence();
            issue_some(EARLY + 2, OPS, pk, left);
            __builtin_amdgcn_s_waitcnt(LGKM | (4 + RS) << 8);            // slice 0
            barrier();
            turn(0, 1);
            barrier();
            read_rows(st, 1, 1);
            fence();
            __builtin_amdgcn_s_waitcnt(LGKM);
            barrier();                                     // (waves 4..7 come to it one turn later: then the stage is free)
            turn(1, 0);
            barrier();
            left = stg;
            stg = stg + 1 == G::NS ? 0 : stg + 1;
            advance();
            fence();
            issue_some(0, EARLY, pk, left);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((G::NS - 2) * OPS + EARLY) : "memory");     // the next step, this wave's part
            barrier();
            turn(1, 1);
            ++ks;
            // Epilogue: both waves of a SIMD at the same time, between the same two barriers
            if (!(last && wm)) barrier();
            if (last) {
                store_tile();
                if (wm) barrier();
                if (!next_tile()) break;
                __builtin_amdgcn_s_waitcnt(LGKM);
            }
        }
        if (!wm) barrier();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no transfer may still be writing this block's LDS when it ends
        return;
    }

    u32x4_t fa[2][MT], fb[2][2];                           // fragment double buffer (slice parity)
    int sa[MT][2], sb[2][2];                               // FP4: scale words of the step, [.][0] slices 0-1, [.][1] slices 2-3
    auto read_frags = [&](int s, int slot, const uint8_t* st) __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) fa[slot][mt] = *reinterpret_cast<const u32x4_t*>(st + a_base + mt * 32 * KB + (f_off0 ^ (s << 5)));
#pragma unroll
        for (int t = 0; t < 2; ++t) fb[slot][t] = *reinterpret_cast<const u32x4_t*>(st + G::REGION_W + b_pos[t] * KB + (f_off0 ^ (s << 5)));
    };
    // the same reads in four parts (part 0: row tile 0 and both column tiles, part 1: row tile 1, ...)
    auto read_frags_part = [&](int part, int s, int slot, const uint8_t* st) __attribute__((always_inline)) {
        fa[slot][part] = *reinterpret_cast<const u32x4_t*>(st + a_base + part * 32 * KB + (f_off0 ^ (s << 5)));
        if (part == 0) {
#pragma unroll
            for (int t = 0; t < 2; ++t) fb[slot][t] = *reinterpret_cast<const u32x4_t*>(st + G::REGION_W + b_pos[t] * KB + (f_off0 ^ (s << 5)));
        }
    };
    u32x2_t ra[MT], rb[2];                                 // FP4: raw scale words as read from LDS
    auto read_scales = [&](int stage) __attribute__((always_inline)) {
        if constexpr (FP4) {
            const uint8_t* sc = smem + G::SC_BASE + stage * G::SC_STAGE;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) ra[mt] = *reinterpret_cast<const u32x2_t*>(sc + (wm * (32 * MT) + mt * 32 + li) * 8);
#pragma unroll
            for (int t = 0; t < 2; ++t) rb[t] = *reinterpret_cast<const u32x2_t*>(sc + G::SC_W + (b_pos[t] + li) * 8);
        }
    };
    auto read_scales_part = [&](int part, int stage) __attribute__((always_inline)) {   // the same in four parts, like the fragments
        if constexpr (FP4) {
            const uint8_t* sc = smem + G::SC_BASE + stage * G::SC_STAGE;
            ra[part] = *reinterpret_cast<const u32x2_t*>(sc + (wm * (32 * MT) + part * 32 + li) * 8);
            if (part == 0) {
#pragma unroll
                for (int t = 0; t < 2; ++t) rb[t] = *reinterpret_cast<const u32x2_t*>(sc + G::SC_W + (b_pos[t] + li) * 8);
            }
        }
    };
    auto take_scales = [&]() __attribute__((always_inline)) {     // this lane's byte pair of each word (op_sel picks the byte)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            sa[mt][0] = FP4 ? (int)(ra[mt].x >> (half * 8)) : 0;
            sa[mt][1] = FP4 ? (int)(ra[mt].y >> (half * 8)) : 0;
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            sb[t][0] = FP4 ? (int)(rb[t].x >> (half * 8)) : 0;
            sb[t][1] = FP4 ? (int)(rb[t].y >> (half * 8)) : 0;
        }
    };
    read_scales(0);
    read_frags(0, 0, smem);
    take_scales();

    while (true) {
        const bool last = ks == nks - 1;
        const bool full = !(tail_half && (STARTS ? ck : ks) == nks - 1);           // all four K-slices present
        const uint8_t* st = smem + stg * G::STAGE;

        // MFMAs of slice s out of fragment slot s&1.  PRODUCE 1: after each row tile's MFMAs one weight
        // transfer (and the two scale transfers) of producer step pk into the other stage; PRODUCE 2:
        // one activation transfer of the producer's new step into the stage just released.
        // Slice s multiplies out of fragment slot s&1.  The fragments of the following slice (next = s+1,
        // or next = 4: the first slice of the next step, with its scales, out of the stage that has just
        // been published) are requested into the other slot, a quarter of them after each row tile's MFMAs
        // (one burst of six reads behind the first row tile measured 0.5-1 % slower: the LDS also takes
        // the transfers' writes); the wait in front of this slice's first MFMA does not cover the new requests.
        auto slice = [&](int s, int produce, bool multiply, int next) __attribute__((always_inline)) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (multiply) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (s & 1) mma<FP4, 2>(acc[mt][t], fb[s & 1][t], fa[s & 1][mt], sb[t][s >> 1], sa[mt][s >> 1]);
                        else mma<FP4, 0>(acc[mt][t], fb[s & 1][t], fa[s & 1][mt], sb[t][s >> 1], sa[mt][s >> 1]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (next >= 0) {
                    if (next < 4) read_frags_part(mt, next, next & 1, st);
                    else { read_scales_part(mt, stg); read_frags_part(mt, 0, 0, smem + stg * G::STAGE); }
                }
                if (produce == 1) {
                    if (FP4 && mt < 2) issue(mt, pk, left);
                    if (FP4 && MT == 1) issue(1, pk, left);
#pragma unroll
                    for (int q = mt * G::OPS_W / MT; q < (mt + 1) * G::OPS_W / MT; ++q) issue(6 + q, pk, left);
                } else if (produce == 2) {
                    issue(2 + mt, pk, left);              // (left: the stage this step has just left)
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        slice(0, 1, true, 1);
        slice(1, 0, true, 2);                             // (half step: slice 2 holds stale bytes that are never multiplied)
        if (full) slice(2, 0, true, 3);
        __builtin_amdgcn_sched_barrier(0);
        // the next step has landed; with more than two stages the transfers of those behind it stay in flight (hence no
        // __syncthreads(), whose release waits for every transfer); this wave's reads of the released stage are done
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((G::NS - 2) * OPS) : "memory");
        left = stg;
        stg = stg + 1 == G::NS ? 0 : stg + 1;
        advance();
        __builtin_amdgcn_sched_barrier(0);
        slice(3, 2, full, 4);                             // (half step: the producer's transfers and the requests only)
        __builtin_amdgcn_sched_barrier(0);
        take_scales();

        ++ks;
        if constexpr (STARTS) ck = ck + 1 == nks ? 0 : ck + 1;
        if (last) {
            store_tile();
            if (!next_tile()) break;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no transfer may still be writing this block's LDS when it ends
}

// Which tiles: the whole rounds of 256 x 256 tiles first (a round = one tile on every block; the 256-row tile costs the least
// per row), then what is left in the smallest shape that still fits ONE round.  A last round of 256-row tiles lasts as long
// as a full one, however empty it is; a round of 192-row tiles lasts 0.80 of it, 128-row tiles 0.63, 64-row tiles 0.41 (gate/up of 256 tiles,
// K = 2048, BF16 53.9, 43.1, 33.7 and 22.3 us; FP4 22.4, 18.1, 14.2 and 10.3).  Measured against 256-row tiles alone, BF16 gate/up,
// I = 1408: 3 548 rows (all in 192-row tiles) 47.5 -> 42.0 us, FP4 18.7 -> 17.5; 13 162 rows 140.8 -> 130.4, 36 183 rows 342.9 -> 331.0.
// Against the best single shape the choice is within 3 % at most sizes; further off: BF16 5 000 rows gate/up 64.9 against 61.3 in 128-row
// tiles, I = 768 1 000 rows down 13.6 / 11.9 (128), 10 000 rows down 40.3 / 36.2 (192); FP4 5 000 rows gate/up 27.8 / 23.7 (128), 7 500 rows
// down 25.5 / 21.0 (128).
// With FP4 operands the second pipeline start eats what 192- or 128-row tiles would save behind whole rounds (down of 11 000 rows,
// K = 768, 19.7 -> 21.8 us, of 13 162 rows, K = 1408, 30.7 -> 32.8; gate/up between 4 % less and 3 % more), so there they are used only
// when they hold all rows.  A block has at most one tile of a chosen small shape; forced to take
// several, 64 x 128 tiles need at least four K-steps: their producer runs up to five steps ahead, and a tile's gather entries
// are fetched one tile ahead.
template <bool FP4, bool GATEUP, bool GATHER>
__device__ __forceinline__ void tile_body(const GemmParams& p, uint8_t* smem) {
    if (p.start_word && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(p.start_word, (unsigned long long)p.start_seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = 0;
    if (lane < p.n_local) { lo = p.offs[lane]; hi = p.offs[lane + 1]; }
    const bool nt_out = stream_output<FP4>(p);
    const int slots = gridDim.x;
    const int nt = GATEUP ? p.n_out / 128 : (p.n_out + 255) / 256;     // column tiles of 256 weight rows
    // Which rows go in 256-row tiles, and the shape of the tiles of the rest.
    int cut = 0x7FFFFFFF, rest = 4;                        // rows [0, cut) of the rank: 256-row tiles
    if (p.tile_mode == 0) {
        const int mine = tiles_of<256>(lo, hi), cum = wave_inclusive_scan(mine);       // row tiles of the experts up to this lane's
        const int m_tiles = __builtin_amdgcn_readlane(cum, 63);
        int c = 0;                                         // first row behind the whole rounds of 256-row tiles
        if (m_tiles * nt >= slots) {
            const int m_keep = m_tiles * nt / slots * slots / nt;      // row tiles that fill those rounds
            const int before = cum - mine;
            const unsigned long long holds = __ballot(before <= m_keep && m_keep < cum);
            c = holds == 0 ? 0x7FFFFFFF : __builtin_amdgcn_readlane(lo + (m_keep - before) * 256, __ffsll((long long)holds) - 1);
        }
        const int tail = max(lo, c);
        const int nt64 = GATEUP ? p.n_out / 32 : p.n_out / 64, nt128 = nt64 / 2;      // column tiles of 64 and 128 weight rows
        const int n64 = wave_sum(tiles_of<64>(tail, hi));
        rest = 4;
        if (n64 * nt <= slots) rest = !FP4 && n64 * nt64 <= slots ? 5 : n64 * nt128 <= slots ? 0 : 1;      // (FP4 weights are a quarter of the bytes)
        else if (!FP4 || c == 0) {
            if (wave_sum(tiles_of<128>(tail, hi)) * nt <= slots) rest = 2;
            else if (wave_sum(tiles_of<192>(tail, hi)) * nt <= slots) rest = 3;
        }
        cut = rest == 4 ? 0x7FFFFFFF : c;
    } else if (p.tile_mode != 4) {
        cut = 0;
        rest = p.tile_mode != 5 ? p.tile_mode : p.K >= (FP4 ? 1024 : 256) ? 0 : 1;
    }
    if (cut > 0) tile_phase<FP4, GATEUP, GATHER, 4, 256>(p, smem, min(lo, cut), min(hi, cut), nt_out);
    if (cut < 0x7FFFFFFF) {
        if (rest == 3) tile_phase<FP4, GATEUP, GATHER, 3, 256>(p, smem, max(lo, cut), max(hi, cut), nt_out);
        else if (rest == 2) tile_phase<FP4, GATEUP, GATHER, 2, 256>(p, smem, max(lo, cut), max(hi, cut), nt_out);
        else if (rest == 1) tile_phase<FP4, GATEUP, GATHER, 1, 256>(p, smem, max(lo, cut), max(hi, cut), nt_out);
        else if (rest == 0) tile_phase<FP4, GATEUP, GATHER, 1, 128>(p, smem, max(lo, cut), max(hi, cut), nt_out);
        else if constexpr (!FP4) tile_phase<FP4, GATEUP, GATHER, 1, 64>(p, smem, max(lo, cut), max(hi, cut), nt_out);
    }
}

template <bool FP4, bool GATEUP, bool GATHER>
__global__ void __launch_bounds__(512, 1) ffn_tile_kernel(const GemmParams p) {
    extern __shared__ __align__(16) uint8_t smem[];
    tile_body<FP4, GATEUP, GATHER>(p, smem);
}

// The same, in the precision that the routing statistics will ask for: launched before the host knows it, so that the GPU
// does not idle while the host waits for the statistics, decides and launches.
template <bool GATEUP, bool GATHER>
__global__ void __launch_bounds__(512, 1) ffn_tile_either_kernel(const GemmParams bf16, const GemmParams fp4, const PrecisionSource prec) {
    extern __shared__ __align__(16) uint8_t smem[];
    if (precision_is_fp4(prec)) tile_body<true, GATEUP, GATHER>(fp4, smem);
    else tile_body<false, GATEUP, GATHER>(bf16, smem);
}

// One persistent block per CU, a multiple of 8 (XCDs); a prefetching layer call leaves some CUs to the weight encoder.
static unsigned tile_grid(const GemmParams& p, bool gate_up, long long max_rows, const Ctx* c) {
    const long long narrowest = gate_up ? p.n_out / 32 : p.n_out / 64;    // column tiles of the narrowest shape
    const long long total_max = ((max_rows + 63) / 64 + p.n_local) * narrowest;
    const long long avail = (long long)c->num_cus - c->gemm_reserve;
    const long long slots = avail >= 16 ? 8ll * (c->gemm_reserve > 0 ? avail / 8 : (avail + 7) / 8) : 8;
    return (unsigned)(total_max < slots ? 8 * ((total_max + 7) / 8) : slots);
}
constexpr size_t max_size(size_t a, size_t b) { return a > b ? a : b; }
constexpr size_t kTileLds = max_size(TileGeo<4, 256>::LDS_BYTES, max_size(max_size(TileGeo<3, 256>::LDS_BYTES, TileGeo<2, 256>::LDS_BYTES), max_size(TileGeo<1, 128>::LDS_BYTES, TileGeo<1, 64>::LDS_BYTES)));
static_assert(TileGeo<1, 256>::LDS_BYTES <= kTileLds && kTileLds <= 160 * 1024, "LDS");

template <typename K>
static int raise_lds_limit(K kernel, std::atomic<unsigned long long>& seen, const Ctx* c) {
    if (first_use_on_device(seen, c->device)) {                     // (setting it twice from two threads is harmless)
        REALB_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
        mark_used_on_device(seen, c->device);
    }
    return REALB_OK;
}

// Column tiles per width, as divisors: exact for every width, and no division on the device (layer calls of 24 and 1000 tokens
// against divisors found there: 1 % less at the most, which is what the runs of one side differ by).
static void set_column_tiles(GemmParams& p, bool gate_up) {
    for (int i = 0; i < 3; ++i) {
        const int cols = (gate_up ? 128 : 256) >> i;                // output columns of a tile
        division_magic((p.n_out + cols - 1) / cols, &p.col_magic[i], &p.col_shift[i]);
    }
}

// mode: GemmParams::tile_mode
template <bool FP4, bool GATEUP, bool GATHER>
static int launch_tile(GemmParams p, long long max_rows, const Ctx* c, hipStream_t s, int mode) {
    p.tile_mode = mode;
    set_column_tiles(p, GATEUP);
    static std::atomic<unsigned long long> seen{0};                 // per instantiation, one bit per device
    const int rc = raise_lds_limit(&ffn_tile_kernel<FP4, GATEUP, GATHER>, seen, c);
    if (rc != REALB_OK) return rc;
    hipLaunchKernelGGL((ffn_tile_kernel<FP4, GATEUP, GATHER>), dim3(tile_grid(p, GATEUP, max_rows, c)), dim3(512), kTileLds, s, p);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}
template <bool GATEUP, bool GATHER>
static int launch_tile_either(GemmParams b, GemmParams f, const PrecisionSource& prec, long long max_rows, const Ctx* c, hipStream_t s, int mode) {
    b.tile_mode = f.tile_mode = mode;
    set_column_tiles(b, GATEUP);
    set_column_tiles(f, GATEUP);
    static std::atomic<unsigned long long> seen{0};
    const int rc = raise_lds_limit(&ffn_tile_either_kernel<GATEUP, GATHER>, seen, c);
    if (rc != REALB_OK) return rc;
    hipLaunchKernelGGL((ffn_tile_either_kernel<GATEUP, GATHER>), dim3(tile_grid(b, GATEUP, max_rows, c)), dim3(512), kTileLds, s, b, f, prec);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}

// Block tile choices (selector g_tile): 0 = the direct-to-LDS kernel above with the shapes it picks (or with the one that
// the context names, see realb_set_gemm_tile_shape), 16 = with 256-row tiles only; the register-staged kernel with 64-byte K-steps as 2 = 256x128, 4 waves,
// two blocks per CU, or 8 = 256x256, 8 waves of 128x64, one block per CU.
template <bool FP4, bool GATEUP, int WN, int WGN, int MINB>
static int launch_gemm_geo(GemmParams p, long long max_rows, const Ctx* c, hipStream_t s) {
    using G = Geo<WN, WGN>;
    const int num_cus = c->num_cus;
    p.n_tiles_n = GATEUP ? p.n_out / G::GC : p.n_out / G::BNW;
    const size_t lds = 2 * (size_t)G::STAGE;
    const size_t lds_cap = MINB == 2 ? 80 * 1024 : 160 * 1024;
    static std::atomic<unsigned long long> attr_seen{0};            // per instantiation, one bit per device
    if (first_use_on_device(attr_seen, c->device)) {
        REALB_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&ffn_gemm_kernel<FP4, GATEUP, WN, WGN, MINB>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_cap));
        mark_used_on_device(attr_seen, c->device);
    }
    const long long m_tiles_max = (max_rows + BM - 1) / BM + p.n_local;
    const long long total_max = m_tiles_max * p.n_tiles_n;
    const long long slots = 8ll * (((long long)num_cus * MINB + 7) / 8);   // one block per residency slot, multiple of 8 (XCDs)
    const long long all_tiles = 8 * ((total_max + 7) / 8);
    const long long grid = (FP4 || total_max < slots) ? all_tiles : slots;                // FP4: one tile per block
    REALB_REQUIRE(grid < (1ll << 31), REALB_ECAP, "too many tiles");
    REALB_REQUIRE(lds <= lds_cap, REALB_ESHAPE, "K=%d needs %zu bytes of LDS", p.K, lds);
    hipLaunchKernelGGL((ffn_gemm_kernel<FP4, GATEUP, WN, WGN, MINB>), dim3((unsigned)grid), dim3(G::NT), lds, s, p);
    REALB_HIP(hipGetLastError());
    return REALB_OK;
}

static std::atomic<int> g_tile{0};    // 0 = automatic; another value forces a kernel (set through realb_set_gemm_tile)

template <bool FP4, bool GATEUP>
static int launch_gemm(const GemmParams& p, long long max_rows, const Ctx* c, hipStream_t s) {
    const int forced = g_tile.load(std::memory_order_relaxed);
    if (forced == 0 || forced == 16)
        return launch_tile<FP4, GATEUP, false>(p, max_rows, c, s, forced == 16 ? 4 : c->gemm_shape);
    if (forced == 8 && (GATEUP || p.n_out % 256 == 0)) return launch_gemm_geo<FP4, GATEUP, 2, 4, 1>(p, max_rows, c, s);
    return launch_gemm_geo<FP4, GATEUP, 2, 2, 2>(p, max_rows, c, s);
}

static int layer_tile_mode() { return g_tile.load(std::memory_order_relaxed) == 16 ? 4 : 0; }

// Whether the layer call's gate/up GEMM can fetch its activation rows from the token matrix (kernel selection, 32-bit row
// offsets); if not, the caller materialises the permuted rows and uses the plain GEMMs.
bool gate_up_gather_supported(const Ctx* c, int T, bool fp4) {
    const long long bytes = (long long)T * c->cfg.H * (fp4 ? 1 : 4) / 2;
    const int forced = g_tile.load(std::memory_order_relaxed);
    return (forced == 0 || forced == 16) && T > 0 && bytes < (1ll << 32);
}

// Gate/up GEMM of a layer call: activation rows come from x [T,H], or from the tokens' codes and scales (row index = token
// index), through row_to_assign.
int launch_layer_gate_up(Ctx* c, const PrecisionSource& prec, const realb_layer_io* io, bool announce, hipStream_t s) {
    const int H = c->cfg.H, I = c->cfg.I;
    GemmParams b{(const uint8_t*)io->x, nullptr, (const uint8_t*)io->w13, nullptr, (uint8_t*)io->h_mid, nullptr, io->expert_offsets, c->n_local,
                 H, 2 * I, I, 0, io->row_to_assign, 0, 0, nullptr, 0, 0};
    division_magic(c->cfg.k, &b.src_magic, &b.src_shift);
    if (announce) { b.start_word = c->start_word; b.start_seq = c->start_seq; }
    GemmParams f = b;
    f.A = io->x_q; f.As = io->x_s; f.W = io->w13_q; f.Ws = io->w13_s; f.outs = io->h_s;
    if (prec.fixed < 0) return launch_tile_either<true, true>(b, f, prec, io->max_rows, c, s, layer_tile_mode());
    return prec.fixed == REALB_FP4 ? launch_tile<true, true, true>(f, io->max_rows, c, s, layer_tile_mode())
                                   : launch_tile<false, true, true>(b, io->max_rows, c, s, layer_tile_mode());
}

int launch_layer_down(Ctx* c, const PrecisionSource& prec, const realb_layer_io* io, hipStream_t s) {
    const int H = c->cfg.H, I = c->cfg.I;
    GemmParams b{(const uint8_t*)io->h_mid, nullptr, (const uint8_t*)io->w2, nullptr, (uint8_t*)io->y_rows, nullptr, io->expert_offsets, c->n_local,
                 I, H, H, 0, nullptr, 0, 0, nullptr, 0, 0};
    GemmParams f = b;
    f.As = io->h_s; f.W = io->w2_q; f.Ws = io->w2_s;
    if (prec.fixed < 0) return launch_tile_either<false, false>(b, f, prec, io->max_rows, c, s, layer_tile_mode());
    return prec.fixed == REALB_FP4 ? launch_tile<true, false, false>(f, io->max_rows, c, s, layer_tile_mode())
                                   : launch_tile<false, false, false>(b, io->max_rows, c, s, layer_tile_mode());
}

}  // namespace realb

using namespace realb;

extern "C" int realb_set_gemm_tile(int wn) {
    REALB_REQUIRE(wn == 0 || wn == 2 || wn == 8 || wn == 16, REALB_EINVAL, "tile selector must be 0, 2, 8 or 16");
    g_tile.store(wn, std::memory_order_relaxed);
    return REALB_OK;
}

extern "C" int realb_set_gemm_tile_shape(realb_ctx* ctx, int shape) {
    REALB_REQUIRE(ctx != nullptr, REALB_EINVAL, "ctx is NULL");
    REALB_REQUIRE(shape == 0 || shape == 1 || shape == 2 || shape == 3 || shape == 5, REALB_EINVAL, "tile shape must be 0, 1, 2, 3 or 5");
    reinterpret_cast<Ctx*>(ctx)->gemm_shape = shape;
    return REALB_OK;
}

static int ffn_stages(realb_ctx* ctx, int prec, int stages, const int32_t* expert_offsets, int n_local, long long max_rows,
                      const void* x, const uint8_t* x_s, const void* w13, const uint8_t* w13_s, const void* w2,
                      const uint8_t* w2_s, void* h_mid, uint8_t* h_s, void* y_rows, void* stream) {
    REALB_REQUIRE(ctx && expert_offsets, REALB_EINVAL, "NULL argument");
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    REALB_REQUIRE(prec == REALB_BF16 || prec == REALB_FP4, REALB_EINVAL, "bad precision %d", prec);
    REALB_REQUIRE(n_local >= 0 && n_local <= c->n_local, REALB_ECAP, "n_local=%d exceeds the context's %d", n_local, c->n_local);
    REALB_REQUIRE(max_rows >= 0, REALB_EINVAL, "max_rows < 0");
    if (max_rows == 0 || n_local == 0) return REALB_OK;
    const bool s1 = stages & 1, s2 = stages & 2;
    REALB_REQUIRE(h_mid && (!s1 || (x && w13)) && (!s2 || (w2 && y_rows)), REALB_EINVAL, "NULL argument");
    REALB_REQUIRE(prec == REALB_BF16 || (h_s && (!s1 || (x_s && w13_s)) && (!s2 || w2_s)), REALB_EINVAL,
                  "NULL scale tensor on the FP4 path");
    if (prec == REALB_BF16) x_s = w13_s = w2_s = h_s = nullptr;      // ignored
    const int H = c->cfg.H, I = c->cfg.I;
    hipStream_t s = as_stream(stream);
    GemmParams g1{(const uint8_t*)x, x_s, (const uint8_t*)w13, w13_s, (uint8_t*)h_mid, h_s, expert_offsets, n_local, H, 2 * I, I, 0, nullptr, 0, 0, nullptr, 0, 0};
    GemmParams g2{(const uint8_t*)h_mid, h_s, (const uint8_t*)w2, w2_s, (uint8_t*)y_rows, nullptr, expert_offsets, n_local, I, H, H, 0, nullptr, 0, 0, nullptr, 0, 0};
    int rc = REALB_OK;
    if (prec == REALB_FP4) {
        if (s1) rc = launch_gemm<true, true>(g1, max_rows, c, s);
        if (rc == REALB_OK && s2) rc = launch_gemm<true, false>(g2, max_rows, c, s);
    } else {
        if (s1) rc = launch_gemm<false, true>(g1, max_rows, c, s);
        if (rc == REALB_OK && s2) rc = launch_gemm<false, false>(g2, max_rows, c, s);
    }
    return rc;
}

extern "C" int realb_grouped_moe_ffn(realb_ctx* ctx, int prec, const int32_t* expert_offsets, int n_local, long long max_rows,
                                     const void* x, const uint8_t* x_s, const void* w13, const uint8_t* w13_s,
                                     const void* w2, const uint8_t* w2_s, void* h_mid, uint8_t* h_s, void* y_rows,
                                     void* stream) {
    return ffn_stages(ctx, prec, 3, expert_offsets, n_local, max_rows, x, x_s, w13, w13_s, w2, w2_s, h_mid, h_s, y_rows, stream);
}

extern "C" int realb_grouped_moe_ffn_gate_up(realb_ctx* ctx, int prec, const int32_t* expert_offsets, int n_local,
                                             long long max_rows, const void* x, const uint8_t* x_s, const void* w13,
                                             const uint8_t* w13_s, void* h_mid, uint8_t* h_s, void* stream) {
    return ffn_stages(ctx, prec, 1, expert_offsets, n_local, max_rows, x, x_s, w13, w13_s, nullptr, nullptr, h_mid, h_s, nullptr, stream);
}

extern "C" int realb_grouped_moe_ffn_down(realb_ctx* ctx, int prec, const int32_t* expert_offsets, int n_local,
                                          long long max_rows, const void* h_mid, const uint8_t* h_s, const void* w2,
                                          const uint8_t* w2_s, void* y_rows, void* stream) {
    return ffn_stages(ctx, prec, 2, expert_offsets, n_local, max_rows, nullptr, nullptr, nullptr, nullptr, w2, w2_s,
                      const_cast<void*>(h_mid), const_cast<uint8_t*>(h_s), y_rows, stream);
}
