// Device code shared by the grouped GEMM kernels of ffn.hip: kernel parameters, the MFMA step, the order of
// weight rows inside a tile, the register epilogues and their stores, direct-to-LDS transfers.
#pragma once
#include "common.h"
#include "mxfp4_device.h"
#include <atomic>

namespace realb {

// Devices (bit = device index) on which a kernel instantiation has had its dynamic-LDS limit raised.
inline bool first_use_on_device(std::atomic<unsigned long long>& seen, int device) {
    const unsigned long long bit = 1ull << (device & 63);
    return (seen.load(std::memory_order_acquire) & bit) == 0;
}
inline void mark_used_on_device(std::atomic<unsigned long long>& seen, int device) {
    seen.fetch_or(1ull << (device & 63), std::memory_order_release);
}

typedef __attribute__((ext_vector_type(8))) int v8i_t;
typedef __attribute__((ext_vector_type(16))) float v16f_t;
typedef __attribute__((ext_vector_type(4))) float v4f_t;
typedef __attribute__((ext_vector_type(8))) __bf16 v8bf_t;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;

struct GemmParams {
    const uint8_t* A;        // activations: bf16 [rows,K] or fp4 codes [rows,K/2]
    const uint8_t* As;       // fp4: scales [rows,K/32]
    const uint8_t* W;        // weights: [n_local, w_rows, K] in the same encoding
    const uint8_t* Ws;
    uint8_t* out;            // gate/up: h (bf16 [rows,I] or codes [rows,I/2]); down: y bf16 [rows,H]
    uint8_t* outs;           // gate/up fp4: h scales [rows,I/32]
    const int32_t* offs;     // expert_offsets [n_local+1]
    int n_local;
    int K;                   // contraction length in elements
    int w_rows;              // weight rows per expert (2I or H)
    int n_out;               // output columns (I or H)
    int n_tiles_n;           // column tiles (I/GC or H/BNW), register-staged kernel
    const int32_t* row_src;  // gathering gate/up GEMM only: row_to_assign; row r's activations are A[row_src[r] / k]
    uint32_t src_magic;      //   a / k == (a * src_magic) >> src_shift for 0 <= a < 2^31  (k = experts per token)
    int src_shift;
    unsigned long long* start_word;   // host-coherent, or NULL: the kernel's first block writes start_seq there
    int start_seq;
    int tile_mode;           // direct-to-LDS kernel: 0 = tile shapes chosen on the device, 4 / 3 / 2 / 1 = 64 times that many rows of
                             //   256 weight rows, 5 = 64 x 128 tiles only
    uint32_t col_magic[3];   // direct-to-LDS kernel: t / (column tiles) for tiles of 256, 128 and 64 weight rows, as src_magic.  From the host:
    int col_shift[3];        //   two dependent divisions on the device stood in front of every block's first transfer
};

// Exact division of 0 <= a < 2^31 by a constant 1 <= k <= 2^30 through one multiplication: with s = ceil(log2 k) and
// m = floor(2^(31+s) / k) + 1 < 2^32, the excess m*k - 2^(31+s) is at most k <= 2^s, so a*m / 2^(31+s) exceeds
// a/k by less than 1/k and the floors agree.
inline void division_magic(int k, uint32_t* magic, int* shift) {
    int s = 0;
    while ((1 << s) < k) ++s;
    *magic = (uint32_t)((1ull << (31 + s)) / (unsigned)k + 1);
    *shift = 31 + s;
}
__device__ __forceinline__ int div_by_magic(int a, uint32_t magic, int shift) {
    return (int)(((unsigned long long)(uint32_t)a * magic) >> shift);
}

// acc += W_tile (A operand, 32 weight rows) x X_tile^T (B operand, 32 activation rows)
template <bool FP4, int OPSEL>
__device__ __forceinline__ void mma(v16f_t& acc, const u32x4_t& w, const u32x4_t& x, int sw, int sx) {
    if constexpr (FP4) {
        v8i_t a8 = {(int)w.x, (int)w.y, (int)w.z, (int)w.w, 0, 0, 0, 0};
        v8i_t b8 = {(int)x.x, (int)x.y, (int)x.z, (int)x.w, 0, 0, 0, 0};
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, acc, 4, 4, OPSEL, sw, OPSEL, sx);
    } else {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_t, w), __builtin_bit_cast(v8bf_t, x), acc, 0, 0, 0);
    }
}

// The same for BF16 on 16 x 16 tiles: 16 weight rows x 16 activation rows over 64 bytes of K.  Lane l feeds the 16 bytes of part l/16
// of row l%16 of either operand and gets output element (weight row 4*(l/16) + r, activation row l%16) in register r.  Its sums
// are those of the 32 x 32 form bit for bit.  What it is for: large products are held back by power, and for the same
// products this form moves half as many accumulators through the register file.  Registers only, random operands, sustained:
// 2041 against 1822 TFLOP/s (operands of zeros: 2405 / 2424).  FP4 has such a form too (7360 against 6700), but there a lane needs its
// scale of each of twelve row tiles, not six, and with the loop that goes with it FP4 gate/up took 138 us instead of 122.
__device__ __forceinline__ void mma16(v4f_t& acc, const u32x4_t& w, const u32x4_t& x) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf_t, w), __builtin_bit_cast(v8bf_t, x), acc, 0, 0, 0);
}

// two floats -> two BF16 (nearest even) in one dword, first in the low half
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf2;
    bf2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

// Weight row (within the expert) of row `br` of the block's weight tile.
template <bool GATEUP, int GC>
__device__ __forceinline__ int w_tile_row(int br, int n0, int I_up) {
    if constexpr (GATEUP) return br < GC ? n0 + br : I_up + n0 + (br - GC);
    else return n0 + br;
}

// LDS slot of weight-tile row br: inside each group of 32 rows, row 16h + 4g + q sits in slot
// 8g + 4h + q.  MFMA output row i = 8g + 4h + q lands in lane half h, register 4g + q, so the
// lane's 16 registers are weight rows 16h .. 16h+15 of the tile, in order.
__device__ __forceinline__ int w_slot(int br) { return (br & ~31) | (((br >> 2) & 3) << 3) | (((br >> 4) & 1) << 2) | (br & 3); }
// inverse: the weight-tile row that lane li (slot li) feeds to the MFMA
__device__ __forceinline__ int w_row_of_lane(int li) { return (((li >> 2) & 1) << 4) | ((li >> 3) << 2) | (li & 3); }

// The order for 16 x 16 tiles, of which two neighbouring ones make a group of 32 rows: the weight-tile row in slot 16a + 4g + q is
// 8g + 4a + q, so that MFMA output rows 4g + q of the tiles a = 0, 1 -- lane group g, register q -- are 8 consecutive ones.
__device__ __forceinline__ int w_row_of_slot16(int slot) { return (((slot >> 2) & 3) << 3) | (((slot >> 4) & 1) << 2) | (slot & 3); }

// K-step (128 bytes of every operand row) at which the sum of an output column starts; from there it runs to the row's end and
// on from the row's front.
// BF16: the front, for every column.  FP32 sums of BF16 products round, and a row's bits shall depend on its expert alone -- not on
// the batch, the tile shape, the expert's local slot (the EP degree) or the column.  What that leaves: blocks that work side by
// side ask for the same part of every row at the same time, that is of few HBM channels.  Starts that differ by slot and column
// took a layer call of 24 tokens, weights from HBM, from 44.0 to 40.0 us (1000 tokens 71.2 -> 69.4); starts by column alone 42.9
// us, but with cached weights 36.0 -> 36.8, and 16 384 tokens on a rank without load 171.7 -> 177.4 us.
// FP4 down: neighbouring column tiles start one step apart, so that they read different parts of the weight rows.  The order
// depends on the column alone.  H = 2048, before -> after: 249 000 rows, K = 768 359 -> 297 us; 100 000 rows, K = 1024 153 -> 137,
// K = 2048 242 -> 228; but 20 000 rows, K = 1408 43.2 -> 44.1, K = 2048 50.8 -> 53.6 us; no difference at 600 and 4000 rows.
// FP4 gate/up: the front; such starts gained nothing from 150 to 36 000 rows and cost up to 3 % (H = 2048, I = 512, 20 000 rows
// 32.4 -> 33.2 us).
template <bool FP4, bool GATEUP>
constexpr bool kHasStarts = FP4 && !GATEUP;
template <bool FP4, bool GATEUP>
__device__ __forceinline__ int k_start(int n0, int nks) {
    if constexpr (kHasStarts<FP4, GATEUP>) return (int)((uint32_t)(n0 >> 8) % (uint32_t)nks);      // (256: column tile of the wide shapes)
    else return 0;
}

struct TileInfo {
    int e;        // local expert
    int row0;     // first activation row of the tile
    int seg_hi;   // end of the expert's row segment
    int n0;       // first output column of the tile
};

// BF16 outputs larger than what the memory-side cache would keep for the kernel that reads them next are streamed past it with
// non-temporal stores (uniform per launch): from 160 MiB on, FP4 GEMMs with K >= 1024 from 136 MiB on.  Layer calls, FP4 limit 160 / 64 MiB,
// H = 2048, us, with three sets of all buffers in turn, and with one set of buffers and three of weights and tokens; two boxes of the
// same kind differ by 1 % in what the limit gives:
//   K = 1408: 80 MiB 185.8 / 183.9, 178.5 / 179.0; 100 MiB 215.0 / 215.2, 211.6 / 213.1; 125 MiB 252.0 / 251.9, 248.8 / 250.3; 133 MiB 264.2 / 261.7,
//             261.5 / 260.1; 141 MiB 279.6 / 275.1, 275.3 / 274.4; 150 MiB 288.5 / 285.1, 284.8 / 284.0
//   K = 1024: 68 MiB 139.1 / 139.4, 134.0 / 135.4; 100 MiB 172.1 / 174.4, 170.4 / 173.4; 125 MiB 205.3 / 206.3, 203.9 / 205.8; 133 MiB 213.4 / 211.6,
//             209.7 / 209.9; 141 MiB 225.0 / 220.5, 219.7 / 217.4; 150 MiB 232.2 / 227.3, 227.7 / 226.3
//   K = 896:  141 MiB 205.3 / 202.5, 201.0 / 200.4;  K = 768: 141 MiB 190.1 / 187.7, 185.5 / 186.5; 158 MiB 205.0 / 205.2, 201.9 / 203.2
//   K = 512, H = 1024: 145 MiB 160.8 / 161.3, 157.6 / 159.0;  BF16, K = 1408: 145 MiB 556.5 / 562.5, 558.5 / 559.1
// From 136 MiB on, FP4 with K >= 1024 and H from 1024 to 4096 takes between 2.7 % less and 0.5 % more time streamed; from 64 to 133 MiB between 2 %
// less and 2.6 % more, with one set of buffers mostly more.
template <bool FP4>
__device__ __forceinline__ bool stream_output(const GemmParams& p) {
    const long long rows = __builtin_amdgcn_readfirstlane(p.offs[p.n_local]);
    const int limit_mib = FP4 && p.K >= 1024 ? 136 : 160;
    return rows * p.n_out * 2 > ((long long)limit_mib << 20);
}

// Stores a 32-row x 32-column BF16 tile held as "lane (li, half) owns 16 consecutive columns of row li"
// (c0 = its first 8 columns, c1 = the next 8).  Writing it as held would touch 32 rows with two
// separate 16-byte pieces per instruction; a CU sustains only ~16 B/clk of such stores.  Neighbouring
// lanes therefore swap halves (DPP quad permute), so that one instruction writes the even rows and the
// next the odd rows, four lanes covering 64 contiguous bytes of a row: 16 rows per instruction, ~3x the
// store rate measured.  `base` points at column 0 of tile row 0; rows >= rows_left are not written.
// NT: non-temporal stores.  They drain faster, but the output then bypasses the memory-side cache, from
// which the next kernel would otherwise read it back: worth it only for outputs too large to stay there.
// (Gate/up: a wave holds 32 columns of h, so BF16 rows above the limit leave in non-temporal half lines, 64 bytes.  Layer calls with and
// without streaming h are the same within 0.5 %: 62 000 rows of I = 1408 899 / 899 us, 250 000 of I = 768 2083 / 2078.)
// Prepares the two store registers of store_tile_rows: ra = this lane's 16-byte piece of the even row of its
// pair, rb = of the odd row.
// (D = 2: the same between lanes two apart.)
template <int D = 1>
__device__ __forceinline__ void swap_halves(int lane, const u32x4_t& c0, const u32x4_t& c1, u32x4_t& ra, u32x4_t& rb) {
    constexpr int CTRL = D == 1 ? 0xB1 : 0x4E;             // quad_perm [1,0,3,2], [2,3,0,1]
    const bool odd = lane & D;
    const uint32_t a0[4] = {c0.x, c0.y, c0.z, c0.w}, a1[4] = {c1.x, c1.y, c1.z, c1.w};
    uint32_t xa[4], xb[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t n0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)a0[d], CTRL, 0xF, 0xF, true);   // the pair neighbour's c0
        const uint32_t n1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)a1[d], CTRL, 0xF, 0xF, true);   //                      c1
        xa[d] = odd ? n1 : a0[d];          // even row of the pair: even lane gives its c0, odd lane the even lane's c1
        xb[d] = odd ? a1[d] : n0;          // odd row of the pair:  even lane gives the odd lane's c0, odd lane its c1
    }
    ra = u32x4_t{xa[0], xa[1], xa[2], xa[3]};
    rb = u32x4_t{xb[0], xb[1], xb[2], xb[3]};
}
template <bool NT>
__device__ __forceinline__ void store16(uint8_t* dst, const u32x4_t& v, bool on) {
    if constexpr (NT) {
        if (on) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(dst));
    } else {
        if (on) *reinterpret_cast<u32x4_t*>(dst) = v;
    }
}
template <bool NT>
__device__ __forceinline__ void store_tile_rows(uint8_t* base, size_t row_pitch, int lane, int rows_left,
                                                const u32x4_t& c0, const u32x4_t& c1) {
    const int li = lane & 31, half = lane >> 5;
    u32x4_t ra, rb;
    swap_halves(lane, c0, c1, ra, rb);
    const int row_a = li & ~1;
    uint8_t* dst = base + (size_t)row_a * row_pitch + (half * 2 + (lane & 1)) * 16;
    store16<NT>(dst, ra, row_a < rows_left);
    store16<NT>(dst + row_pitch, rb, row_a + 1 < rows_left);
}
// Two neighbouring 32-column tiles of the same 32 rows (128 contiguous bytes per row).  The two 64-byte halves of
// a row's line are written by consecutive instructions, so that they reach the memory side together.
// NT: non-temporal halves are not put together again on their way to memory, so a second swap, between lanes two apart, makes whole lines:
// 8 rows x 128 bytes per instruction.  1 GB of such stores alone: 3.0 TB/s in halves, 5.1 TB/s in lines; in the down GEMM of 249 000 rows
// (FP4, K = 768) 314 -> 277 us.  (Temporal stores: 6.2 TB/s in halves, 5.4 in lines, but they push the operands out of the L2: 339 us.)
template <bool NT>
__device__ __forceinline__ void store_tile_pair(uint8_t* base, size_t row_pitch, int lane, int rows_left, const u32x4_t& p0,
                                                const u32x4_t& p1, const u32x4_t& q0, const u32x4_t& q1) {
    const int li = lane & 31, half = lane >> 5;
    u32x4_t pa, pb, qa, qb;
    swap_halves(lane, p0, p1, pa, pb);
    swap_halves(lane, q0, q1, qa, qb);
    if constexpr (NT) {
        u32x4_t r0, r1, r2, r3;
        swap_halves<2>(lane, pa, qa, r0, r2);
        swap_halves<2>(lane, pb, qb, r1, r3);
        const int row = li & ~3;
        uint8_t* dst = base + (size_t)row * row_pitch + ((lane & 2) * 2 + half * 2 + (lane & 1)) * 16;
        store16<NT>(dst, r0, row < rows_left);
        store16<NT>(dst + row_pitch, r1, row + 1 < rows_left);
        store16<NT>(dst + 2 * row_pitch, r2, row + 2 < rows_left);
        store16<NT>(dst + 3 * row_pitch, r3, row + 3 < rows_left);
    } else {
        const int row_a = li & ~1;
        uint8_t* dst = base + (size_t)row_a * row_pitch + (half * 2 + (lane & 1)) * 16;
        store16<NT>(dst, pa, row_a < rows_left);
        store16<NT>(dst + 64, qa, row_a < rows_left);
        store16<NT>(dst + row_pitch, pb, row_a + 1 < rows_left);
        store16<NT>(dst + row_pitch + 64, qb, row_a + 1 < rows_left);
    }
}

// Epilogue of one 32-row tile of a wave, straight from registers.  a[t][r] belongs to activation row tile_row0 + li of the
// block tile and to column 16*half + r of the wave's t-th 32-column tile (wn = the wave's place along the columns).
// rows_valid = rows of the block tile that exist (may exceed the tile height).
template <bool FP4, bool GATEUP, int WN, bool NT>
__device__ __forceinline__ void epilogue_mt(const GemmParams& p, v16f_t (&a)[WN], int tile_row0, int row0, int rows_valid, int n0,
                                            int wn, int li, int half) {
    const int lane = half * 32 + li;
    if constexpr (GATEUP) {
        constexpr int HT = WN / 2;                     // h column tiles per wave
        const int m = tile_row0 + li;
        const bool valid = m < rows_valid;
        const size_t grow = (size_t)(row0 + m);
#pragma unroll
        for (int t = 0; t < HT; ++t) {
            const int ctile = n0 + wn * HT * 32 + t * 32;  // first h column of the 32-column tile
            uint32_t hb[8];                                // 16 BF16 values: columns ctile + 16*half + 0..15
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float g0 = a[t][2 * q], u0 = a[t + HT][2 * q];
                const float g1 = a[t][2 * q + 1], u1 = a[t + HT][2 * q + 1];
                hb[q] = pack_bf16x2(g0 * u0 * __builtin_amdgcn_rcpf(1.0f + __expf(-g0)),
                                    g1 * u1 * __builtin_amdgcn_rcpf(1.0f + __expf(-g1)));
            }
            if constexpr (FP4) {
                const u32x4_t v0 = {hb[0], hb[1], hb[2], hb[3]}, v1 = {hb[4], hb[5], hb[6], hb[7]};
                uint32_t amax = max(amax_bits8(v0), amax_bits8(v1));
                // the block's other 16 columns sit in lane^32: swapping the upper half of one copy with the lower half of
                // another leaves {lo, lo} and {hi, hi}, whose maximum is the pair's -- one VALU instruction, no LDS round trip
                const auto halves = __builtin_amdgcn_permlane32_swap(amax, amax, false, false);
                amax = max(halves[0], halves[1]);
                const uint32_t byte = e8m0_from_amax(amax);
                const float scl = scale_operand(byte);
                const u32x2_t codes = {encode8(v0, scl), encode8(v1, scl)};
                if (valid) {
                    *reinterpret_cast<u32x2_t*>(p.out + grow * (size_t)(p.n_out >> 1) + (ctile >> 1) + half * 8) = codes;
                    if (half == 0) p.outs[scale_byte_offset((long long)grow, ctile >> 5, p.n_out >> 7)] = (uint8_t)byte;
                }
            } else {
                store_tile_rows<NT>(p.out + ((size_t)(row0 + tile_row0) * p.n_out + ctile) * 2, (size_t)p.n_out * 2, lane,
                                    rows_valid - tile_row0, u32x4_t{hb[0], hb[1], hb[2], hb[3]}, u32x4_t{hb[4], hb[5], hb[6], hb[7]});
            }
        }
    } else {
        auto lo8 = [&](int t) __attribute__((always_inline)) {
            return u32x4_t{pack_bf16x2(a[t][0], a[t][1]), pack_bf16x2(a[t][2], a[t][3]),
                           pack_bf16x2(a[t][4], a[t][5]), pack_bf16x2(a[t][6], a[t][7])};
        };
        auto hi8 = [&](int t) __attribute__((always_inline)) {
            return u32x4_t{pack_bf16x2(a[t][8], a[t][9]), pack_bf16x2(a[t][10], a[t][11]),
                           pack_bf16x2(a[t][12], a[t][13]), pack_bf16x2(a[t][14], a[t][15])};
        };
        static_assert(WN % 2 == 0, "column tiles are stored in pairs");
#pragma unroll
        for (int t = 0; t < WN; t += 2) {
            const int col0 = n0 + wn * WN * 32 + t * 32;
            store_tile_pair<NT>(p.out + ((size_t)(row0 + tile_row0) * p.n_out + col0) * 2, (size_t)p.n_out * 2, lane,
                                rows_valid - tile_row0, lo8(t), hi8(t), lo8(t + 1), hi8(t + 1));
        }
    }
}

// The same for 32 rows of BF16 on 16 x 16 tiles: a[i][c][r] belongs to activation row tile_row0 + 16*i + lane%16 of the block tile
// and to weight row 8*(lane/16) + 4*(c&1) + r of the wave's group c/2 of 32 weight rows (gate/up: gate rows, up rows).
template <bool GATEUP, bool NT>
__device__ __forceinline__ void epilogue16(const GemmParams& p, const v4f_t (&a)[2][4], int tile_row0, int row0, int rows_valid, int n0, int wn, int lane) {
    // 8 columns of either tile's row per lane -> 16 columns of row lane%32 of the pair, half lane/32 (c0, c1), as the stores want
    // them: four lanes 16 apart that write one row's 64 bytes do not count as contiguous (down GEMM of 249 000 rows 740 -> 855 us)
    auto side_by_side = [&](const u32x4_t& v0, const u32x4_t& v1, u32x4_t& c0, u32x4_t& c1) __attribute__((always_inline)) {
        const uint32_t a0[4] = {v0.x, v0.y, v0.z, v0.w}, a1[4] = {v1.x, v1.y, v1.z, v1.w};
        uint32_t r0[4], r1[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const auto t = __builtin_amdgcn_permlane16_swap(a0[d], a1[d], false, false);
            r0[d] = t[0];
            r1[d] = t[1];
        }
        c0 = u32x4_t{r0[0], r0[1], r0[2], r0[3]};
        c1 = u32x4_t{r1[0], r1[1], r1[2], r1[3]};
    };
    if constexpr (GATEUP) {
        u32x4_t h[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t hb[4];                            // columns 8*(lane/16) + 2*q, 2*q + 1
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float g0 = a[i][q >> 1][(q & 1) * 2], u0 = a[i][2 + (q >> 1)][(q & 1) * 2];
                const float g1 = a[i][q >> 1][(q & 1) * 2 + 1], u1 = a[i][2 + (q >> 1)][(q & 1) * 2 + 1];
                hb[q] = pack_bf16x2(g0 * u0 * __builtin_amdgcn_rcpf(1.0f + __expf(-g0)),
                                    g1 * u1 * __builtin_amdgcn_rcpf(1.0f + __expf(-g1)));
            }
            h[i] = u32x4_t{hb[0], hb[1], hb[2], hb[3]};
        }
        u32x4_t c0, c1;
        side_by_side(h[0], h[1], c0, c1);
        store_tile_rows<NT>(p.out + ((size_t)(row0 + tile_row0) * p.n_out + n0 + wn * 32) * 2, (size_t)p.n_out * 2, lane, rows_valid - tile_row0, c0, c1);
    } else {
        u32x4_t c[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            auto packed = [&](int i) __attribute__((always_inline)) {
                const v4f_t lo = a[i][2 * t], hi = a[i][2 * t + 1];
                return u32x4_t{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
            };
            side_by_side(packed(0), packed(1), c[t][0], c[t][1]);
        }
        store_tile_pair<NT>(p.out + ((size_t)(row0 + tile_row0) * p.n_out + n0 + wn * 64) * 2, (size_t)p.n_out * 2, lane, rows_valid - tile_row0,
                            c[0][0], c[0][1], c[1][0], c[1][1]);
    }
}

__device__ __forceinline__ void lds_dma16(const uint8_t* g, uint8_t* l) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
__device__ __forceinline__ void lds_dma4(const uint32_t* g, uint8_t* l) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)l, 4, 0, 0);
}

}  // namespace realb
