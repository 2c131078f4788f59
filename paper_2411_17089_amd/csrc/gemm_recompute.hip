// Recompute GEMM for gfx950 (Eq. 7 with fused bias):
//     C[M, N] = A[M, K] . W[N, K]^T + bias[N]        float16 in / float32 accumulate / float16 out
// A = X[0:l] flattened to [l*batch, hidden], W = [Wk^T ; Wv^T] ([2h, h], K contiguous), C = rows
// [0, l) of the device KV buffer (row stride ldc = 2h), so the result needs no copy or merge pass.
//
// Design (MI355X):
//  * One workgroup of 8 waves owns a BM x BN tile of C and walks K in stages of 64: one whole 128-byte
//    line of every operand row.  The A rows and the W rows of a stage are separate blocks in LDS, each
//    operand with a ring of them, as deep as 160 KiB allow: 2 stages ahead with 256 x 256 tiles, 3 with
//    256 x 128 and 192 x 128, 4 with 128 x 128, 6 with 64 x 128.
//  * Six tile sizes (kTiles, pick_tile).  A 256 x 256 tile is the cheapest per flop (operand bytes), but
//    432 rows by 8192 columns are 64 of them and take 75 us on a chip of 256 compute units; 128 x 128
//    tiles take 36 there (hidden 4096).  With small tiles the depth of the ring counts: few operand bytes
//    are in flight per compute unit, and their latency under load is about 2 us (128 x 128, 4 waves,
//    2 stages ahead: 43 us at M = 256; 4 stages ahead: 38; 8 waves, 4 stages: 33).
//  * Waves of a 256 x 256 tile as 2 x 4 rather than 4 x 2: 1.5 - 2 % at M = 8192 .. 24576 (3755 -> 3680 us
//    at M = 24576, N = 14336, K = 7168), the LDS bytes and registers being equal.
//  * Blocks are filled by direct global->LDS DMA (global_load_lds_dwordx4): no staging registers, no
//    ds_write.  An instruction covers 8 rows x 128 B.  What limits this kernel is that path: measured
//    alone it delivers 40 B/clk/CU with 64-byte row pieces, 50 with 128-byte ones and 56 with 256-byte
//    ones, against the 32 B/clk/CU that a 256 x 256 tile consumes at the full MFMA rate; with the DMA
//    taken out of the loop the same schedule runs 25 % faster.  Whole lines per row is what moved it.
//  * The 16-byte chunks of a row are XOR-swizzled by (row/2)%8 on the global-address side so that the
//    ds_read_b128 of 16 consecutive rows touches 16 different bank groups.
//  * The loop is software-pipelined by hand: per stage four groups of MFMAs, each covering the LDS
//    latency of the next operand fragments; one workgroup barrier per stage, placed before the last
//    group; the wait in front of it is a counted vmcnt (the youngest block stays in flight).
//  * v_mfma_f32_16x16x32_f16, not 32x32x16: at the board's power limit throughput is set by energy per
//    flop, and the 16 x 16 form moves fewer accumulator bytes through the register file per flop.  A
//    register-only loop on N(0, 1) x N(0, 0.02) operands runs at 1625 TFLOP/s with the 32 x 32 form and
//    at 1835 with this one; this kernel went from 1225 to 1400 (M = 24576, N = 14336, K = 7168).
//  * The MFMA is issued "transposed" (W rows feed the instruction's row operand, X rows its column
//    operand) so a lane owns 4 consecutive output columns of one row per accumulator tile.
//  * Epilogue: bias + conversion in registers, C tile staged through LDS, global stores of whole
//    512-byte row pieces.  Stores straight from registers (8-byte pieces, or 16-byte pieces after a
//    v_permlane32_swap) cost 10-15 % of the kernel: 32 rows x 32 bytes per instruction is a poor write.
//  * Workgroup ids are remapped so that the workgroups an XCD runs concurrently (ids equal mod 8)
//    form a compact block of tiles sharing A/W panels in that XCD's L2.  Across XCDs there are two
//    mappings: each XCD takes a contiguous share of the tile rows (W is re-read by all XCDs and lives in
//    the memory-side cache; best while W is small), or each XCD takes a band of tile columns and all
//    walk the tile rows together (the A panels in flight are shared by the eight XCDs; best for large W).
//  * Tail rows in M / N are clamped on load (they re-read the last valid row) and skipped on store.
//  * Rotary models (HD = head width 64 or 128): the cache holds K after the rotary embedding, so the
//    recomputed K columns are rotated in the epilogue with the position of their row
//    (pos0 + row / batch), in float32 and in registers: the columns of a
//    wave are chosen so that a column and its partner at distance HD/2 sit in the same lane, a fixed
//    number of accumulator tiles apart.  cos/sin come from a float2 table [position][HD/2] (L1/L2 hits: a tile spans few positions).
#include "kvpr_internal.h"
#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

namespace kvpr {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gbl_ptr_t;

constexpr int BK = 64;           // halfs per stage: one 128-byte line per row
constexpr int ROW_BYTES = 128;   // one LDS row of a block

// rotary epilogue: table[pos * HD/2 + i] = (cos, sin)(pos * theta_i); columns [0, cols) of C are rotated
struct RopeArgs {
    const float2* table;
    int cols, batch, pos0;
};

template <int VM, int LGKM0>
__device__ __forceinline__ void wait_counts() {
    // vmcnt(VM) [bits 3:0 and 15:14], expcnt untouched (7), lgkmcnt(0) if LGKM0 else untouched (15)
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x0070 | (LGKM0 ? 0 : 0x0F00));
}

template <int BM, int BN, int WM, int WN, int GROUP_M, int D, int HD, bool BESIDE>
__global__ __launch_bounds__(WM * WN * 64) void gemm_bias_f16(
    const _Float16* __restrict__ A, const _Float16* __restrict__ W, const _Float16* __restrict__ bias,
    _Float16* __restrict__ C, int64_t M, int N, int K, int64_t ldc, int tiles_m, int tiles_n, int tiles_per_xcd,
    int xcd_split_n, RopeArgs rope, const CopyJob beside) {
    constexpr int NW = WM * WN;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int TM = WTM / 16, TN = WTN / 16, TMH = TM / 2, TNH = TN / 2;
    constexpr int LA = BM / 8 / NW, LW = BN / 8 / NW;     // DMA instructions per wave per block (8 rows x 128 B each)
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile/waves mismatch");
    // LDS: a ring of A blocks and a ring of W blocks, one block per stage.  The operand with the smaller block is issued
    // early in a stage and has D + 1 slots, the other one after the stage's barrier and has D (see the ring protocol)
    constexpr int A_BLK = BM * ROW_BYTES, W_BLK = BN * ROW_BYTES;
    constexpr bool A_EARLY = BM <= BN;
    constexpr int NA = A_EARLY ? D + 1 : D, NB = A_EARLY ? D : D + 1;
    constexpr int W_RING = NA * A_BLK;                    // byte offset of the W ring
    constexpr int NMFMA = TM * TNH;                       // per group: all A rows of the wave tile x half of its W rows, K = 32
    static_assert(TN % 2 == 0, "a wave's columns must split in halves");
    static_assert(D >= 2, "a stage's loads are issued D stages ahead");
    // columns of a wave: WTN consecutive ones, or (rotary heads wider than that) two runs of WTN/2 at the same place of
    // the two halves of a head, so that a column and its rotary partner stay in one lane
    constexpr bool HALVES = HD > WTN;
    constexpr int HEAD_WAVES = HALVES ? HD / WTN : 1;     // waves that share a head's columns

    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    int pid = blockIdx.x;
    // In front of the tiles: copies that go along, in a multiple of 8 workgroups, which leaves the tiles on their XCDs.  (An
    // instantiation of its own: the branch in all of them costs the large product 1.6 %, 3690 -> 3750 us at M = 24576, N = 14336,
    // K = 7168.)
    if constexpr (BESIDE) {
        const int front = (beside.blocks + 7) / 8 * 8;
        if (pid < front) {
            if (pid < beside.blocks) run_copy_job(beside, pid);
            return;
        }
        pid -= front;
    }
    int tile_m, tile_n;
    if (xcd_split_n) {
        const int xcd = pid & 7, i = pid >> 3;
        const int n_lo = xcd * tiles_n / 8, width = (xcd + 1) * tiles_n / 8 - n_lo;
        if (i >= width * tiles_m) return;
        const int group_sz = GROUP_M * width;
        const int group = i / group_sz;
        const int first_m = group * GROUP_M;
        const int gm = min(tiles_m - first_m, GROUP_M);
        const int in_group = i - group * group_sz;
        tile_m = first_m + in_group % gm;
        tile_n = n_lo + in_group / gm;
    } else {
        const int logical = (pid & 7) * tiles_per_xcd + (pid >> 3);
        if (logical >= tiles_m * tiles_n) return;
        const int group_sz = GROUP_M * tiles_n;
        const int group = logical / group_sz;
        const int first_m = group * GROUP_M;
        const int gm = min(tiles_m - first_m, GROUP_M);
        const int in_group = logical - group * group_sz;
        tile_m = first_m + in_group % gm;
        tile_n = in_group / gm;
    }
    const int64_t m0 = (int64_t)tile_m * BM;
    const int n0 = tile_n * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    // first tile column of the wave's lower / upper TNH accumulator tiles
    const int col_lo = HALVES ? wn / HEAD_WAVES * HD + wn % HEAD_WAVES * (WTN / 2) : wn * WTN;
    constexpr int UPPER = HALVES ? HD / 2 : WTN / 2;
    auto col_of = [&](int i) { return col_lo + (i >= TNH ? UPPER : 0) + (i % TNH) * 16; };

    // DMA: instruction i of this wave fills block rows [8*(wave + NW*i), +8); lane L lands at row 8*blk + L/8,
    // physical 16-byte chunk L%8, and therefore fetches logical chunk (L%8) ^ ((row/2)%8): with 128-byte rows the
    // ds_read_b128 of 16 consecutive rows then touches 16 different bank groups.
    const _Float16* srca[LA];
    const _Float16* srcw[LW];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int row = (wave + NW * i) * 8 + (lane >> 3);
        int64_t gr = m0 + row;
        if (gr > M - 1) gr = M - 1;
        srca[i] = A + gr * K + (((lane & 7) ^ ((row >> 1) & 7)) << 3);
    }
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int row = (wave + NW * i) * 8 + (lane >> 3);
        int gr = n0 + row;
        if (gr > N - 1) gr = N - 1;
        srcw[i] = W + (int64_t)gr * K + (((lane & 7) ^ ((row >> 1) & 7)) << 3);
    }
    auto issue_a = [&](int kt, int slot) {
        unsigned char* base = lds + slot * A_BLK + wave * 1024;
#pragma unroll
        for (int i = 0; i < LA; ++i)
            __builtin_amdgcn_global_load_lds((gbl_ptr_t)(srca[i] + kt * BK), (lds_ptr_t)(base + i * NW * 1024), 16, 0, 0);
    };
    auto issue_w = [&](int kt, int slot) {
        unsigned char* base = lds + W_RING + slot * W_BLK + wave * 1024;
#pragma unroll
        for (int i = 0; i < LW; ++i)
            __builtin_amdgcn_global_load_lds((gbl_ptr_t)(srcw[i] + kt * BK), (lds_ptr_t)(base + i * NW * 1024), 16, 0, 0);
    };
    auto next_a = [](int s) { return s + 1 == NA ? 0 : s + 1; };
    auto next_w = [](int s) { return s + 1 == NB ? 0 : s + 1; };

    // fragment addresses: row r = lane%16 of a 16-row tile, k-step kk (32 halfs = four 16-byte chunks, lane/16 picks one).
    // The swizzle term (r/2)%8 depends only on lane%16 because every wave / tile offset is a multiple of 16 rows.
    const int frow = lane & 15, fchunk = lane >> 4;
    int koff[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) koff[kk] = frow * ROW_BYTES + (((kk * 4 + fchunk) ^ ((frow >> 1) & 7)) << 4);

    floatx4 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // operand fragments: A of k-step 0 / 1, and the lower / upper half of the wave tile's W rows
    half8 a0[TM], a1[TM], wlo[TNH], whi[TNH];
    auto load_a = [&](int sa, int kk, half8* a, int t0, int t1) {
        const unsigned char* p = lds + sa * A_BLK + wm * WTM * ROW_BYTES + koff[kk];
#pragma unroll
        for (int t = t0; t < t1; ++t) a[t] = *reinterpret_cast<const half8*>(p + t * 16 * ROW_BYTES);
    };
    auto load_w = [&](int sw, int kk, half8* w, int upper) {
        const unsigned char* p = lds + W_RING + sw * W_BLK + (col_lo + upper * UPPER) * ROW_BYTES + koff[kk];
#pragma unroll
        for (int t = 0; t < TNH; ++t) w[t] = *reinterpret_cast<const half8*>(p + t * 16 * ROW_BYTES);
    };
    auto mfma_group = [&](const half8* a, const half8* w, int upper) {
#pragma unroll
        for (int i = 0; i < TNH; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
                acc[upper * TNH + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[i], a[j], acc[upper * TNH + i][j], 0, 0, 0);
    };
    // one LDS read behind each of the group's first MFMAs
    auto interleave = [&](auto id, auto reads) {
        constexpr int ID = decltype(id)::value, READS = decltype(reads)::value, PAIRS = READS < NMFMA ? READS : NMFMA;
#pragma unroll
        for (int x = 0; x < PAIRS; ++x) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, ID);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, ID);
        }
        if constexpr (NMFMA > PAIRS) __builtin_amdgcn_sched_group_barrier(0x008, NMFMA - PAIRS, ID);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Ring protocol.  The early operand's block of stage kt lives in slot kt % (D + 1), the late one's in slot kt % D.
    // Stage kt issues the early block of stage kt + D in its first k-step, into the slot that stage kt - 1 has left, and
    // the late block of stage kt + D after its barrier, into its own slot: by then every wave has read all of stage kt.
    const int KT = K / BK;
#pragma unroll
    for (int t = 0; t < D; ++t)
        if (t < KT) {
            issue_a(t, t);
            issue_w(t, t);
        }
    if (KT >= D) wait_counts<(D - 1) * (LA + LW), 0>();
    else wait_counts<0, 0>();
    __builtin_amdgcn_s_barrier();
    load_a(0, 0, a0, 0, TM);
    load_w(0, 0, wlo, 0);

    // consumes the stage whose rows sit in slots sa and sw; on return a0 and wlo hold k-step 0 of the next.
    // Four groups of MFMAs; each covers the LDS latency of what the next ones need.
    int sa = 0, sw = 0;
    auto stage = [&](int kt, auto more) {
        constexpr bool MORE = decltype(more)::value;   // stage kt + D exists
        const int sa2 = next_a(sa), sw2 = next_w(sw);
        // the early ring's slot before this one, i.e. the one after the D that are in use
        if (MORE) {
            if constexpr (A_EARLY) issue_a(kt + D, sa == 0 ? D : sa - 1);
            else issue_w(kt + D, sw == 0 ? D : sw - 1);
        }
        load_w(sw, 0, whi, 1);
        load_a(sa, 1, a1, 0, TMH);
        mfma_group(a0, wlo, 0);
        interleave(std::integral_constant<int, 0>{}, std::integral_constant<int, TNH + TMH>{});
        load_a(sa, 1, a1, TMH, TM);
        load_w(sw, 1, wlo, 0);
        mfma_group(a0, whi, 1);
        interleave(std::integral_constant<int, 1>{}, std::integral_constant<int, TM - TMH + TNH>{});
        load_w(sw, 1, whi, 1);
        mfma_group(a1, wlo, 0);
        interleave(std::integral_constant<int, 2>{}, std::integral_constant<int, TNH>{});
        // this wave's reads of the stage are complete and its share of the next stage has landed
        // (the last stages issue nothing: they wait for all that is left)
        if (MORE) wait_counts<(D - 2) * (LA + LW) + (A_EARLY ? LA : LW), 1>();
        else wait_counts<0, 1>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (MORE) {
            if constexpr (A_EARLY) issue_w(kt + D, sw);
            else issue_a(kt + D, sa);
        }
        load_a(sa2, 0, a0, 0, TM);
        load_w(sw2, 0, wlo, 0);
        mfma_group(a1, whi, 1);
        interleave(std::integral_constant<int, 3>{}, std::integral_constant<int, TM + TNH>{});
        sa = sa2;
        sw = sw2;
    };
    int kt = 0;
    for (; kt + D < KT; ++kt) stage(kt, std::true_type{});
    for (; kt + 1 < KT; ++kt) stage(kt, std::false_type{});
    {   // last stage: nothing follows
        load_w(sw, 0, whi, 1);
        load_a(sa, 1, a1, 0, TM);
        mfma_group(a0, wlo, 0);
        mfma_group(a0, whi, 1);
        load_w(sw, 1, wlo, 0);
        load_w(sw, 1, whi, 1);
        mfma_group(a1, wlo, 0);
        mfma_group(a1, whi, 1);
    }

    // ---- epilogue: bias + float16 conversion in registers, then through LDS so that every global
    //      store instruction writes whole 512-byte pieces of C rows (accumulator register e of tile
    //      (i, j) holds n = 16*i + 4*(lane/16) + e, m = 16*j + lane%16 of the wave tile).
    //      Rows are padded by 16 bytes: the 8-byte writes of 16 consecutive rows then spread over all banks.
    constexpr int CROW = BN * 2 + 16;
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): this wave's operand reads are done
    __builtin_amdgcn_s_barrier();                  // ... and everybody else's: the stages can be overwritten
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        const int nl = col_of(i) + 4 * fchunk;
        if (bias && n0 + nl < N) {
            const half4 b4 = *reinterpret_cast<const half4*>(bias + n0 + nl);
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] += (float)b4[e];
        }
    }
    if constexpr (HD > 0) {
        constexpr int IH = HALVES ? TNH : HD / 32; // accumulator tiles between a column and its partner HD/2 columns on
        static_assert(HALVES || (WTN % HD == 0 && TN % (2 * IH) == 0), "a wave tile must hold whole heads");
        if (n0 + col_lo < rope.cols) {             // wave-uniform: this wave's columns are K columns
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                int64_t m = m0 + wm * WTM + j * 16 + frow;
                if (m > M - 1) m = M - 1;
                const float2* trow = rope.table + (int64_t)(rope.pos0 + (int)(m / rope.batch)) * (HD / 2);
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    if ((i / IH) % 2 != 0) continue;   // second half of a head: handled with its partner
                    const int f = (HALVES ? wn % HEAD_WAVES * (WTN / 2) : 0) + (i % IH) * 16 + 4 * fchunk;
                    const float4 cs0 = *reinterpret_cast<const float4*>(trow + f);
                    const float4 cs1 = *reinterpret_cast<const float4*>(trow + f + 2);
                    const float cv[4] = {cs0.x, cs0.z, cs1.x, cs1.z}, sv[4] = {cs0.y, cs0.w, cs1.y, cs1.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x1 = acc[i][j][e], x2 = acc[i + IH][j][e];
                        // which product is rounded first is spelled out: left to contraction it differs between tiles
                        acc[i][j][e] = fmaf(x1, cv[e], -(x2 * sv[e]));
                        acc[i + IH][j][e] = fmaf(x2, cv[e], x1 * sv[e]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        const int nl = col_of(i) + 4 * fchunk;
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            const int ml = wm * WTM + j * 16 + frow;
            half4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (_Float16)acc[i][j][e];
            *reinterpret_cast<half4*>(lds + ml * CROW + nl * 2) = o;
        }
    }
    __syncthreads();
    constexpr int CHUNKS_PER_ROW = BN / 8;         // 16-byte pieces
    constexpr int NT = NW * 64;
#pragma unroll 4
    for (int q = tid; q < BM * CHUNKS_PER_ROW; q += NT) {
        const int ml = q / CHUNKS_PER_ROW, cc = q % CHUNKS_PER_ROW;
        const int64_t m = m0 + ml;
        const int n = n0 + cc * 8;
        if (m < M && n < N)
            __builtin_nontemporal_store(*reinterpret_cast<const half8*>(lds + ml * CROW + cc * 16),
                                        reinterpret_cast<half8*>(C + m * ldc + n));   // C is not re-read here: keep it out of L2
    }
}

int g_gemm_xcd_split_n = -1;   // -1 = default choice (debug hook; process-wide, set it only while no launch is in progress)

// Which mapping of workgroups to tiles: giving every XCD a band of W wins once W no longer sits comfortably in the
// memory-side cache next to the A panels in flight (1410 against 1396 TFLOP/s at M = 24576, N = 14336, K = 7168, 196 MiB)
// and is even with the row mapping or 0.5 % behind it at 100 and 64 MiB (hidden 5120 and 4096).
bool band_mapping(int N, int K) {
    if ((N + 255) / 256 < 8) return false;
    if (g_gemm_xcd_split_n >= 0) return g_gemm_xcd_split_n != 0;
    return (int64_t)N * K * 2 > ((int64_t)128 << 20);
}

template <int BM, int BN, int WM, int WN, int D, int HD, bool BESIDE = false>
int launch_tile(const void* a, const void* w, const void* bias, void* c, int64_t M, int N, int K, int64_t ldc,
                hipStream_t st, RopeArgs rope, const CopyJob& beside) {
    // raster groups of 4 tile rows: 32 compute units of an XCD cover a 4 x 8 block.  8 rows per group: 1337 instead of
    // 1410 TFLOP/s at M = 24576, N = 14336, K = 7168 (band mapping), 1330 instead of 1386 at M = 26624, N = 8192,
    // K = 4096 (row mapping); 2 rows within 1 % of 4, 5 and 6 as 8.
    if constexpr (!BESIDE)
        if (beside.blocks > 0) return launch_tile<BM, BN, WM, WN, D, HD, true>(a, w, bias, c, M, N, K, ldc, st, rope, beside);
    auto kern = gemm_bias_f16<BM, BN, WM, WN, 4, D, HD, BESIDE>;
    constexpr int ring_bytes = (D * (BM + BN) + (BM < BN ? BM : BN)) * ROW_BYTES, c_bytes = BM * (BN * 2 + 16);
    constexpr int lds_bytes = ring_bytes > c_bytes ? ring_bytes : c_bytes;
    static_assert(lds_bytes <= 160 * 1024, "LDS of a compute unit");
    // once per process and instantiation; call_once makes concurrent first launches from several threads safe
    static std::once_flag configured;
    static hipError_t configure_status = hipSuccess;
    std::call_once(configured, [&] {
        configure_status = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    KVPR_HIP(configure_status);
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN;
    const int64_t total = (int64_t)tiles_m * tiles_n;
    const int xcd_split_n = band_mapping(N, K) ? 1 : 0;
    const int max_width = (tiles_n + 7) / 8;
    const int tiles_per_xcd = xcd_split_n ? max_width * tiles_m : (int)((total + 7) / 8);
    const unsigned grid = (unsigned)(tiles_per_xcd * 8 + (beside.blocks + 7) / 8 * 8);
    static_assert(WM * WN * 64 == kCopyThreads, "copies are cut for workgroups of this size");
    hipLaunchKernelGGL(kern, dim3(grid), dim3(WM * WN * 64), lds_bytes, st, (const _Float16*)a, (const _Float16*)w,
                       (const _Float16*)bias, (_Float16*)c, M, N, K, ldc, tiles_m, tiles_n, tiles_per_xcd, xcd_split_n, rope, beside);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

int g_gemm_variant = 0;   // 0 = choose from the shape, 1.. = force that entry of kTiles (tests and tuning sweeps)

// The tiles, and what a stage (64 of K) of one costs in ns: `full` when all compute units work on one, `least` when few do
// and the latency of the global -> LDS path sets it.  Smaller tiles cost more per output (operand bytes per flop) but leave
// fewer compute units idle when M is small or ragged.
struct TileCost { int bm, bn, full, least; };
constexpr TileCost kTiles[] = {{256, 256, 1537, 1114}, {192, 256, 1199, 926}, {256, 128, 873, 662},
                               {192, 128, 661, 530},   {128, 128, 529, 444},  {64, 128, 358, 383}};

// One workgroup per compute unit at a time: whole rounds cost `full`, the last one in proportion to what it fills but not
// less than `least`.  (K is a common factor: all tiles take the same number of stages.)  The costs are a fit to 378 timings
// (hidden 4096 / 5120 / 7168, N = 2 hidden, M = 1 .. 4096, all six tiles): they predict them to 9 % (rms), and the tile they
// pick is within 0.2 % of the fastest on average and 8 % at worst.
int pick_tile(int64_t M, int N, int64_t* stage_ns = nullptr) {
    const int64_t cus = compute_units();
    int best = 0;
    int64_t best_cost = INT64_MAX;
    for (int i = 0; i < (int)(sizeof kTiles / sizeof kTiles[0]); ++i) {
        const TileCost& t = kTiles[i];
        const int64_t tiles = (M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn), rem = tiles % cus;
        const int64_t cost = tiles / cus * t.full + (rem ? std::max<int64_t>(t.least, t.full * rem / cus) : 0);
        if (cost < best_cost) { best_cost = cost; best = i; }
    }
    if (stage_ns) *stage_ns = best_cost;
    return best;
}

template <int HD>
int launch_any(const void* a, const void* w, const void* bias, void* c, int64_t M, int N, int K, int64_t ldc, hipStream_t st,
               RopeArgs rope, const CopyJob& beside) {
    switch (g_gemm_variant > 0 ? g_gemm_variant - 1 : pick_tile(M, N)) {
        case 1: return launch_tile<192, 256, 4, 2, 2, HD>(a, w, bias, c, M, N, K, ldc, st, rope, beside);
        case 2: return launch_tile<256, 128, 4, 2, 3, HD>(a, w, bias, c, M, N, K, ldc, st, rope, beside);
        case 3: return launch_tile<192, 128, 4, 2, 3, HD>(a, w, bias, c, M, N, K, ldc, st, rope, beside);
        case 4: return launch_tile<128, 128, 4, 2, 4, HD>(a, w, bias, c, M, N, K, ldc, st, rope, beside);
        case 5: return launch_tile<64, 128, 2, 4, 6, HD>(a, w, bias, c, M, N, K, ldc, st, rope, beside);
        default: return launch_tile<256, 256, 2, 4, 2, HD>(a, w, bias, c, M, N, K, ldc, st, rope, beside);
    }
}

}  // namespace

int64_t gemm_workgroups(int64_t M, int N) {
    const TileCost& t = kTiles[g_gemm_variant > 0 ? (g_gemm_variant <= 6 ? g_gemm_variant - 1 : 0) : pick_tile(M, N)];
    return (M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn);
}

double gemm_estimate_s(int64_t M, int N, int K) {
    int64_t stage_ns = 0;
    if (M > 0) pick_tile(M, N, &stage_ns);
    return 1e-9 * (double)stage_ns * (K / BK);
}

int launch_gemm(const void* a, const void* w, const void* bias, void* c, int64_t M, int N, int K, int64_t ldc,
                hipStream_t st, const CopyJob& beside) {
    if (M == 0) return launch_copy(beside, kCopyThreads, st);
    return launch_any<0>(a, w, bias, c, M, N, K, ldc, st, RopeArgs{nullptr, 0, 1, 0}, beside);
}

// Eq. 7 for a rotary model: as launch_gemm, with columns [0, rope_cols) (the K half) rotated by the position
// pos0 + row / batch of their row.  table: float2 [positions][head_dim/2] on the device.
int launch_gemm_rope(const void* a, const void* w, const void* bias, void* c, int64_t M, int N, int K, int64_t ldc,
                     const void* table, int rope_cols, int head_dim, int batch, int pos0, hipStream_t st, const CopyJob& beside) {
    if (M == 0) return launch_copy(beside, kCopyThreads, st);
    const RopeArgs r{(const float2*)table, rope_cols, batch, pos0};
    return head_dim == 64 ? launch_any<64>(a, w, bias, c, M, N, K, ldc, st, r, beside)
                          : launch_any<128>(a, w, bias, c, M, N, K, ldc, st, r, beside);
}

}  // namespace kvpr

extern "C" int kvpr_debug_set_gemm_variant(int v) {
    kvpr::g_gemm_variant = v;
    return KVPR_OK;
}

extern "C" int kvpr_debug_set_gemm_mapping(int xcd_split_n) {
    kvpr::g_gemm_xcd_split_n = xcd_split_n;
    return KVPR_OK;
}
