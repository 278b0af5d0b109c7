// gdn_linear: the layers' projections y = x w^T + bias on the bf16 matrix cores (see include/gdn_linear.h).
//
// One workgroup of four or eight waves makes a BM (tokens) x BN (outputs) tile, a wave its part of it as tiles of
// v_mfma_f32_16x16x32_bf16.  Both operands are read along k, so a k step of BK needs a BM x BK tile of x and a
// BN x BK tile of w; they come from memory with 16-byte buffer loads straight to LDS (no registers) into a ring of
// STAGES stages, STAGES - 1 k steps ahead of the matrix cores: one barrier per k step.  The shapes that are built:
//   0: 128 x 128 x 64, 2 stages, four waves, two workgroups per compute unit   many small tiles: one workgroup's waits under the other's products
//   1: 256 x 256 x 64, 2 stages, four waves, one workgroup per compute unit: a wave holds 128 x 128 outputs in 256
//      accumulator registers: fewer operand bytes from LDS per flop, one wave per SIMD (kept for comparison: within 3 % of 2 either way)
//   2: 256 x 256 x 64, 2 stages, eight waves of 128 tokens x 64 outputs, two per SIMD: while one wave of a SIMD is held up
//      issuing its loads to LDS the other feeds the matrix pipe, and a barrier covers 64 of k (the default for large problems)
//   3: 64 x 64 x 64, 5 stages, four waves of 32 x 32 outputs, two workgroups per compute unit: problems whose 64 x 64 tiles fit
//      the chip in one round, where a larger tile would walk k on too few compute units (512 x 2048 x 2048 9.9 us against 16 of
//      shape 4 and 21 of shape 0)
//   4: 128 x 128 x 64, 4 stages, eight waves, one workgroup per compute unit: problems of at most one round of such tiles are bound by
//      the latency of a k step's loads (0.9 us where the weights come from memory), of which this shape has three in flight
//      (384 x 8224 x 2048 23 us against 31 of shape 0)
//   5: 128 x 160 x 64, 4 stages, four waves, one workgroup per compute unit: the same for problems that shape 4 just does not
//      fit in one round (512 x 8224: 260 tiles of 128 outputs for 256 compute units, 208 of 160; 27 us against 36 of shape 4, 32 of shape 0)
// The products are v_mfma_f32_16x16x32_bf16: half the accumulator traffic per flop of the 32 x 32 x 16 instruction, at the same rate on
// paper; on a chip held by its power limit 8192 x 2048 x 2048 takes 51 us with it and 56 with the other, 512 x 2048 10.4 and 12.3.
// A load to LDS writes a wave's 1 KiB contiguously (lane i at 16 i), so rows are unpadded (2 BK bytes) and bank
// conflicts are avoided by choosing WHICH 16-byte piece of its row a lane fetches: piece p of row r is stored at
// position p ^ swz(r), swz(r) = (r / rows per 256 bytes) % pieces per row, which makes the 16 lanes that read the
// same piece of 16 consecutive rows hit 16 different 16-byte bank groups.  Rows past the end of x or w read as
// zeros (the buffer descriptor ends with the matrix); they only feed outputs that are never stored.  The products
// are taken transposed (w rows as the left operand), so that a lane holds four consecutive outputs of ONE token
// and writes them to LDS, for the turn to whole rows, with one 8- or 16-byte store.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>

#include "gdn_linear.h"

namespace gdn {
namespace linear {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));


constexpr int LIN_MAX_SEG = 8;

struct LinearArgs {
    const void* x;
    const void* w;
    const float* bias;
    void* y;
    int64_t ldx, ldw, ldy;
    int64_t T;
    int32_t N, K;
    int32_t tiles_m, tiles_n;
    int32_t per_xcd;                    // tiles per XCD
    // gdn_linear_split: the outputs go to n_seg destinations by column range; n_seg = 0: everything to y
    int32_t n_seg;
    int32_t seg_col[LIN_MAX_SEG + 1];   // segment s holds outputs seg_col[s] .. seg_col[s + 1] - 1
    void* seg_y[LIN_MAX_SEG];
    int64_t seg_ld[LIN_MAX_SEG];
};

inline int32_t hip_err(hipError_t e) { return e == hipSuccess ? GDN_OK : GDN_ERR_HIP - (int32_t)e; }

// s_waitcnt vmcnt(N) (gfx9 encoding: vmcnt in bits 3:0 and 15:14; other counters left alone)
template <int N>
__device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt(((N & 0x30) << 10) | (N & 0xF) | 0x0F70);
}

template <int BM_, int BN_, int BK_, int STAGES_, int WGS_PER_CU_, int WAVES_M_, int WAVES_N_>
struct LinCfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, STAGES = STAGES_, WGS_PER_CU = WGS_PER_CU_;
    static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, NW = WAVES_M * WAVES_N, THREADS = 64 * NW;   // the wave grid over the tile
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;   // a wave's tokens and outputs
    static constexpr int RB = BK * 2;                  // bytes of a tile row
    static constexpr int PP = RB / 16;                 // 16-byte pieces per row
    static constexpr int RL = 256 / RB;                // rows per 256 bytes (the span of the 64 banks)
    static constexpr int ROWS_PER_LOAD = 1024 / RB;    // rows a wave-wide load covers
    static constexpr int X_BYTES = BM * RB, W_BYTES = BN * RB, STAGE_BYTES = X_BYTES + W_BYTES;
    static constexpr int SMEM = STAGES * STAGE_BYTES;
    static constexpr int TI = WM / 16, TJ = WN / 16;   // 16 x 16 tiles of a wave along tokens / outputs
    static constexpr int XL = BM / ROWS_PER_LOAD / NW, WL = BN / ROWS_PER_LOAD / NW;   // loads per wave and stage
    static constexpr int LPS = XL + WL;
    static constexpr int AHEAD = (STAGES - 2) * LPS;   // loads that may still be in flight when a stage is handed over
    static_assert(PP * RL == 16 && (STAGES - 1) * LPS < 64 && SMEM * WGS_PER_CU <= 160 * 1024 && (BK / 32) % 2 == 0 &&
                  XL * ROWS_PER_LOAD * NW == BM && WL * ROWS_PER_LOAD * NW == BN && TI * 16 == WM && TJ * 16 == WN, "tile shape");
};
typedef LinCfg<128, 128, 64, 2, 2, 2, 2> LinSmall;
typedef LinCfg<256, 256, 64, 2, 1, 2, 2> LinBig;      // four waves, 128 x 128 outputs each
typedef LinCfg<256, 256, 64, 2, 1, 2, 4> LinBig8;     // eight waves, 128 tokens x 64 outputs each: two waves per SIMD
typedef LinCfg<64, 64, 64, 5, 2, 2, 2> LinTiny;       // four waves of 32 x 32 outputs each, four k steps of 64 in flight
typedef LinCfg<128, 128, 64, 4, 1, 2, 4> LinDeep;     // eight waves, 64 x 32 outputs each, three k steps of 64 in flight
typedef LinCfg<128, 160, 64, 4, 1, 2, 2> LinWide;     // four waves, 64 x 80 outputs each, three k steps of 64 in flight

// The loads of one wave for one stage: 1 KiB each, XL of its quarter of the x tile, then WL of the w tile.
template <typename CFG>
struct LinLoad {
    static __device__ __forceinline__ void one(int j, char* smem, int stage, int k0, int wave, const char* xb, int x_bytes, const char* wb,
                                               int w_bytes, const int* xoff, const int* woff) {
        // buffer descriptors that end with the matrices: rows past T or N arrive as zeros
        char* xs = smem + stage * CFG::STAGE_BYTES;
        char* ws = xs + CFG::X_BYTES;
        if (j < CFG::XL) {
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(xb), 0, x_bytes, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(xs + ((CFG::BM / CFG::NW) * wave + CFG::ROWS_PER_LOAD * j) * CFG::RB), 16, xoff[j], k0 * 2, 0, 0);
        } else {
            const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(wb), 0, w_bytes, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (__attribute__((address_space(3))) void*)(ws + ((CFG::BN / CFG::NW) * wave + CFG::ROWS_PER_LOAD * (j - CFG::XL)) * CFG::RB), 16, woff[j - CFG::XL], k0 * 2, 0, 0);
        }
    }
    static __device__ __forceinline__ void all(char* smem, int stage, int k0, int wave, const char* xb, int x_bytes, const char* wb, int w_bytes,
                                               const int* xoff, const int* woff) {
#pragma unroll
        for (int j = 0; j < CFG::LPS; ++j) one(j, smem, stage, k0, wave, xb, x_bytes, wb, w_bytes, xoff, woff);
    }
};

template <typename CFG, bool OUT_BF16>
__global__ void __launch_bounds__(CFG::THREADS) __attribute__((amdgpu_waves_per_eu(CFG::WGS_PER_CU * CFG::NW / 4, CFG::WGS_PER_CU * CFG::NW / 4)))
gdn_linear_kernel(LinearArgs a) {
    constexpr int BM = CFG::BM, BN = CFG::BN, BK = CFG::BK, STAGES = CFG::STAGES, RB = CFG::RB, PP = CFG::PP, RL = CFG::RL;
    constexpr int RPL = CFG::ROWS_PER_LOAD, TI = CFG::TI, TJ = CFG::TJ, XL = CFG::XL, WL = CFG::WL;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / CFG::WAVES_N, wn = wave % CFG::WAVES_N;   // the wave's part: tokens WM wm .., outputs WN wn ..
    const int lr = lane & 15, g = lane >> 4;
    // ---- which tile.  Workgroups are dealt to the 8 XCDs (each with an L2 of its own) in turn: XCD x takes a consecutive run of the
    // tiles, which are numbered GROUP_M tile rows at a time, down the rows first, so that the tiles an XCD works on together
    // share their rows of x and of w in its L2.  (Row by row over the whole output, an XCD's 32 tiles touched nearly every row of w.)
    constexpr int GROUP_M = CFG::BM == 256 ? 4 : 8;
    // Each XCD enters its run an eighth further on than the one before: XCDs that walk the same columns in step would all wait for the
    // same cold rows of w on every k step; so a row comes from memory for one or two of them and from the memory-side cache for
    // the others (8192 x 8192 x 2048 with cold weights 226 -> 209 us; 197 with warm ones either way).
    const int xcd = (int)blockIdx.x & 7;
    int in_run = ((int)blockIdx.x >> 3) + xcd * a.per_xcd / 8;
    if (in_run >= a.per_xcd) in_run -= a.per_xcd;
    const int seq = xcd * a.per_xcd + in_run;
    if (seq >= a.tiles_m * a.tiles_n) return;      // (the grid is 8 per_xcd)
    const int grp = seq / (GROUP_M * a.tiles_n), in_grp = seq % (GROUP_M * a.tiles_n);
    const int grp_rows = min(a.tiles_m - grp * GROUP_M, GROUP_M);
    const int tile_m = grp * GROUP_M + in_grp % grp_rows, tile_n = in_grp / grp_rows;
    const int64_t m0 = (int64_t)tile_m * BM;
    const int n0 = tile_n * BN;

    const int64_t rows_x = a.T - m0 < BM ? a.T - m0 : BM;
    const int rows_w = a.N - n0 < BN ? a.N - n0 : BN;
    const char* xb = reinterpret_cast<const char*>(a.x) + m0 * a.ldx * 2;
    const char* wb = reinterpret_cast<const char*>(a.w) + (int64_t)n0 * a.ldw * 2;
    const int x_bytes = (int)((rows_x - 1) * a.ldx * 2 + (int64_t)a.K * 2), w_bytes = (int)((int64_t)(rows_w - 1) * a.ldw * 2 + (int64_t)a.K * 2);

    // a wave-wide load writes RPL rows of RB bytes: lane i lands at row i / PP, position i % PP, and fetches the piece that belongs there
    const int ld_row = lane / PP, ld_pos = lane % PP;
    int xoff[XL], woff[WL];      // byte offsets (k = 0) of the loads this wave issues per stage
#pragma unroll
    for (int j = 0; j < XL; ++j) {
        const int row = (BM / CFG::NW) * wave + RPL * j + ld_row;
        xoff[j] = (int)(row * a.ldx * 2) + ((ld_pos ^ ((row / RL) % PP)) << 4);
    }
#pragma unroll
    for (int j = 0; j < WL; ++j) {
        const int row = (BN / CFG::NW) * wave + RPL * j + ld_row;
        woff[j] = (int)(row * a.ldw * 2) + ((ld_pos ^ ((row / RL) % PP)) << 4);
    }
    f32x4 acc[TJ][TI];           // [output tile][token tile]: lane lr = token, register e = output 4 g + e
#pragma unroll
    for (int i = 0; i < TJ; ++i)
#pragma unroll
        for (int j = 0; j < TI; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

    // fragment reads: row r of a tile, piece 4 kk + g, stored at (4 kk + g) ^ swz(r); tile origins are multiples of 16 rows
    const int sw = lr / RL;
    const int xrow = (CFG::WM * wm + lr) * RB, wrow = (CFG::WN * wn + lr) * RB;
    const int n_steps = a.K / BK;
    constexpr int KK = BK / 32;              // matrix-instruction steps per stage (even)
    // The stages are consumed through two fragment sets: while the matrix cores work on one k step of 32, the fragments of
    // the next are read from LDS, also across the stage boundary.  The hand-over of a stage therefore sits before the LAST
    // k step of the stage in front of it: wait for this wave's loads of the next stage, for its own fragment reads, then the
    // barrier; after it the next stage is readable by every wave and the current one (whose last fragments are in
    // registers) is free and is refilled with the stage STAGES ahead.
    bf16x8 xf[2][TI], wf[2][TJ];
    auto read_frags = [&](int stage, int kk, int set) {
        const char* xs = smem + stage * CFG::STAGE_BYTES;
        const char* ws = xs + CFG::X_BYTES;
        const int pos = ((4 * kk + g) ^ sw) * 16;
#pragma unroll
        for (int t = 0; t < TI; ++t) xf[set][t] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(xs + xrow + 16 * t * RB + pos));
#pragma unroll
        for (int t = 0; t < TJ; ++t) wf[set][t] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ws + wrow + 16 * t * RB + pos));
    };
    // Loads are issued for every stage slot, also past the last k step: there the descriptor is empty and the scalar offset
    // zero (no lane is in range by definition, nothing is fetched), so that the number of loads in flight, and with it every
    // wait below, is the same in every round and the loop body has no branch for the scheduler to stop at.
    auto mma_all = [&](int set) {
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
            for (int ti = 0; ti < TI; ++ti)
                acc[tj][ti] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[set][tj], xf[set][ti], acc[tj][ti], 0, 0, 0);
    };
#pragma unroll
    for (int p = 0; p < STAGES; ++p) {
        const bool live = p < n_steps;
        LinLoad<CFG>::all(smem, p, live ? p * BK : 0, wave, xb, live ? x_bytes : 0, wb, live ? w_bytes : 0, xoff, woff);
    }
    wait_vm<(STAGES - 1) * CFG::LPS>();
    __syncthreads();
    read_frags(0, 0, 0);
    int stage = 0;                           // step % STAGES
    for (int step = 0; step + 1 < n_steps; ++step) {
        const int next_stage = stage + 1 == STAGES ? 0 : stage + 1;
#pragma unroll
        for (int kk = 0; kk + 1 < KK; ++kk) {
            // The fragments of k step kk + 1 go into the other register set while the matrix instructions of k step kk are
            // issued, one read behind every matrix instruction or two, pinned in that order: left to itself the scheduler
            // reads them into the registers the matrix instructions have just used, behind them, and waits out the LDS
            // latency with the matrix pipe idle; and a burst of reads in front keeps the issue port from the matrix pipe.
            const int rs = (kk & 1) ^ 1, ms = kk & 1;
            const char* xs = smem + stage * CFG::STAGE_BYTES;
            const char* ws = xs + CFG::X_BYTES;
            const int pos = ((4 * (kk + 1) + g) ^ sw) * 16;
            constexpr int NM = TI * TJ, NR = TI + TJ;
            constexpr int SLOTS = NM < NR ? NM : NR;
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
#pragma unroll
                for (int q = i * NM / SLOTS; q < (i + 1) * NM / SLOTS; ++q)
                    acc[q / TI][q % TI] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ms][q / TI], xf[ms][q % TI], acc[q / TI][q % TI], 0, 0, 0);
#pragma unroll
                for (int r = i * NR / SLOTS; r < (i + 1) * NR / SLOTS; ++r) {
                    if (r < TI) xf[rs][r] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(xs + xrow + 16 * r * RB + pos));
                    else wf[rs][r - TI] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ws + wrow + 16 * (r - TI) * RB + pos));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // (the matrix instructions above stay above: left to itself the scheduler sinks them below the barrier, and the
        // fragment reads and the barrier are then waited for with the matrix pipe idle)
        __builtin_amdgcn_sched_barrier(0);
        // the next stage has landed for this wave (the STAGES - 2 stages behind it may still be in flight) ...
        wait_vm<CFG::AHEAD>();
        __builtin_amdgcn_s_waitcnt(0xC07F);          // ... and this wave's last fragment reads of the current stage are done (lgkmcnt(0))
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        {
            // The last k step of the stage (fragment set 1; KK is even), written out in issue order and pinned there: a load
            // to LDS takes tens of cycles to issue, so one goes out in each slot of a few matrix instructions, which cover it, from
            // the first slot on: a load has from here to the hand-over STAGES - 1 stages on to arrive, and with two stages one that goes out in
            // the last slot has half a stage.  (Spread over all slots, cold weights, shape 2: 4096 x 2560 x 2048 49.9 us
            // against 47.3, 3000 x 4096 x 4096 90.4 / 85.9, 1000 x 8224 x 2048 50.4 / 48.7; warm 8192 x 8192 x 2048 189 / 191; two loads a slot: 48.0, 87.1, 49.1, 192.)
            // The fragments of the next stage's first k step are read in between as well.
            const bool live = step + STAGES < n_steps;
            const int xbytes = live ? x_bytes : 0, wbytes = live ? w_bytes : 0, k_ahead = live ? (step + STAGES) * BK : 0;
            const char* xs = smem + next_stage * CFG::STAGE_BYTES;
            const char* ws = xs + CFG::X_BYTES;
            const int pos = (g ^ sw) * 16;
            constexpr int NM = TI * TJ, NL = CFG::LPS, NR = TI + TJ;
            constexpr int SLOTS = NM < (NL > NR ? NL : NR) ? NM : (NL > NR ? NL : NR);   // interleave slots
            static_assert(NL <= SLOTS, "every load has a slot");
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
#pragma unroll
                for (int q = i * NM / SLOTS; q < (i + 1) * NM / SLOTS; ++q)
                    acc[q / TI][q % TI] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[1][q / TI], xf[1][q % TI], acc[q / TI][q % TI], 0, 0, 0);
#pragma unroll
                for (int r = i * NR / SLOTS; r < (i + 1) * NR / SLOTS; ++r) {
                    if (r < TI) xf[0][r] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(xs + xrow + 16 * r * RB + pos));
                    else wf[0][r - TI] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ws + wrow + 16 * (r - TI) * RB + pos));
                }
                if (i < NL) LinLoad<CFG>::one(i, smem, stage, k_ahead, wave, xb, xbytes, wb, wbytes, xoff, woff);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        stage = next_stage;
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {        // the last stage: nothing behind it
        if (kk + 1 < KK) read_frags(stage, kk + 1, (kk & 1) ^ 1);
        mma_all(kk & 1);
    }

    // ---- epilogue: bias, one rounding, and out through LDS.  A lane holds runs of four outputs of ONE token, 16 tokens per product:
    //      stored from there, every instruction would touch 16 rows of the output with 32 or 64 bytes each.  Each wave turns its
    //      outputs around in its own share (REGION) of the now idle stage ring instead: rows of 64, 128 or 256 bytes, one for a token,
    //      with as many of the wave's outputs as 256 bytes hold (of shape 5's 80 all in bf16, in a pitch of 256 bytes, and 16 in
    //      fp32), the 16-byte pieces of a row XOR-swizzled with the token so that both the writes (lane = token) and the reads (lane =
    //      piece) spread over the banks; then 4, 8 or 16 lanes store one row's contiguous bytes.  A wave's LDS operations execute in
    //      order, so no barrier stands between its writes and reads; the one barrier before keeps the other waves' last
    //      fragment reads out of the way.
    constexpr int ES = OUT_BF16 ? 2 : 4;
    constexpr int WN = CFG::WN, WM = CFG::WM;                      // the wave's outputs and tokens
    constexpr int REGION = CFG::SMEM / CFG::NW;                    // the wave's part of the ring
    constexpr int PW = WN * ES <= 256 ? WN : WN % (256 / ES) == 0 ? 256 / ES : 16;   // outputs per pass: a row of at most 256 bytes
    constexpr int RBY = PW * ES <= 64 ? 64 : PW * ES <= 128 ? 128 : 256, PPR = RBY / 16;   // row bytes (a power of two), 16-byte pieces per row
    constexpr int RPI = 1024 / RBY;                                // rows a wave-wide 16-byte access covers
    constexpr int TP = (WM * RBY <= REGION) ? WM : REGION / RBY >= 64 ? 64 : 32;   // tokens per pass
    static_assert(TP * RBY <= REGION && TP % RPI == 0 && WM % TP == 0 && WN % PW == 0 && PW % 16 == 0, "epilogue region");
    wait_vm<0>();
    __syncthreads();
    char* const reg = smem + wave * REGION;
    const int64_t tok0 = m0 + WM * wm;
    const int col0 = n0 + WN * wn;
#pragma unroll
    for (int c0 = 0; c0 < WN; c0 += PW) {
#pragma unroll
        for (int t0 = 0; t0 < WM; t0 += TP) {
#pragma unroll
            for (int tj = c0 / 16; tj < (c0 + PW) / 16; ++tj) {
                const int cl = 16 * tj + 4 * g;                    // first of the lane's four outputs, within the wave's part
                f32x4 bv = {0.f, 0.f, 0.f, 0.f};
                if (a.bias) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col0 + cl + e < a.N) bv[e] = a.bias[col0 + cl + e];
                }
#pragma unroll
                for (int ti = t0 / 16; ti < (t0 + TP) / 16; ++ti) {
                    const int row = 16 * ti + lr - t0;
                    f32x4 v = {acc[tj][ti][0] + bv[0], acc[tj][ti][1] + bv[1], acc[tj][ti][2] + bv[2], acc[tj][ti][3] + bv[3]};
                    const int byte = (cl - c0) * ES;
                    char* const dst = reg + row * RBY + (((byte >> 4) ^ (row % PPR)) << 4) + (byte & 15);
                    if (OUT_BF16) *reinterpret_cast<bf16x4*>(dst) = __builtin_convertvector(v, bf16x4);
                    else *reinterpret_cast<f32x4*>(dst) = v;
                }
            }
#pragma unroll
            for (int i = 0; i < TP / RPI; ++i) {
                const int row = RPI * i + lane / PPR, piece = lane % PPR;
                const u32x4 val = *reinterpret_cast<const u32x4*>(reg + row * RBY + ((piece ^ (row % PPR)) << 4));
                const int64_t tok = tok0 + t0 + row;
                const int col = col0 + c0 + piece * (16 / ES);
                if (tok < a.T && col < a.N && (RBY == PW * ES || piece * 16 < PW * ES)) {
                    // the destination of this piece: the whole output, or the segment its first column lies in (segment
                    // boundaries are multiples of 8 columns, so a piece lies in one segment)
                    char* base = reinterpret_cast<char*>(a.y);
                    int64_t ld = a.ldy;
                    int c_lo = 0, c_hi = a.N;
                    if (a.n_seg > 0) {
#pragma unroll
                        for (int sg = 0; sg < LIN_MAX_SEG; ++sg)
                            if (sg < a.n_seg && col >= a.seg_col[sg]) {
                                base = reinterpret_cast<char*>(a.seg_y[sg]);
                                ld = a.seg_ld[sg];
                                c_lo = a.seg_col[sg];
                                c_hi = a.seg_col[sg + 1];
                            }
                    }
                    char* const p = base + (tok * ld + (col - c_lo)) * ES;
                    if (col + 16 / ES <= c_hi) {
                        *reinterpret_cast<u32x4*>(p) = val;
                    } else {
#pragma unroll
                        for (int e = 0; e < 16 / ES; ++e)
                            if (col + e < c_hi) {
                                if (OUT_BF16) reinterpret_cast<uint16_t*>(p)[e] = (uint16_t)(val[e >> 1] >> (16 * (e & 1)));
                                else reinterpret_cast<uint32_t*>(p)[e] = val[e];
                            }
                    }
                }
            }
        }
    }
}

template <typename CFG, bool OUT_BF16>
hipError_t launch_linear(LinearArgs a, hipStream_t stream) {
    static hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gdn_linear_kernel<CFG, OUT_BF16>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, CFG::SMEM);
    if (attr_err != hipSuccess) return attr_err;
    const int64_t tiles_m = (a.T + CFG::BM - 1) / CFG::BM;
    a.tiles_n = (a.N + CFG::BN - 1) / CFG::BN;
    a.tiles_m = (int32_t)tiles_m;
    a.per_xcd = (int32_t)((tiles_m * a.tiles_n + 7) / 8);
    hipLaunchKernelGGL((gdn_linear_kernel<CFG, OUT_BF16>), dim3((unsigned)(8 * (int64_t)a.per_xcd)), dim3(CFG::THREADS), CFG::SMEM, stream, a);
    return hipGetLastError();
}

std::atomic<int32_t> g_linear_shape{-1};

int chip_cus_linear() {
    static const int n = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
            (void)hipGetLastError();
            return 256;
        }
        return cus;
    }();
    return n;
}

// The estimated time of a problem in a tile shape, in us: full rounds of workgroups over the chip, and a last one that costs its latency (a
// workgroup alone walks k no faster) and more the fuller it is, since the compute units share power and memory.  A round has a part that
// grows with k and a part that does not (first loads, outputs): at K = 64 the second is the larger, and the more so
// the larger the tile, so a choice made at K = 2048 is up to 24 % off there (3000 x 6144 x 64 16.3 us in shape 2, 13.8 in shape 0; 8192 x 2560 x 256 22.9 / 19.9).
// Fitted to T = 1 .. 12000, N = 32 .. 8224, K = 64 .. 8192, all shapes at each, weights in the caches and not: the shape
// chosen is 0.5 % from the best of the five on average, 4 % and more in one case of twenty, at K >= 512 7 % at most, below (all of them calls
// of 4 to 7 us) 25 %; its estimate is within 14 % in nine of ten.  us, cold weights, K = 2048, in shapes 3 / 0 / 4 / 5 / 2:
// 512 x 2048 9.5 / 21 / 16 / 19 / 38, 1400 x 2048 20 / 23 / 18 / 21 / 39, 384 x 8224 31 / 31 / 22 / 27 / 47, 512 x 8224 39 / 31 / 36 / 27 / 49,
// 1000 x 8224 60 / 54 / 53 / 49 / 47, 700 x 6144 36 / 31 / 33 / 24 / 47, 2048 x 6144 76 / 58 / 57 / 63 / 47, 8192 x 2048 92 / 57 / 67 / 77 / 50,
// 8192 x 6144 283 / 173 / 205 / 204 / 147.
struct ShapeCost {
    int id, bm, bn, per_cu;
    double full_k, full, alone_k, alone;      // us of a full round, of a workgroup alone: per 2048 of k, and whatever k
    bool square;                              // the fullness of the last round counts squared
};
constexpr ShapeCost SHAPES[5] = {{3, 64, 64, 2, 10.4, 1.8, 3.9, 2.0, false},
                                 {0, 128, 128, 2, 26.0, 3.3, 14.4, 1.8, false},
                                 {4, 128, 128, 1, 14.2, 2.6, 10.4, 2.1, false},
                                 {5, 128, 160, 1, 15.9, 5.0, 12.9, 3.9, false},
                                 {2, 256, 256, 1, 41.9, 6.9, 32.6, 4.0, true}};
double shape_cost(const ShapeCost& c, int64_t T, int64_t N, int32_t K) {
    const int64_t tiles = ((T + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn), slots = (int64_t)chip_cus_linear() * c.per_cu;
    const double k = (double)K / 2048.0, f = (double)(tiles % slots) / (double)slots;
    const double full = c.full_k * k + c.full, alone = c.alone_k * k + c.alone;
    return (double)(tiles / slots) * full + (f > 0 ? alone + (full - alone) * (c.square ? f * f : f) : 0.0);
}

// Which tile shape a problem gets, and how many of its columns: a problem whose tiles leave a last round nearly empty may be cut
// into columns that fill whole rounds of 256 x 256 tiles and a rest in a smaller shape, a launch of its own.  Measured, whole / cut: 8192 x
// 8224 (33 tile columns where 32 fill four rounds) 233 / 211 us, 8192 x 2560 88 / 76, 2048 x 8224 90 / 65, 4096 x 8224 138 / 113.
struct LinearPlan { int shape, rest_shape; int32_t cols; };   // outputs 0 .. cols - 1 in `shape`, the others in `rest_shape`
LinearPlan plan_linear(int64_t T, int32_t N, int32_t K) {
    const int forced = g_linear_shape.load();
    if (forced >= 0) return {forced, 0, N};
    auto best_of = [&](int64_t n, int shapes, double* t) {
        int best = 0;
        for (int i = 0; i < shapes; ++i) {
            const double ti = shape_cost(SHAPES[i], T, n, K);
            if (i == 0 || ti < *t) { best = SHAPES[i].id; *t = ti; }
        }
        return best;
    };
    double whole = 0.0;
    LinearPlan p = {best_of(N, 5, &whole), 0, N};
    const double launch = 2.5;                           // a launch beyond its estimate
    double least = 0.97 * whole;                         // (a cut has to be worth it)
    const int64_t tiles_m = (T + 255) / 256, cus = chip_cus_linear();
    for (int64_t r = 1; r <= 64; ++r) {                  // the most columns that r rounds of 256 x 256 tiles hold
        const int64_t cols = r * cus / tiles_m * 256;
        if (cols >= N) break;
        if (cols == 0) continue;
        double rest = 0.0;
        const int rest_shape = best_of(N - cols, 4, &rest);
        const double t = shape_cost(SHAPES[4], T, cols, K) + rest + launch;
        if (t < least) { least = t; p = {2, rest_shape, (int32_t)cols}; }
    }
    return p;
}

}  // namespace linear
}  // namespace gdn

using namespace gdn;
using namespace gdn::linear;

namespace {
int32_t linear_checks(const void* x, int64_t ldx, const void* w, int64_t ldw, const float* bias, int32_t out_dtype, int64_t T, int32_t N,
                      int32_t K) {
    if (T < 0 || N < 0 || K < 0) return GDN_ERR_COUNT;
    if (out_dtype != GDN_BF16 && out_dtype != GDN_F32) return GDN_ERR_SHAPE;
    if (K % 64 != 0 || ldx < K || ldw < K) return GDN_ERR_SHAPE;
    if (T == 0 || N == 0) return GDN_OK;
    if (K == 0) return GDN_ERR_SHAPE;
    if (!x || !w) return GDN_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(x) & 15u) || (reinterpret_cast<uintptr_t>(w) & 15u) || (bias && (reinterpret_cast<uintptr_t>(bias) & 3u)))
        return GDN_ERR_ALIGN;
    if ((ldx & 7) || (ldw & 7)) return GDN_ERR_ALIGN;
    // a tile's rows must be addressable with 31-bit byte offsets
    if ((int64_t)256 * ldx * 2 >= ((int64_t)1 << 31) || (int64_t)256 * ldw * 2 >= ((int64_t)1 << 31)) return GDN_ERR_COUNT;
    if (((T + 127) / 128) * (((int64_t)N + 127) / 128) > INT32_MAX) return GDN_ERR_COUNT;
    return GDN_OK;
}

int32_t launch_shape(const LinearArgs& a, int shape, bool bf, hipStream_t stream) {
    hipError_t e;
    switch (shape) {
        case 1: e = bf ? launch_linear<LinBig, true>(a, stream) : launch_linear<LinBig, false>(a, stream); break;
        case 2: e = bf ? launch_linear<LinBig8, true>(a, stream) : launch_linear<LinBig8, false>(a, stream); break;
        case 3: e = bf ? launch_linear<LinTiny, true>(a, stream) : launch_linear<LinTiny, false>(a, stream); break;
        case 4: e = bf ? launch_linear<LinDeep, true>(a, stream) : launch_linear<LinDeep, false>(a, stream); break;
        case 5: e = bf ? launch_linear<LinWide, true>(a, stream) : launch_linear<LinWide, false>(a, stream); break;
        default: e = bf ? launch_linear<LinSmall, true>(a, stream) : launch_linear<LinSmall, false>(a, stream); break;
    }
    return hip_err(e);
}

// Columns c0 .. c1 - 1 of a projection as a projection of its own (c0 a multiple of 256: every alignment holds).
LinearArgs column_range(const LinearArgs& a, int32_t c0, int32_t c1, int es) {
    LinearArgs b = a;
    b.w = static_cast<const char*>(a.w) + (int64_t)c0 * a.ldw * 2;
    if (a.bias) b.bias = a.bias + c0;
    b.N = c1 - c0;
    if (a.n_seg == 0) {
        b.y = static_cast<char*>(a.y) + (int64_t)c0 * es;
        return b;
    }
    b.n_seg = 0;
    for (int32_t sg = 0; sg < a.n_seg; ++sg) {
        const int32_t lo = std::max(a.seg_col[sg], c0), hi = std::min(a.seg_col[sg + 1], c1);
        if (lo >= hi) continue;
        b.seg_col[b.n_seg] = lo - c0;
        b.seg_y[b.n_seg] = static_cast<char*>(a.seg_y[sg]) + (int64_t)(lo - a.seg_col[sg]) * es;
        b.seg_ld[b.n_seg] = a.seg_ld[sg];
        ++b.n_seg;
    }
    for (int32_t sg = b.n_seg; sg <= LIN_MAX_SEG; ++sg) b.seg_col[sg] = b.N;
    return b;
}

int32_t linear_launch(const LinearArgs& a, int32_t out_dtype, hipStream_t stream) {
    const bool bf = out_dtype == GDN_BF16;
    const LinearPlan p = plan_linear(a.T, a.N, a.K);
    if (p.cols == a.N) return launch_shape(a, p.shape, bf, stream);
    const int es = bf ? 2 : 4;
    const int32_t rc = launch_shape(column_range(a, 0, p.cols, es), p.shape, bf, stream);
    return rc != GDN_OK ? rc : launch_shape(column_range(a, p.cols, a.N, es), p.rest_shape, bf, stream);
}
}  // namespace

extern "C" int32_t gdn_linear(const void* x, int64_t ldx, const void* w, int64_t ldw, const float* bias, void* y, int64_t ldy,
                              int32_t out_dtype, int64_t T, int32_t N, int32_t K, void* stream_) {
    const int32_t rc = linear_checks(x, ldx, w, ldw, bias, out_dtype, T, N, K);
    if (rc != GDN_OK) return rc;
    if (ldy < N) return GDN_ERR_SHAPE;
    if (T == 0 || N == 0) return GDN_OK;
    if (!y) return GDN_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(y) & (out_dtype == GDN_BF16 ? 7u : 15u)) || (ldy & 3)) return GDN_ERR_ALIGN;
    LinearArgs a = {};
    a.x = x; a.w = w; a.bias = bias; a.y = y;
    a.ldx = ldx; a.ldw = ldw; a.ldy = ldy;
    a.T = T; a.N = N; a.K = K;
    a.n_seg = 0;
    return linear_launch(a, out_dtype, (hipStream_t)stream_);
}

extern "C" int32_t gdn_linear_split(const void* x, int64_t ldx, const void* w, int64_t ldw, const float* bias, int32_t n_seg,
                                    const int32_t* seg_cols, void* const* seg_y, const int64_t* seg_ld, int32_t out_dtype, int64_t T,
                                    int32_t K, void* stream_) {
    if (n_seg < 1 || n_seg > LIN_MAX_SEG) return GDN_ERR_COUNT;
    if (!seg_cols || !seg_y || !seg_ld) return GDN_ERR_NULL;
    if (seg_cols[0] != 0) return GDN_ERR_SHAPE;
    for (int32_t sg = 0; sg < n_seg; ++sg) {
        if (seg_cols[sg + 1] <= seg_cols[sg]) return GDN_ERR_SHAPE;                 // empty or decreasing
        if (sg + 1 < n_seg && (seg_cols[sg + 1] & 7)) return GDN_ERR_ALIGN;         // inner boundaries: whole 16-byte pieces
    }
    const int32_t N = seg_cols[n_seg];
    const int32_t rc = linear_checks(x, ldx, w, ldw, bias, out_dtype, T, N, K);
    if (rc != GDN_OK) return rc;
    for (int32_t sg = 0; sg < n_seg; ++sg) {
        if (seg_ld[sg] < seg_cols[sg + 1] - seg_cols[sg]) return GDN_ERR_SHAPE;
        if (T > 0 && !seg_y[sg]) return GDN_ERR_NULL;
        if ((reinterpret_cast<uintptr_t>(seg_y[sg]) & (out_dtype == GDN_BF16 ? 7u : 15u)) || (seg_ld[sg] & 3)) return GDN_ERR_ALIGN;
    }
    if (T == 0) return GDN_OK;
    LinearArgs a = {};
    a.x = x; a.w = w; a.bias = bias; a.y = seg_y[0];
    a.ldx = ldx; a.ldw = ldw; a.ldy = seg_ld[0];
    a.T = T; a.N = N; a.K = K;
    a.n_seg = n_seg;
    for (int32_t sg = 0; sg < n_seg; ++sg) {
        a.seg_col[sg] = seg_cols[sg];
        a.seg_y[sg] = seg_y[sg];
        a.seg_ld[sg] = seg_ld[sg];
    }
    for (int32_t sg = n_seg; sg <= LIN_MAX_SEG; ++sg) a.seg_col[sg] = N;
    return linear_launch(a, out_dtype, (hipStream_t)stream_);
}

extern "C" int32_t gdn_linear_plan(int64_t T, int32_t N, int32_t K, int32_t* shape, int32_t* cols, int32_t* rest_shape) {
    if (T <= 0 || N <= 0 || K <= 0) return GDN_ERR_COUNT;
    if (K % 64 != 0) return GDN_ERR_SHAPE;
    if (!shape || !cols || !rest_shape) return GDN_ERR_NULL;
    const LinearPlan p = plan_linear(T, N, K);
    *shape = p.shape;
    *cols = p.cols;
    *rest_shape = p.rest_shape;
    return GDN_OK;
}

extern "C" int32_t gdn_linear_tune(int32_t shape) {
    return g_linear_shape.exchange(shape < 0 || shape > 5 ? -1 : shape);
}
