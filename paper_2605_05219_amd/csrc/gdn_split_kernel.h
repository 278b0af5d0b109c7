// Fewer chains than keep the compute units busy (bf16 inputs, d_k = d_v = D = 128 or 64): the operand blocks of all chunks in one launch,
// parallel over the chunks (gdn_blocks_kernel), then the recurrence, CW = 32 or 64 columns of d_v to a workgroup (gdn_subst_kernel).
// The arithmetic is that of the fused kernels, result for result.
//
// What bounds the calls this is for is their longest chain.  The pipelined fused kernel takes a chain through at 3.3 us a chunk, the pace of its
// preparation waves, on one compute unit, while others stand idle; the two-kernel path's preparation forms the full inverse and an image of 72 KB a
// unit, 27 ns a unit with the whole chip, and its latency variant shares the chip with it (1.2 us a chunk for 16 chains, 2.4 for
// 32, 3.4 for 64).  Here a unit's blocks are 14.5 KB (pair tiles, gam, dec) at 10 ns (47 KB read and written: 4.7 TB/s), and a chunk takes the recurrence waves alone: 1.7 us with 32
// columns to a workgroup, 2.1 with 64 (clocks: substitution and outputs 2750, update 830, barrier 150; a recurrence wave has 16
// columns, the four helper waves, which bring and stage K, Q, V and the blocks, wait half of the time).  Measured at D = 128, two-kernel / pipelined / CW = 64 /
// CW = 32, us: 48 chains of 128 chunks 344 / 446 / 340 / 303, of 8 chunks 35 / 46 / 33 / 29; 64 chains of 128 441 / 450 / 377 / 348, of 32 111 / 126 / 96 / 86; 96 ragged
// chains of up to 86 chunks 340 / 308 / 220 / 192; 96 of 32 chunks 186 / 127 / 110 / 148, of 2 chunks 29 / 26 / 21 / 24; 128 of 128 838 / 455 / 538 / 668.  D = 64: 64 of
// 32 95 / 85 / 67 / 61, 128 ragged 234 / 206 / 166 / 146.
//
// Tried without gain: LDS operands read where they are used instead of one to two block rows ahead (the same); fetches one step ahead
// instead of two (1.85 us a chunk); one unit to a preparation workgroup (16 ns a unit), 1 KB more of LDS to one, which leaves room for two instead of
// three (12 ns).
#pragma once
#include <type_traits>
#include "gdn_chunk_ops.h"

namespace gdn {

// What the blocks of one (chunk, layer, value head) unit look like in the workspace: the pair tiles, gam and dec.
struct BlockUnit {
    static constexpr int GAM_OFF = PairTiles::BYTES, DEC_OFF = GAM_OFF + 256, BYTES = DEC_OFF + 256;
    static_assert(BYTES % 256 == 0, "aligned units");
};

struct SplitArgs {
    const void* q;
    const void* k;
    const void* v;
    const void* beta;
    const void* gate;
    void* o;
    char* blocks;                    // n_units units, chunk-major: ((chunk L) + layer) H_v + value head
    const int32_t* chunk_tok0;
    const int32_t* chunk_len;
    const int32_t* chunk_emit_slot;
    const int32_t* req_chunk_cu;
    const int32_t* req_src_slot;
    const int32_t* req_order;        // requests, longest chain first
    const float* state_src;
    float* state_dst;
    int64_t src_slot_stride, dst_slot_stride;
    int32_t n_chains, n_units;
    int32_t L, H_qk, H_v;
    int64_t T_alloc;
    float scale;
    int32_t o_bf16;
    HostFetch fetch;
};

// A workgroup of four waves per compute-unit third takes units at the grid's stride and fetches the next one's rows while it works.
template <int D>
struct BlocksSmem {
    static constexpr int TILE_BYTES = 64 * D * 2;
    static constexpr int K_OFF = 0, Q_OFF = TILE_BYTES, PAIRS_OFF = 2 * TILE_BYTES, TF_OFF = PAIRS_OFF + PairTiles::BYTES, TF_FLOATS = 16 * 16;
    static constexpr int GATES_OFF = TF_OFF + 4 * TF_FLOATS * 4, BYTES = GATES_OFF + GateVecs::BYTES;
    static_assert(3 * ((BYTES + 1279) / 1280 * 1280) <= 160 * 1024, "three workgroups per compute unit (LDS is given out in 1280 bytes)");
};

template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) gdn_blocks_kernel(SplitArgs a) {
    typedef Elem<half_t> EL;
    typedef EL::In In;
    typedef EL::Raw8 Raw8;
    typedef BlocksSmem<D> SM;
    constexpr int PCS = D / 8, ROWS = D / 32;
    __shared__ __align__(16) char smem[SM::BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int n_work = (int)gridDim.x - a.fetch.n_copy_wgs, wg = (int)blockIdx.x - a.fetch.n_copy_wgs;
    if (wg < 0) {         // first in the grid: the copies begin with the launch
        copy_staged(a.fetch, (int)blockIdx.x, tid);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int heads = a.L * a.H_v, qk_step = a.H_qk * D * 2;
    const int tg = tid / PCS, d0 = (tid % PCS) * 8;
    float* const gates = reinterpret_cast<float*>(smem + SM::GATES_OFF);
    float* const Tf = reinterpret_cast<float*>(smem + SM::TF_OFF) + wave * SM::TF_FLOATS;
    // a unit's rows and gates, fetched while the one before it is worked on
    Raw8 kraw[ROWS], qraw[ROWS];
    In graw = In();
    int n = 0;
#define GDN_FETCH_UNIT(u_)                                                                                                      \
    do {                                                                                                                        \
        const int c_ = (u_) / heads, lh_ = (u_) % heads, hv_ = lh_ % a.H_v, hq_ = hv_ / (a.H_v / a.H_qk);                       \
        n = plan_word(a.chunk_len, c_);                                                                                         \
        const int64_t row_ = (int64_t)(lh_ / a.H_v) * a.T_alloc + plan_word(a.chunk_tok0, c_);                                  \
        const int bytes_ = (n - 1) * qk_step + D * 2;                                                                           \
        const __amdgpu_buffer_rsrc_t rk_ = __builtin_amdgcn_make_buffer_rsrc(                                                   \
            const_cast<In*>(reinterpret_cast<const In*>(a.k) + (row_ * a.H_qk + hq_) * D), 0, bytes_, 0x00020000);              \
        const __amdgpu_buffer_rsrc_t rq_ = __builtin_amdgcn_make_buffer_rsrc(                                                   \
            const_cast<In*>(reinterpret_cast<const In*>(a.q) + (row_ * a.H_qk + hq_) * D), 0, bytes_, 0x00020000);              \
        _Pragma("unroll") for (int r_ = 0; r_ < ROWS; ++r_) {                                                                   \
            kraw[r_] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(rk_, (ROWS * tg + r_) * qk_step + d0 * 2, 0, 0)); \
            qraw[r_] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(rq_, (ROWS * tg + r_) * qk_step + d0 * 2, 0, 0)); \
        }                                                                                                                       \
        if (wave < 2 && lane < n)                                                                                               \
            graw = (reinterpret_cast<const In*>(wave == 0 ? a.gate : a.beta) + (row_ * a.H_v + hv_))[lane * a.H_v];             \
    } while (0)
    int u = wg;
    if (u >= a.n_units) return;
    GDN_FETCH_UNIT(u);
    for (;;) {
        if (wave == 0) gate_vectors(gates, lane < n ? fmaxf(EL::log_(EL::widen(graw)), -88.f) : 0.f, lane);
        else if (wave == 1) gates[GateVecs::B + lane] = lane < n ? EL::widen(graw) : 0.f;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            stage_piece<D>(smem + SM::K_OFF, kraw[r], ROWS * tg + r, d0);
            stage_piece<D>(smem + SM::Q_OFF, qraw[r], ROWS * tg + r, d0);
        }
        const int next = u + n_work;
        if (next < a.n_units) GDN_FETCH_UNIT(next);
        __syncthreads();
        auto blocks = [&](auto ab_) {
            operand_blocks<D, decltype(ab_)::value>(smem + SM::K_OFF, smem + SM::Q_OFF, gates, Tf, smem + SM::PAIRS_OFF, a.scale, lane);
        };
        if (wave == 0) blocks(std::integral_constant<int, 0>());
        else if (wave == 1) blocks(std::integral_constant<int, 1>());
        else if (wave == 2) blocks(std::integral_constant<int, 2>());
        else blocks(std::integral_constant<int, 3>());
        __syncthreads();
        char* const dst = a.blocks + (int64_t)u * BlockUnit::BYTES;
        for (int i = tid; i < PairTiles::BYTES / 16; i += 256)
            reinterpret_cast<u32x4*>(dst)[i] = reinterpret_cast<const u32x4*>(smem + SM::PAIRS_OFF)[i];
        if (tid < 128) reinterpret_cast<float*>(dst + BlockUnit::GAM_OFF)[tid] = gates[GateVecs::GAM + tid];     // gam, then dec
        if (next >= a.n_units) break;
        u = next;
        __syncthreads();       // the tiles have been read: the next unit's may be staged
    }
#undef GDN_FETCH_UNIT
}

template <int D, int CW>
struct SubstSmem {
    static constexpr int TILE_BYTES = 64 * D * 2, ROWS_BYTES = 2 * TILE_BYTES;     // [K | Q] of a chunk, two in turn
    static constexpr int VD = 64, V_BYTES = 64 * VD * 2;                           // the workgroup's columns of V (in the first CW)
    static constexpr int UNIT_BYTES = 16 * 1024;                                   // a unit of blocks (BlockUnit::BYTES of it used), two in turn
    static constexpr int ROWS_OFF = 0, V_OFF = 2 * ROWS_BYTES, UNIT_OFF = V_OFF + 2 * V_BYTES, BYTES = UNIT_OFF + 2 * UNIT_BYTES;
    static_assert(BYTES <= 160 * 1024, "a compute unit's LDS");
};

// CW / 16 recurrence waves behind four helper waves.  Grid: the n_chains chains' column blocks, block b = columns CW ((b / 8) % (D / CW)) of chain (b / (8 D / CW)) 8 + b % 8, so that the
// workgroups of a chain sit on one XCD and share its rows and blocks in the L2.
template <bool O_BF16, int D, int CW>
__global__ void __launch_bounds__(256 + 4 * CW) __attribute__((amdgpu_waves_per_eu(2, 2))) gdn_subst_kernel(SplitArgs a) {
    typedef Elem<half_t> EL;
    typedef EL::In In;
    typedef EL::Raw8 Raw8;
    typedef SubstSmem<D, CW> SM;
    constexpr int DK = D, DV = D, MT = D / 16, PCS = D / 8, ROWS = D / 32, NCB = D / CW;
    static_assert(CW == 32 || CW == 64, "whole pieces of V for every helper thread");
    constexpr int VP = CW / 32;                       // 16-byte pieces of V per helper thread
    constexpr int UP = SM::UNIT_BYTES / 16 / 256;     // pieces of a unit per helper thread
    const int chain = (int)(blockIdx.x / (8 * NCB)) * 8 + (int)(blockIdx.x & 7), col0 = CW * (int)((blockIdx.x >> 3) % NCB);
    if (chain >= a.n_chains) return;
    const int tid = threadIdx.x & 255;
    const int lane_ = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool helper = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8) == 0;
    extern __shared__ __align__(16) char smem[];

    const int heads = a.L * a.H_v;
    const int r = plan_word(a.req_order, chain / heads), lh = chain % heads, l = lh / a.H_v, hv = lh % a.H_v, hq = hv / (a.H_v / a.H_qk);
    const int c0 = plan_word(a.req_chunk_cu, r), n_items = plan_word(a.req_chunk_cu, r + 1) - c0;
    const int qk_step = a.H_qk * DK * 2, v_step = a.H_v * DV * 2;

    // The plan's words of 64 items, one per lane, read again every 64 items.
    int w_tok = 0, w_len = 0, w_slot = 0;
    auto words = [&](int base) {
        const int c = c0 + min(base + lane_, n_items - 1);
        w_tok = a.chunk_tok0[c];
        w_len = a.chunk_len[c];
        w_slot = a.chunk_emit_slot[c];
        wait_vmcnt<0>();
    };
#define GDN_ROWS(name_, base_, row_, n_, heads_, head_, step_)                                                                  \
    const __amdgpu_buffer_rsrc_t name_ = __builtin_amdgcn_make_buffer_rsrc(                                                     \
        const_cast<In*>(reinterpret_cast<const In*>(base_) + ((row_) * (heads_) + (head_)) * D), 0, (n_) > 0 ? ((n_) - 1) * (step_) + D * 2 : 0, 0x00020000)

    // Step t: the recurrence works on item t - 2, item t - 1 is staged from registers to LDS, item t + 1 fetched; one barrier ends a
    // step.  Two sets of registers: a fetch has two steps to arrive in.
    if (helper) {
        Raw8 kraw[2][ROWS], qraw[2][ROWS], uraw[2][UP], vraw[2][VP];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) kraw[s][i] = qraw[s][i] = EL::zero_raw();
#pragma unroll
            for (int i = 0; i < UP; ++i) uraw[s][i] = EL::zero_raw();
#pragma unroll
            for (int i = 0; i < VP; ++i) vraw[s][i] = EL::zero_raw();
        }
        auto step = [&](int t, auto set_) {          // set = (t - 1) & 1
            constexpr int set = decltype(set_)::value;
            int tu = tid;
            pin(tu);
            const int tg = tu / PCS, d0 = (tu % PCS) * 8, vr = tu / (CW / 8), vc = tu % (CW / 8);     // row groups and pieces of K and Q, of V
            const int it = t + 1;
            if ((it & 63) == 0) words(it);
            const int n = it < n_items ? __builtin_amdgcn_readlane(w_len, it & 63) : 0;
            const int64_t row = (int64_t)l * a.T_alloc + __builtin_amdgcn_readlane(w_tok, it & 63);
            char* const Kt = smem + SM::ROWS_OFF + set * SM::ROWS_BYTES;
            char* const Ut = smem + SM::UNIT_OFF + set * SM::UNIT_BYTES;
            char* const Vt = smem + SM::V_OFF + set * SM::V_BYTES;
            GDN_ROWS(rk, a.k, row, n, a.H_qk, hq, qk_step);
            GDN_ROWS(rq, a.q, row, n, a.H_qk, hq, qk_step);
            GDN_ROWS(rv, a.v, row, n, a.H_v, hv, v_step);
            const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(
                a.blocks + ((int64_t)(c0 + min(it, n_items - 1)) * heads + lh) * BlockUnit::BYTES, 0, it < n_items ? BlockUnit::BYTES : 0, 0x00020000);
#pragma unroll
            for (int i = 0; i < UP; ++i) {
                reinterpret_cast<Raw8*>(Ut)[256 * i + tu] = uraw[set][i];
                __builtin_amdgcn_sched_barrier(0);
                uraw[set][i] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(ru, (256 * i + tu) * 16, 0, 0));
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                stage_piece<D>(Kt, kraw[set][i], ROWS * tg + i, d0);
                stage_piece<D>(Kt + SM::TILE_BYTES, qraw[set][i], ROWS * tg + i, d0);
                __builtin_amdgcn_sched_barrier(0);
                kraw[set][i] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(rk, (ROWS * tg + i) * qk_step + d0 * 2, 0, 0));
                qraw[set][i] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(rq, (ROWS * tg + i) * qk_step + d0 * 2, 0, 0));
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < VP; ++i) {
                const int vrow = vr + i * (256 / (CW / 8));
                // (true for every row; as a condition it keeps the write in a block of its own: CW = 32, 64 ragged chains of up to 125 chunks 243 -> 238 us)
                if (CW == 64 || vrow < 64) stage_piece<SM::VD>(Vt, vraw[set][i], vrow, 8 * vc);
                __builtin_amdgcn_sched_barrier(0);
                vraw[set][i] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(rv, vrow * v_step + col0 * 2 + vc * 16, 0, 2));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (t >= 0) __syncthreads();
        };
        words(0);
        step(-1, std::integral_constant<int, 0>());       // fetches item 0 (and stages nothing that is read)
        for (int t = 0; t < n_items + 2; t += 2) {
            step(t, std::integral_constant<int, 1>());
            if (t + 1 < n_items + 2) step(t + 1, std::integral_constant<int, 0>());
        }
    } else {
        const int64_t state_off = (int64_t)lh * DV * DK + (int64_t)(col0 + 16 * wave) * DK;
        f32x4 accS[MT][1];
        const int slot = plan_word(a.req_src_slot, r);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) accS[mt][0] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (slot >= 0) {           // the start state, from the pool slot or zero
            const float* src = a.state_src + slot * a.src_slot_stride + state_off;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                accS[mt][0] = *reinterpret_cast<const f32x4*>(src + (lane_ & 15) * DK + 32 * (mt >> 1) + 8 * (lane_ >> 4) + 4 * (mt & 1));
        }
        __syncthreads();
        __syncthreads();           // the first item has been staged
        for (int it = 0; it < n_items; ++it) {
            int lane = lane_;
            pin(lane);
            const int m = lane & 15, g4 = lane >> 4;
            if ((it & 63) == 0) words(it);
            const int n = __builtin_amdgcn_readlane(w_len, it & 63), eslot = __builtin_amdgcn_readlane(w_slot, it & 63);
            const int64_t row = (int64_t)l * a.T_alloc + __builtin_amdgcn_readlane(w_tok, it & 63);
            const char* const Kt = smem + SM::ROWS_OFF + (it & 1) * SM::ROWS_BYTES;
            const char* const Ut = smem + SM::UNIT_OFF + (it & 1) * SM::UNIT_BYTES;
            const float* const gamS = reinterpret_cast<const float*>(Ut + BlockUnit::GAM_OFF);
            const float* const decS = reinterpret_cast<const float*>(Ut + BlockUnit::DEC_OFF);
            constexpr int OB = O_BF16 ? 2 : 4;
            const int o_step = a.H_v * DV * OB;
            half8 ud[2][1];
            substitute<O_BF16, D, 1, SM::VD, true>(Kt, Kt + SM::TILE_BYTES, smem + SM::V_OFF + (it & 1) * SM::V_BYTES, 2 * wave, Ut, gamS, decS,
                                                   accS, ud, reinterpret_cast<const char*>(a.o) + ((row * a.H_v + hv) * DV + col0 + 16 * wave) * OB,
                                                   (n - 1) * o_step + 16 * OB, o_step, a.scale, lane);
            update_state<D, 1>(Kt, gamS[63], ud, accS, lane);
            if (eslot >= 0) {       // checkpoint emission: exact state after the last token of this chunk
                float* dst = a.state_dst + eslot * a.dst_slot_stride + state_off;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    *reinterpret_cast<f32x4*>(dst + m * DK + 32 * (mt >> 1) + 8 * g4 + 4 * (mt & 1)) = accS[mt][0];
            }
            __syncthreads();
        }
    }
#undef GDN_ROWS
}

}  // namespace gdn
