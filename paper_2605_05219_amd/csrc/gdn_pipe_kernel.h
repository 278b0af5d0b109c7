// Pipelined fused kernel (bf16 inputs, d_k = d_v = D = 128 or 64, one value head per workgroup): the arithmetic of
// gdn_fused_kernel.h, result for result, with the preparation of a chain's next chunk on four waves of their own, beside the
// four waves that run the recurrence of the present one.
//
// What bounds it, and why this split: in the fused kernel a chunk of a chain takes the sum of its two dependent halves, the
// preparation (staging, diagonal inverse, L and P blocks) and the recurrence (four block rows of substitution, outputs,
// update), 12 k clocks alone on a compute unit, 16 to 18 k with a second workgroup beside it.  Neither half keeps the matrix pipe
// busy for a third of its time; they are chains of latencies.  Only the recurrence needs the state, so the preparation can run
// ahead: a chain then advances at the pace of the slower half, 7.8 k clocks a chunk with a preparation and a recurrence wave on
// every SIMD (preparation alone 6.2 k, recurrence alone 5.4 k).  One workgroup of eight waves per compute unit does as much work per
// clock as two of the fused kernel's (32768 chains the same time), and a chain goes twice as fast.  Measured at D = 128, before (fused kernel, or for
// the third the two-kernel path) and after: 1024 chains of up to 66 chunks, 15.3 k (chunk, chain) units 428 -> 299 us; 1024 chains of up to
// 345 chunks, 100 k units 2280 -> 1860; 96 chains of 128 chunks 648 -> 455; 8192 chains, 230 k units 4120 -> 4110.  With all compute units busy
// the clock is held at 1.8 to 1.95 GHz by the power limit (2.4 with half of them): the same 7.8 k clocks are 4.2 to 4.6 us or 3.3.
//
// Pipeline.  A workgroup's items are the chunks of one chain after the other.  The chains come longest first: workgroup b begins with
// chain b and draws each further one from a counter in memory, when the item of its present chain's last chunk is made out: a step
// before the draw's result is needed and three before the recurrence is done with that chunk, so no workgroup keeps a chain that another could
// start.  (Held in reserve a whole chain ahead, as the fused kernel does, the fullest of 256 workgroups got 76 chunks of 1024 chains with
// 60 on average and 66 in the longest, against 66: 293 -> 276 us; 458 of 391 on average and 345 in the longest, against 437: 1803 -> 1757.)
// Where a second round dealt backwards, chain 2 gridDim.x - 1 - b to workgroup b, keeps every pair within the longest chain, it is dealt so (deal_back): no
// deal is better, and draws among chains of a few chunks follow the order in which the workgroups happen to start (432 chains of up to 5 chunks, 2 on average, 42 us
// drawn, 37 dealt; 448 of up to 10 57 / 54; 256 of 3 32 / 31).
// In step t
//     the recurrence waves work on item t - 3: substitution, outputs, state update, emission,
//     the preparation waves prepare item t - 2 out of LDS, stage item t - 1 from registers to LDS (fp16) and fetch item t,
// and one barrier ends the step.  K and Q are held for three items in turn, pair tiles for two, gate vectors for three.  V is the
// recurrence waves' own: a wave fetches, converts and stages only its own columns, behind its last reads of the previous
// chunk's, so V needs one buffer and no barrier.  Rows are fetched a whole step ahead of their staging: staged and at once fetched again
// at the top of a step; a fetch half a step later costs 8 %, since the load then has half a step to arrive in (5 % in calls bound by volume).
//
// Rows come by ordinary loads (the fused kernel's are non-temporal): value heads that share a query/key head find each other's rows in
// the L2, 1024 chains of up to 345 chunks with two value heads to a query/key head 1895 -> 1832 us, 8192 chains without the same.
//
// Preparation wave a owns block row a and the P blocks of query block 3 - a; its code is instantiated per wave, so that all
// of it is one straight line in which the diagonal inverse's dependent products, the other blocks' products and the loads overlap.
// Wave 1 also walks the list of items one step ahead and leaves what the others need to know of an item in LDS (eight words,
// four items in turn): with every wave walking the list itself the plan's scalar loads and the registers they spilled cost 3 %.
//
// Tried without gain: raised priority of either kind of wave (preparation 0, recurrence 15 % slower); staging in the middle of the
// preparation (10 %: LDS writes there keep the compiler from reading ahead); V staged behind the update instead of before it (6 %).
//
// LDS (PipeSmem<D>: 150 KB at D = 128, 94 KB at D = 64: one workgroup per compute unit): tiles and swizzle as in the fused kernel, pair tiles unpadded
// (PairTiles).
#pragma once
#include <type_traits>
#include "gdn_chunk_ops.h"

namespace gdn {

// Profiling build only (-DGDN_PHASE_STAMPS, a library of its own: see build.py): cycle stamps at the phase boundaries of
// the 40th step of every fourth workgroup, one set per wave, read back by gdn_phase_stamps.  The product build has none.
#ifdef GDN_PHASE_STAMPS
__device__ unsigned long long g_pipe_ts[64 * 8 * 16];
#define GDN_STAMP(role_, k_)                                                                                        \
    do {                                                                                                            \
        if (gdn_step == 40 && (blockIdx.x & 3) == 0 && blockIdx.x < 256 && lane_ == 0)                              \
            g_pipe_ts[((blockIdx.x >> 2) * 8 + 4 * (role_) + wave) * 16 + (k_)] = __builtin_readcyclecounter();     \
    } while (0)
#define GDN_STAMP_STEP() (++gdn_step)
#else
#define GDN_STAMP(role_, k_) do {} while (0)
#define GDN_STAMP_STEP() ((void)0)
#endif

template <int D_>
struct PipeSmem {
    static constexpr int C = 64, D = D_;
    static constexpr int TILE_BYTES = C * D * 2;             // one of K, Q, V
    static constexpr int ROWS_OFF = 0, ROWS_BYTES = 2 * TILE_BYTES;      // [K | Q] of a chunk, three in turn
    static constexpr int V_OFF = ROWS_OFF + 3 * ROWS_BYTES;
    static constexpr int PAIRS_OFF = V_OFF + TILE_BYTES;                 // the pair tiles of a chunk, two in turn
    static constexpr int TF_OFF = PAIRS_OFF + 2 * PairTiles::BYTES;       // fp32 [16][16] per preparation wave
    static constexpr int TF_FLOATS = 16 * 16;
    static constexpr int GATES_OFF = TF_OFF + 4 * TF_FLOATS * 4;         // the gate vectors of a chunk, three in turn
    static constexpr int ITEM_OFF = GATES_OFF + 3 * GateVecs::BYTES;     // four items in turn, eight words each
    static constexpr int BYTES = ITEM_OFF + 4 * 32;
    static_assert(BYTES <= 160 * 1024, "a compute unit's LDS");
};

template <bool O_BF16, int D>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) gdn_pipe_kernel(FusedArgs a) {
    typedef Elem<half_t> EL;
    typedef EL::In In;
    typedef EL::Raw8 Raw8;
    typedef PipeSmem<D> SM;
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    constexpr int DK = D, DV = D;
    constexpr int NT = D / 64;        // 16-column tiles of the state per wave (a wave owns D / 4 columns of d_v)
    constexpr int MT = D / 16;        // 16-wide tiles over d_k
    constexpr int PCS = D / 8;        // 16-byte pieces per row
    constexpr int ROWS = D / 32;      // rows of K and of Q a preparation thread stages (256 threads, 64 rows of PCS pieces)
    constexpr int WC = D / 4;         // d_v columns per recurrence wave
    constexpr int WP = WC / 8;        // 16-byte pieces of a recurrence wave's part of a V row; as many pieces per lane

    const int tid = threadIdx.x & 255;
    const int lane_ = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool prep = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8) == 0;

    extern __shared__ __align__(16) char smem[];
    char* const Vt = smem + SM::V_OFF;
    const int units = a.L * a.H_v;
    const In* const qg = reinterpret_cast<const In*>(a.q);
    const In* const kg = reinterpret_cast<const In*>(a.k);
    const In* const vg = reinterpret_cast<const In*>(a.v);
    const int qk_step = a.H_qk * DK * 2, v_step = a.H_v * DV * 2;      // bytes from token to token

    // What a wave needs to know of an item (a chunk of a chain): eight words, in LDS.  n = 0: none; src: the pool slot of a new
    // chain's start state (-1: the zero state), or SAME_CHAIN.
    struct Item { int n, hq, hv, row_lo, row_hi, state, eslot, src; };
    int* const items = reinterpret_cast<int*>(smem + SM::ITEM_OFF);
    auto read_item = [&](int t) -> Item {
        const i32x4 x = *reinterpret_cast<const i32x4*>(items + 8 * (t & 3)), y = *reinterpret_cast<const i32x4*>(items + 8 * (t & 3) + 4);
        Item it;
        it.n = __builtin_amdgcn_readfirstlane(x[0]); it.hq = __builtin_amdgcn_readfirstlane(x[1]);
        it.hv = __builtin_amdgcn_readfirstlane(x[2]); it.row_lo = __builtin_amdgcn_readfirstlane(x[3]);
        it.row_hi = __builtin_amdgcn_readfirstlane(y[0]); it.state = __builtin_amdgcn_readfirstlane(y[1]);
        it.eslot = __builtin_amdgcn_readfirstlane(y[2]); it.src = __builtin_amdgcn_readfirstlane(y[3]);
        return it;
    };
    auto row_of = [](const Item& it) -> int64_t { return (int64_t)(uint32_t)it.row_lo | ((int64_t)it.row_hi << 32); };
    constexpr int SAME_CHAIN = -2;
    // the walk over the workgroup's items, by one wave (wave 1 of the preparation): the present chain and chunk
    struct Walk { int c, c_end, l, hv, hq, src; };
    Walk wk;
    int drawn = 0;                                              // in lane 0: the next chain less gridDim.x, drawn with the present one's last chunk
    const bool deal_back = a.deal_back && a.n_chains <= 2 * (int)gridDim.x;
    if (deal_back) drawn = (int)gridDim.x - 1 - (int)blockIdx.x;
    auto publish = [&](int t, bool live, bool fresh) {          // item t as the walk stands
        int w[8] = {0, 0, 0, 0, 0, 0, -1, SAME_CHAIN};
        if (live) {
            const int64_t row = (int64_t)wk.l * a.T_alloc + plan_word(a.chunk_tok0, wk.c);
            w[0] = plan_word(a.chunk_len, wk.c);
            w[1] = wk.hq; w[2] = wk.hv;
            w[3] = (int)(uint32_t)row; w[4] = (int)(row >> 32);
            w[5] = wk.l * a.H_v + wk.hv;
            w[6] = plan_word(a.chunk_emit_slot, wk.c);
            if (fresh) w[7] = wk.src;
        }
        if (lane_ < 8) {
            int x = w[0];
#pragma unroll
            for (int i = 1; i < 8; ++i) x = lane_ == i ? w[i] : x;
            items[8 * (t & 3) + lane_] = x;
        }
    };
    auto open_chain = [&](int chain) -> bool {
        if (chain >= a.n_chains) return false;
        const int r = plan_word(a.req_order, chain / units), lh = chain % units;
        wk.l = lh / a.H_v;
        wk.hv = lh % a.H_v;
        wk.hq = wk.hv / (a.H_v / a.H_qk);
        wk.c = plan_word(a.req_chunk_cu, r);
        wk.c_end = plan_word(a.req_chunk_cu, r + 1);
        wk.src = plan_word(a.req_src_slot, r);
        return true;
    };
    bool live = true;
    auto draw_behind_last = [&] {     // a step ahead of its use
        if (live && !deal_back && wk.c + 1 == wk.c_end && lane_ == 0) {
            int z = 0;
            pin(z);     // not a wave-uniform address to the compiler, which would wait for the result at once
            drawn = __hip_atomic_fetch_add(a.next_chain + z, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    auto walk_on = [&](int t) {       // publishes item t, the one after the walk's present one
        bool fresh = false;
        if (live) {
            if (wk.c + 1 < wk.c_end) {
                ++wk.c;
            } else {
                live = fresh = open_chain((int)gridDim.x + __builtin_amdgcn_readfirstlane(drawn));
                if (deal_back) drawn = a.n_chains;      // (no third)
            }
            draw_behind_last();
        }
        publish(t, live, fresh);
    };
    // A descriptor over the rows of an item's head in one tensor (no rows when there is no item).
#define GDN_ROWS(name_, base_, it_, heads_, head_, step_)                                                                       \
    const __amdgpu_buffer_rsrc_t name_ = __builtin_amdgcn_make_buffer_rsrc(                                                     \
        const_cast<In*>((base_) + (row_of(it_) * (heads_) + (head_)) * D), 0, (it_).n > 0 ? ((it_).n - 1) * (step_) + D * 2 : 0, 0x00020000)

    // Step t: the recurrence works on item t - 3, the preparation on item t - 2, staging on t - 1, the fetch on item t.
    if (prep && wave == 1) {
        if (lane_ < 32) items[lane_] = (lane_ & 7) == 7 ? SAME_CHAIN : (lane_ & 7) == 6 ? -1 : 0;    // none
        live = open_chain((int)blockIdx.x);
        draw_behind_last();
        publish(0, live, true);
    }
    __syncthreads();
    int t = 0;                       // every wave leaves after the step in which the recurrence worked on the last item
    int s0 = 0, s1 = 1, s2 = 2;      // K/Q and gate buffers of the three items held in LDS
    int gdn_step = 0;
    (void)gdn_step;
    int p0 = 0;                      // pair tiles read by the recurrence; the preparation writes the other

    if (prep) {
        Raw8 kraw[ROWS], qraw[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) kraw[r] = qraw[r] = EL::zero_raw();
        In graw = In();
        int n1 = 0, n2 = 0;
        for (;;) {
            GDN_STAMP_STEP();
            GDN_STAMP(0, 0);
            int lane = lane_, tg = tid / PCS, d0 = (tid % PCS) * 8;
            pin(lane); pin(tg); pin(d0);
            const Item i3 = read_item(t);
            char* const Kt2 = smem + SM::ROWS_OFF + s2 * SM::ROWS_BYTES;
            float* const gates2 = reinterpret_cast<float*>(smem + SM::GATES_OFF + s2 * GateVecs::BYTES);
            const char* const Kt = smem + SM::ROWS_OFF + s1 * SM::ROWS_BYTES;
            const float* const gates = reinterpret_cast<const float*>(smem + SM::GATES_OFF + s1 * GateVecs::BYTES);
            float* const Tf = reinterpret_cast<float*>(smem + SM::TF_OFF) + wave * SM::TF_FLOATS;
            char* const pairs = smem + SM::PAIRS_OFF + (p0 ^ 1) * PairTiles::BYTES;
            auto step = [&](auto ab_) {
                constexpr int ab = decltype(ab_)::value;
                GDN_ROWS(rk, kg, i3, a.H_qk, i3.hq, qk_step);
                GDN_ROWS(rq, qg, i3, a.H_qk, i3.hq, qk_step);
                auto fetch = [&](int r) {
                    if (r < ROWS) kraw[r < ROWS ? r : 0] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(rk, (ROWS * tg + r) * qk_step + d0 * 2, 0, 0));
                    else qraw[r >= ROWS ? r - ROWS : 0] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(rq, (ROWS * tg + r - ROWS) * qk_step + d0 * 2, 0, 0));
                };
                // a quarter of the staging of i2, and of the fetch of i3 into the registers that this frees
                auto place = [&](int p) {
#pragma unroll
                    for (int r = p * ROWS / 4; r < (p + 1) * ROWS / 4; ++r) {
                        stage_piece<D>(Kt2, kraw[r], ROWS * tg + r, d0);
                        stage_piece<D>(Kt2 + SM::TILE_BYTES, qraw[r], ROWS * tg + r, d0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int r = p * ROWS / 4; r < (p + 1) * ROWS / 4; ++r) { fetch(r); fetch(ROWS + r); }
                    __builtin_amdgcn_sched_barrier(0);
                };
                place(0); place(1); place(2); place(3);
                if (ab == 0) gate_vectors(gates2, lane < n2 ? fmaxf(EL::log_(EL::widen(graw)), -88.f) : 0.f, lane);
                else if (ab == 1) gates2[GateVecs::B + lane] = lane < n2 ? EL::widen(graw) : 0.f;
                __builtin_amdgcn_sched_barrier(0);
                if (ab < 2) {
                    if (lane < i3.n)
                        graw = (reinterpret_cast<const In*>(ab == 0 ? a.gate : a.beta) + (row_of(i3) * a.H_v + i3.hv))[lane * a.H_v];
                }
                __builtin_amdgcn_sched_barrier(0);
                operand_blocks<D, ab>(Kt, Kt + SM::TILE_BYTES, gates, Tf, pairs, a.scale, lane);
            };
            // (items that are none are staged and prepared like any other: their rows read as zeros, their results go nowhere)
            if (wave == 0) step(std::integral_constant<int, 0>());
            else if (wave == 1) step(std::integral_constant<int, 1>());
            else if (wave == 2) step(std::integral_constant<int, 2>());
            else step(std::integral_constant<int, 3>());
            GDN_STAMP(0, 1);
            if (wave == 1) walk_on(t + 1);
            __syncthreads();
            GDN_STAMP(0, 2);
            if (t >= 3 && n1 == 0) break;
            n1 = n2; n2 = i3.n;
            ++t;
            const int x = s0; s0 = s1; s1 = s2; s2 = x;
            p0 ^= 1;
        }
    } else {
        Raw8 vraw[WP];
        Item i0 = {0, 0, 0, 0, 0, 0, -1, SAME_CHAIN}, i1 = i0;
#pragma unroll
        for (int r = 0; r < WP; ++r) vraw[r] = EL::zero_raw();
        f32x4 accS[MT][NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) accS[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (;;) {
            GDN_STAMP_STEP();
            GDN_STAMP(1, 0);
            int lane = lane_;
            pin(lane);
            const int m = lane & 15, g4 = lane >> 4;
            const Item i2 = read_item(t - 1);
            const int vrow = lane / WP, vpc = WP * wave + lane % WP;     // row (+ 64 / WP r) and piece of V this lane moves

            const int64_t head_off = (int64_t)i0.state * DV * DK;
            half8 ud[2][NT];   // diag(dec) U, like uh
            const char* const Kt = smem + SM::ROWS_OFF + s0 * SM::ROWS_BYTES;
            const float* const gates = reinterpret_cast<const float*>(smem + SM::GATES_OFF + s0 * GateVecs::BYTES);
            {
                constexpr int OB = O_BF16 ? 2 : 4;
                const int o_step = a.H_v * DV * OB;
                substitute<O_BF16, D, NT, D, false>(Kt, Kt + SM::TILE_BYTES, Vt, WP * wave, smem + SM::PAIRS_OFF + p0 * PairTiles::BYTES, gates + GateVecs::GAM,
                                             gates + GateVecs::DEC, accS, ud,
                                             reinterpret_cast<const char*>(a.o) + ((row_of(i0) * a.H_v + i0.hv) * DV + WC * wave) * OB,
                                             i0.n > 0 ? (i0.n - 1) * o_step + WC * OB : 0, o_step, a.scale, lane);
            }
            GDN_STAMP(1, 1);
            __builtin_amdgcn_sched_barrier(0);
            // ---- V of i1 into the wave's own columns of the tile, V of i2 from memory
#pragma unroll
            for (int r = 0; r < WP; ++r) {
                const int i = (64 / WP) * r + vrow;
                stage_piece<D>(Vt, vraw[r], i, 8 * vpc);
            }
            {
                GDN_ROWS(rv, vg, i2, a.H_v, i2.hv, v_step);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < WP; ++r)
                    vraw[r] = __builtin_bit_cast(Raw8, __builtin_amdgcn_raw_buffer_load_b128(rv, ((64 / WP) * r + vrow) * v_step + vpc * 16, 0, 0));
                __builtin_amdgcn_sched_barrier(0);
            }
            GDN_STAMP(1, 2);
            update_state<D, NT>(Kt, gates[GateVecs::GAM + 63], ud, accS, lane);
            GDN_STAMP(1, 3);
            if (i0.eslot >= 0) {     // checkpoint emission: exact state after the last token of this chunk
                {
                    float* dst = a.state_dst + i0.eslot * a.dst_slot_stride + head_off;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            *reinterpret_cast<f32x4*>(dst + (WC * wave + 16 * nt + m) * DK + 32 * (mt >> 1) + 8 * g4 + 4 * (mt & 1)) = accS[mt][nt];
                }
            }
            GDN_STAMP(1, 4);
            if (i1.src != SAME_CHAIN) {     // a new chain: its start state, from the pool slot or zero
                const int slot = i1.src;
                if (slot >= 0) {
                    const float* src = a.state_src + slot * a.src_slot_stride + (int64_t)i1.state * DV * DK;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            accS[mt][nt] = *reinterpret_cast<const f32x4*>(src + (WC * wave + 16 * nt + m) * DK + 32 * (mt >> 1) + 8 * g4 + 4 * (mt & 1));
                    wait_vmcnt<0>();     // here, so that no other path has to wait for loads at the top of a step
                } else {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) accS[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
            GDN_STAMP(1, 5);
            __syncthreads();
            GDN_STAMP(1, 6);
            if (t >= 3 && i1.n == 0) break;
            i0 = i1; i1 = i2;
            ++t;
            const int x = s0; s0 = s1; s1 = s2; s2 = x;
            p0 ^= 1;
        }
    }
}

#undef GDN_ROWS

}  // namespace gdn
