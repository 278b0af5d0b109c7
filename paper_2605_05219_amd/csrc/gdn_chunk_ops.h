// The steps of one 64-token chunk as the kernels with separate preparation and recurrence waves (or launches) use them: the
// gate vectors, the operand blocks, substitution and outputs, the state update.  The mathematics, the tile layouts and the swizzle are
// those of gdn_fused_kernel.h, and so is the arithmetic, result for result.
//
// Pair tiles here are [16][2 x 16] fp16, rows unpadded: lane (m, g4) reads 16 bytes at row m, piece g4, so that a wave's
// read of a tile is the tile's 1 KiB in order, free of bank conflicts.
#pragma once
#include "gdn_fused_kernel.h"

namespace gdn {

// The pair tiles of a chunk: TbTg[a] = [T_aa diag(b) | -T_aa diag(b gam)] (4 tiles), M = -T_aa L_ac (4), P (6); a lone block's
// partner half is zero.
struct PairTiles {
    static constexpr int LD = 32, TILE = 16 * LD * 2;        // halfs per row, bytes of a tile
    static constexpr int TBTG = 0, M = 4 * TILE, P = 8 * TILE, BYTES = 14 * TILE;
    static constexpr __host__ __device__ int m_pair(int a, int c) { return (a == 1 ? 0 : a == 2 ? 1 : 2) + (c >> 1); }
    static constexpr __host__ __device__ int p_pair(int a, int c) { return (a == 0 ? 0 : a == 1 ? 1 : a == 2 ? 2 : 4) + (c >> 1); }
};

// The gate vectors of a chunk, fp32 [64] each: g, b, gam, dec, s and three r (see the gates of gdn_fused_kernel.h).
struct GateVecs {
    static constexpr int C = 64, G = 0, B = C, GAM = 2 * C, DEC = 3 * C, S = 4 * C, R = 5 * C, FLOATS = 8 * C, BYTES = FLOATS * 4;
};
// All but b, by one wave: la = the lane's log gate (0 past the chunk's end).
__device__ __forceinline__ void gate_vectors(float* v, float la, int lane) {
    typedef Elem<half_t> EL;
    const float s = wave_running_sum(la);
    const int sbits = __builtin_bit_cast(int, s);
    const float e0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(sbits, 15));
    const float e1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(sbits, 31));
    const float e2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(sbits, 47));
    const float g_last = wave_last_lane(s);
    const float eb = lane < 16 ? e0 : lane < 32 ? e1 : lane < 48 ? e2 : g_last;
    v[GateVecs::G + lane] = s;
    v[GateVecs::GAM + lane] = EL::exp_(s);
    v[GateVecs::DEC + lane] = EL::exp_(g_last - s);
    v[GateVecs::S + lane] = EL::exp_(fminf(eb - s, 0.f));
    v[GateVecs::R + lane] = EL::exp_(fminf(s - e0, 0.f));
    v[GateVecs::R + 64 + lane] = EL::exp_(fminf(s - e1, 0.f));
    v[GateVecs::R + 128 + lane] = EL::exp_(fminf(s - e2, 0.f));
}

// Raw bf16 piece (8 columns from d0 on) of row i, widened exactly to fp16, into a [64][D] tile.
template <int D>
__device__ __forceinline__ void stage_piece(char* tile, const Elem<half_t>::Raw8& raw, int i, int d0) {
    float x[8];
    Elem<half_t>::unpack(raw, x);
    half8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (half_t)x[e];
    *reinterpret_cast<half8*>(tile + i * 2 * D + (((d0 >> 3) ^ swz<D>(i)) << 4)) = h;
}

// operand over d_k columns 32 s + 8 g4 .. + 7 of row 16 blk + m of a [64][D] tile
template <int D>
__device__ __forceinline__ half8 row_operand(const char* tile, int blk, int s, int m, int g4) {
    return *reinterpret_cast<const half8*>(tile + (m * 2 * D + 16 * ((4 * s + g4) ^ swz<D>(m))) + blk * 16 * 2 * D);
}

// One preparation wave's operand blocks: block row ab of L and the P blocks of query block 3 - ab, straight-line code in
// which the diagonal inverse's dependent products and the other blocks' products overlap.  Tf: fp32 [16][16] of the wave's own (read in order).
template <int D, int ab>
__device__ __forceinline__ void operand_blocks(const char* Kt, const char* Qt, const float* gates, float* Tf, char* pairs, float scale, int lane) {
    typedef Elem<half_t> EL;
    constexpr int SS = D / 32, ia = 3 - ab, TF_LD = 16, LD = PairTiles::LD;
    const int m = lane & 15, g4 = lane >> 4;
    const float* const gS = gates + GateVecs::G;
    const float* const bS = gates + GateVecs::B;
    const float* const gamS = gates + GateVecs::GAM;
    const float* const sS = gates + GateVecs::S;
    const float* const rS = gates + GateVecs::R;
    half_t* const tbtg = reinterpret_cast<half_t*>(pairs + PairTiles::TBTG);
    half_t* const mimg = reinterpret_cast<half_t*>(pairs + PairTiles::M);
    half_t* const pimg = reinterpret_cast<half_t*>(pairs + PairTiles::P);
    half8 ka[SS], qf[SS];
#pragma unroll
    for (int s = 0; s < SS; ++s) {
        ka[s] = row_operand<D>(Kt, ab, s, m, g4);
        qf[s] = row_operand<D>(Qt, ia, s, m, g4);
    }
    // diagonal block, gates and betas (see gdn_fused_kernel.h for each of the steps)
    const f32x4 gi = *reinterpret_cast<const f32x4*>(gS + 16 * ab + 4 * g4);
    const f32x4 bi = *reinterpret_cast<const f32x4*>(bS + 16 * ab + 4 * g4);
    const float gj = gS[16 * ab + m], bj = bS[16 * ab + m];
    f32x4 gr = {0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < SS; ++s) gr = mma32(ka[s], ka[s], gr);
    f32x4 d, dt, y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4 * g4 + e;
        float x = bi[e] * EL::exp_(fminf(gi[e] - gj, 0.f)) * gr[e];     // D[i][m]
        float xt = bj * EL::exp_(fminf(gj - gi[e], 0.f)) * gr[e];       // D[m][i]
        pin(x); pin(xt);       // in every lane: no branch around an exponential
        d[e] = m < i ? x : 0.f;
        dt[e] = i < m ? xt : 0.f;
        y[e] = (i == m ? 1.f : 0.f) - d[e];
    }
    // The diagonal inverse (the products of inv16_tiles), between them the other blocks' raw products
    f32x4 acl[4], acp[4];
    auto block = [&](int c) {
        half8 kc[SS];
#pragma unroll
        for (int s = 0; s < SS; ++s) kc[s] = row_operand<D>(Kt, c, s, m, g4);
        if (c < ab) {
            acl[c] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < SS; ++s) acl[c] = mma32(ka[s], kc[s], acl[c]);   // rows i in block ab, lanes j in block c
        }
        if (c <= ia) {
            acp[c] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < SS; ++s) acp[c] = mma32(kc[s], qf[s], acp[c]);
        }
    };
    const f32x4 zero = {0, 0, 0, 0};
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 p2 = mm16_rr(zero, dt, d), p2t = mm16_rr(zero, d, dt);
    block(0);
    __builtin_amdgcn_sched_barrier(0);
    y = mm16_rr(y, p2t, y);
    const f32x4 p4 = mm16_rr(zero, p2t, p2), p4t = mm16_rr(zero, p2, p2t);
    block(1);
    __builtin_amdgcn_sched_barrier(0);
    y = mm16_rr(y, p4t, y);
    const f32x4 p8t = mm16_rr(zero, p4, p4t);
    if (ab > 2 || ia >= 2) block(2);
    __builtin_amdgcn_sched_barrier(0);
    y = mm16_rr(y, p8t, y);
    if (ia >= 3) block(3);
    // a pair tile is written whole, 16 bytes a lane in order (its two blocks one by one, 8 bytes at a stride of 16, are two-way conflicts:
    // 1024 chains of up to 345 chunks 1819 -> 1794 us, 8192 chains 4159 -> 4135)
    auto put = [&](half_t* img, int tile, const half4& lo, const half4& hi) {
        *reinterpret_cast<half8*>(img + (tile * 16 + m) * LD + 8 * g4) = cat8(lo, hi);
    };
    const half4 none = {(half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f};
    half4 even = none;
    const float gq = gS[16 * ia + m];
#pragma unroll
    for (int c = 0; c <= ia; ++c) {
        f32x4 p;
        if (c < ia) {
            const float pr = scale * rS[c * 64 + 16 * ia + m];
            const f32x4 sk = *reinterpret_cast<const f32x4*>(sS + 16 * c + 4 * g4);
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = pr * (sk[e] * acp[c][e]);
        } else {
            const f32x4 gk = *reinterpret_cast<const f32x4*>(gS + 16 * c + 4 * g4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float val = scale * EL::exp_(fminf(gq - gk[e], 0.f)) * acp[c][e];
                pin(val);
                p[e] = (4 * g4 + e <= m) ? val : 0.f;
            }
        }
        const half4 h = cvt4(p);
        if (c & 1) put(pimg, PairTiles::p_pair(ia, c), even, h);
        else if (c == ia) put(pimg, PairTiles::p_pair(ia, c), h, none);
        else even = h;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) Tf[(4 * g4 + e) * TF_LD + m] = y[e];
    const f32x4 at = *reinterpret_cast<const f32x4*>(Tf + m * TF_LD + 4 * g4);   // T[m][4 g4 + e]
    {
        const f32x4 gm = *reinterpret_cast<const f32x4*>(gamS + 16 * ab + 4 * g4);
        f32x4 tb, tgm;
#pragma unroll
        for (int e = 0; e < 4; ++e) { tb[e] = at[e] * bi[e]; tgm[e] = -tb[e] * gm[e]; }
        *reinterpret_cast<half8*>(tbtg + (ab * 16 + m) * LD + 8 * g4) = cat8(cvt4(tb), cvt4(tgm));
    }
#pragma unroll
    for (int c = 0; c < ab; ++c) {
        const float sj = sS[16 * c + m];
        const f32x4 ri = *reinterpret_cast<const f32x4*>(rS + c * 64 + 16 * ab + 4 * g4);
        f32x4 lt;
#pragma unroll
        for (int e = 0; e < 4; ++e) lt[e] = (bi[e] * ri[e]) * (sj * acl[c][e]);   // L_ac[4 g4 + e][m]
        const f32x4 mt_ = mm16_rr(zero, lt, at);     // (L^T T^T): element e of lane (m, g4) = (T L)[m][4 g4 + e]
        f32x4 neg;
#pragma unroll
        for (int e = 0; e < 4; ++e) neg[e] = -mt_[e];
        const half4 h = cvt4(neg);
        if (c & 1) put(mimg, PairTiles::m_pair(ab, c), even, h);
        else if (c == ab - 1) put(mimg, PairTiles::m_pair(ab, c), h, none);
        else even = h;
    }
}

// Substitution and outputs of one recurrence wave, NT 16-column tiles of d_v: u from the pair tiles, K, Q, V and the state
// (accS: tile (mt = 2 s + h, nt), element e of lane (m, g4) is S[16 nt + m][32 s + 8 g4 + 4 h + e]), o rows through a descriptor over
// o_bytes from o (the wave's first column of the chunk's first row).  Vt: [64][VD], the wave's columns from piece v_piece on.
// ud: diag(dec) U, as the operand of the state update over the tokens of block pair p.
template <bool O_BF16, int D, int NT, int VD, bool AHEAD>
__device__ __forceinline__ void substitute(const char* Kt, const char* Qt, const char* Vt, int v_piece, const char* pairs, const float* gamS,
                           const float* decS, const f32x4 (&accS)[D / 16][NT], half8 (&ud)[2][NT], const char* o, int o_bytes,
                           int o_step, float scale, int lane) {
    constexpr int SS = D / 32, LD = PairTiles::LD;
    const int m = lane & 15, g4 = lane >> 4, trow = 4 * g4 + (m >> 2);
    const half_t* const tbtg = reinterpret_cast<const half_t*>(pairs + PairTiles::TBTG);
    const half_t* const mimg = reinterpret_cast<const half_t*>(pairs + PairTiles::M);
    const half_t* const pimg = reinterpret_cast<const half_t*>(pairs + PairTiles::P);
    int tv[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
        tv[nt] = trow * 2 * VD + 16 * ((v_piece + 2 * nt + ((m & 3) >> 1)) ^ swz<VD>(trow)) + 8 * (m & 1);   // + tok0 * 2 VD
    half8 sf[SS][NT];        // the state as an operand over d_k: step s = state tiles 2 s, 2 s + 1
#pragma unroll
    for (int s = 0; s < SS; ++s)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) sf[s][nt] = cat8(cvt4(accS[2 * s][nt]), cvt4(accS[2 * s + 1][nt]));
    half8 uh[2][NT];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 8; ++e) uh[p][nt][e] = (half_t)0.f;
    constexpr int OB = O_BF16 ? 2 : 4;
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(o), 0, o_bytes, 0x00020000);
    const int o_lane = m * o_step + 4 * g4 * OB;
    // LDS operands.  AHEAD: read one to two block rows ahead of the products that take them and pinned there, so that a wave alone
    // on its SIMD does not stand in every read's latency; otherwise read where they are used.
    half8 kr[2][SS], qr[2][SS];                  // K and Q rows of two block rows
    half8 tfs[4], mfs[4], pfs[6];
    half4 vts[4][NT];
    auto read_rows = [&](int ab) {
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            kr[ab & 1][s] = row_operand<D>(Kt, ab, s, m, g4);
            qr[ab & 1][s] = row_operand<D>(Qt, ab, s, m, g4);
        }
    };
    auto pair_operand = [&](const half_t* img, int tile) -> half8 { return *reinterpret_cast<const half8*>(img + (tile * 16 + m) * LD + 8 * g4); };
    auto read_pairs = [&](int ab) {              // what block row ab takes of the pair tiles and of V
        tfs[ab] = pair_operand(tbtg, ab);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) vts[ab][nt] = tr_read(Vt + tv[nt] + ab * 16 * 2 * VD);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (2 * p < ab) mfs[PairTiles::m_pair(ab, 2 * p)] = pair_operand(mimg, PairTiles::m_pair(ab, 2 * p));
            if (2 * p <= ab) pfs[PairTiles::p_pair(ab, 2 * p)] = pair_operand(pimg, PairTiles::p_pair(ab, 2 * p));
        }
    };
    // K_a S0^T (tokens in registers) and (Q_a S0^T)^T (d_v in registers, lane = token): 8 NT independent products for every step
    auto state_products = [&](int ab, f32x4 (&ks)[NT], f32x4 (&ot)[NT]) {
        if (!AHEAD) read_rows(ab);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) { ks[nt] = f32x4{0, 0, 0, 0}; ot[nt] = f32x4{0, 0, 0, 0}; }
#pragma unroll
        for (int s = 0; s < SS; ++s)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                ks[nt] = mma32(kr[ab & 1][s], sf[s][nt], ks[nt]);
                ot[nt] = mma32(sf[s][nt], qr[ab & 1][s], ot[nt]);
            }
    };
    f32x4 ks_n[NT], ot_n[NT];
    if (AHEAD) {
        read_rows(0);
        read_pairs(0);
        read_rows(1);
        read_pairs(1);
        __builtin_amdgcn_sched_barrier(0);
    }
    state_products(0, ks_n, ot_n);
#pragma unroll
    for (int ab = 0; ab < 4; ++ab) {
        const int row = 16 * ab + m;
        f32x4 ks[NT], ot[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) { ks[nt] = ks_n[nt]; ot[nt] = ot_n[nt]; }
        if (AHEAD && ab < 2) {
            __builtin_amdgcn_sched_barrier(0);
            read_rows(ab + 2);
            read_pairs(ab + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!AHEAD) read_pairs(ab);
        if (ab < 3) state_products(ab + 1, ks_n, ot_n);
        const half8 tf = tfs[ab];
        f32x4 u[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const f32x4 zero = {0, 0, 0, 0};
            u[nt] = mma32(tf, cat8(vts[ab][nt], cvt4(ks[nt])), zero);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
            if (2 * p < ab) {
                const half8 mf = mfs[PairTiles::m_pair(ab, 2 * p)];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) u[nt] = mma32(mf, uh[p][nt], u[nt]);
            }
        const f32x4 dc = *reinterpret_cast<const f32x4*>(decS + 16 * ab + 4 * g4);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const half4 h = cvt4(u[nt]);
            f32x4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = u[nt][e] * dc[e];
            const half4 hd = cvt4(x);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uh[ab >> 1][nt][4 * (ab & 1) + e] = h[e];
                ud[ab >> 1][nt][4 * (ab & 1) + e] = hd[e];
            }
        }
        const float gm = gamS[row] * scale;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 4; ++e) ot[nt][e] *= gm;
#pragma unroll
        for (int p = 0; p < 2; ++p)
            if (2 * p <= ab) {
                const half8 pf = pfs[PairTiles::p_pair(ab, 2 * p)];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) ot[nt] = mma32(uh[p][nt], pf, ot[nt]);
            }
        if (O_BF16) {
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, __builtin_convertvector(ot[nt], bf16x4)), ro,
                                                      o_lane + ab * 16 * o_step + 32 * nt, 0, 0);
        } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, ot[nt]), ro, o_lane + ab * 16 * o_step + 64 * nt, 0, 0);
        }
    }
}

// S^T = gam_last S^T + sum_j K^T[.][j] ud[j][.], two token blocks per product
template <int D, int NT>
__device__ __forceinline__ void update_state(const char* Kt, float gam_last, const half8 (&ud)[2][NT], f32x4 (&accS)[D / 16][NT], int lane) {
    constexpr int SS = D / 32;
    const int m = lane & 15, g4 = lane >> 4, trow = 4 * g4 + (m >> 2);
    int tr_b[SS];
#pragma unroll
    for (int s = 0; s < SS; ++s) tr_b[s] = trow * (2 * D) + 16 * ((4 * s + (m & 3)) ^ swz<D>(trow));   // + tok0 * (2 * D) + 8 h
                #pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) {
        const char* kt = Kt + tr_b[mt >> 1] + 8 * (mt & 1);
        const half8 k0 = cat8(tr_read(kt), tr_read(kt + 16 * (2 * D)));
        const half8 k1 = cat8(tr_read(kt + 32 * (2 * D)), tr_read(kt + 48 * (2 * D)));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int e = 0; e < 4; ++e) accS[mt][nt][e] *= gam_last;
            accS[mt][nt] = mma32(k0, ud[0][nt], accS[mt][nt]);
            accS[mt][nt] = mma32(k1, ud[1][nt], accS[mt][nt]);
        }
    }
}

}  // namespace gdn
