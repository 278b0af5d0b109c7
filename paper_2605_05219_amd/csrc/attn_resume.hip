// attn_resume: host side of the attention layers' part of a cache hit (see include/attn_resume.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "attn_kernel.h"
#include "attn_resume.h"
#include "gdn_host.h"

namespace attn {
namespace {

inline int32_t hip_err(hipError_t e) { return e == hipSuccess ? GDN_OK : GDN_ERR_HIP - (int32_t)e; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int32_t check_shape(const attn_shape* s) {
    if (!s) return GDN_ERR_NULL;
    if (s->H_q <= 0 || s->H_kv <= 0 || s->H_q % s->H_kv != 0) return GDN_ERR_SHAPE;
    if (s->d != 64 && s->d != 128 && s->d != 256) return GDN_ERR_SHAPE;
    if (s->o_dtype != GDN_F32 && s->o_dtype != GDN_BF16) return GDN_ERR_SHAPE;
    if (!(s->scale > 0.f) || !std::isfinite(s->scale)) return GDN_ERR_SHAPE;
    return GDN_OK;
}

// geometry of a pool of sequence slots
int32_t check_pool(const attn_shape* s, int64_t slot_stride, int32_t n_slots, int32_t cap) {
    if (n_slots < 0 || cap < 0) return GDN_ERR_COUNT;
    if (slot_stride < 0 || slot_stride % 8 != 0) return GDN_ERR_ALIGN;
    if (slot_stride < (int64_t)cap * s->H_kv * s->d) return GDN_ERR_SHAPE;   // slots would overlap
    // a slot is addressed with 32-bit byte offsets, which may run up to two key tiles past its last row
    if (((int64_t)cap + 128) * s->H_kv * s->d * 2 > INT32_MAX) return GDN_ERR_SHAPE;
    return GDN_OK;
}

int32_t check_slots(const int32_t* ids, int32_t n, int32_t n_slots, bool skip_empty, const int32_t* len) {
    std::vector<int32_t> seen;
    seen.reserve(n);
    for (int32_t r = 0; r < n; ++r) {
        if (ids[r] < 0 || ids[r] >= n_slots) return GDN_ERR_SLOT_RANGE;
        if (skip_empty && len[r] == 0) continue;
        seen.push_back(ids[r]);
    }
    std::sort(seen.begin(), seen.end());
    if (std::adjacent_find(seen.begin(), seen.end()) != seen.end()) return GDN_ERR_SLOT_DUP;
    return GDN_OK;
}

// Splitting the key walk: calls with fewer than SPLIT_BELOW workgroups cut the walks of their pieces
// into parts of at least SPLIT_MIN_KEYS keys (whole tiles), aiming at SPLIT_BELOW workgroups in all; the
// partial results of at most SPLIT_MAX_WGS (part, head) pairs live in the workspace.  (A few-rows request's has NAR_ROWS rows
// there instead of ATT_BQ.)
constexpr int SPLIT_BELOW = 512;       // two workgroups per compute unit
constexpr int SPLIT_MIN_KEYS = 512;
constexpr int SPLIT_MAX_WGS = 768;
// The few-rows kernel's walks are cut into at most NARROW_WGS workgroups in all: two per compute unit, one round, at d = 64 and
// 128 (64 one-token requests behind 4 to 10 thousand keys, d = 128: at most 256 / 384 / 512 / 640 / 768 / 1024 workgroups 104 / 109 /
// 91 / 98 / 90 / 107 us; four such requests 24 / 24 / 20 / 20 / 20 / 20 us).  At d = 256 one workgroup fills a compute unit's LDS and
// they run in two rounds; other limits were measured at d = 128 only.
constexpr int NARROW_WGS = 512;

// ints of the uploaded index arrays: cu (n_req+1), start, slot (n_req each), five per unit of the 128-row kernel, eight per unit
// of the few-rows kernel, four per split piece
// (with packed rows a piece is 128 / G tokens, G the heads per key/value head: at most G times as many pieces)
constexpr int WIDE_INTS = 5, UNIT_INTS = NAR_REC;
static_assert(WIDE_INTS <= UNIT_INTS && NARROW_WGS <= SPLIT_MAX_WGS, "plan_ints and the partial results hold either kernel's units");
inline int64_t max_items(int32_t n_req, int64_t T, int G) { return T * G / ATT_BQ + n_req; }
inline int64_t max_units(int32_t n_req, int64_t T, int G) { return max_items(n_req, T, G) + SPLIT_MAX_WGS; }
inline int64_t plan_ints(int32_t n_req, int64_t T, int G) {
    return 3 * (int64_t)n_req + 1 + NAR_REC + UNIT_INTS * max_units(n_req, T, G) + 4 * max_items(n_req, T, G);
}
inline int64_t plan_bytes(int32_t n_req, int64_t T, int G) {
    return (plan_ints(n_req, T, G) * (int64_t)sizeof(int32_t) + 255) / 256 * 256;
}
inline int64_t part_ml_bytes() { return (int64_t)SPLIT_MAX_WGS * ATT_BQ * 2 * sizeof(float); }
inline int64_t part_o_bytes(int d) { return (int64_t)SPLIT_MAX_WGS * ATT_BQ * d * sizeof(float); }

template <int D, typename OT, int NH>
hipError_t launch_attn(const AttnArgs& a, unsigned blocks, hipStream_t stream) {
    hipLaunchKernelGGL((attn_suffix_kernel<D, OT, NH>), dim3(blocks), dim3(ATT_THREADS * NH), 0, stream, a);
    return hipGetLastError();
}

// NH: head blocks per workgroup; 2 is built for d = 128 only
template <typename OT>
hipError_t launch_attn_d(int d, int NH, const AttnArgs& a, unsigned blocks, hipStream_t stream) {
    if (NH != 1 && d != 128) return hipErrorInvalidValue;
    switch (d) {
        case 64: return launch_attn<64, OT, 1>(a, blocks, stream);
        case 128: return NH == 2 ? launch_attn<128, OT, 2>(a, blocks, stream) : launch_attn<128, OT, 1>(a, blocks, stream);
        default: return launch_attn<256, OT, 1>(a, blocks, stream);
    }
}

template <int D, typename OT, bool NT>
hipError_t launch_narrow(const AttnArgs& a, const AppendArgs& ap, unsigned blocks, hipStream_t stream) {
    hipLaunchKernelGGL((attn_narrow_kernel<D, OT, NT>), dim3(blocks), dim3(ATT_THREADS), 0, stream, a, ap);
    return hipGetLastError();
}

template <typename OT, bool NT>
hipError_t launch_narrow_d(int d, const AttnArgs& a, const AppendArgs& ap, unsigned blocks, hipStream_t stream) {
    switch (d) {
        case 64: return launch_narrow<64, OT, NT>(a, ap, blocks, stream);
        case 128: return launch_narrow<128, OT, NT>(a, ap, blocks, stream);
        default: return launch_narrow<256, OT, NT>(a, ap, blocks, stream);
    }
}

template <typename OT>
hipError_t launch_combine_d(int d, const CombineArgs& a, hipStream_t stream) {
    const dim3 grid((unsigned)(a.set[0].blocks + a.set[1].blocks)), block(ATT_THREADS);
    switch (d) {
        case 64: hipLaunchKernelGGL((attn_combine_kernel<64, OT>), grid, block, 0, stream, a); break;
        case 128: hipLaunchKernelGGL((attn_combine_kernel<128, OT>), grid, block, 0, stream, a); break;
        default: hipLaunchKernelGGL((attn_combine_kernel<256, OT>), grid, block, 0, stream, a); break;
    }
    return hipGetLastError();
}

// The work of one attn_suffix_prefill call (host, integer): how the rows of a workgroup are made up, the pieces
// (row tiles of a request), the cut of long key walks into parts, and the units (whole walks or parts) in launch order.
std::atomic<int32_t> g_allow_split{1}, g_allow_pack{1};   // attn_tune_split / attn_tune_pack
std::atomic<int32_t> g_pairs{1};                           // attn_tune_pairs: 0 never, 1 per call, 2 wherever they are built
struct Unit { int32_t req, tile, t0, t1, part; bool few; };      // part: slot among those of its kind of request, or -1
struct Piece { int32_t req, tile, n_tiles, parts, base; };       // base: first slot
struct UnitPlan {
    int pack = 1;                     // 128-row kernel: query heads per token in a workgroup's rows: 1, or H_q / H_kv
    bool apart = false;               // the few-rows requests are walked by the few-rows kernel
    std::vector<char> few;            // per request
    std::vector<Unit> units;          // of both kernels, those with the most key tiles first
    // of the other requests, of the few-rows requests
    int32_t longest[2] = {0, 0};      // longest suffix
    int64_t n_units[2] = {0, 0};
    std::vector<Piece> split[2];      // the split pieces and their workspace slots
    int32_t n_slots[2] = {0, 0};
};

// The requests the few-rows kernel is for: at most 16 rows, and a walk long enough for the split below (shorter walks stay
// whole and on the 128-row kernel, where a row's result does not depend on the suffix around it either).  Measured, whole call,
// 64 one-token requests of 8 heads per key/value head behind 4 to 10 thousand keys, 128-row kernel against this one: d = 64 57
// against 52 us, d = 128 131 against 91 (465 MB read: 73 us at the rate of a plain copy), d = 256 235 against 168; d = 128, four of
// them 34 against 22, one 31 against 20.
inline bool few_rows(int32_t len, int32_t start, int G) {
    return len > 0 && ATT_BQ % G == 0 && (int64_t)len * G <= NAR_ROWS && start + len >= 2 * SPLIT_MIN_KEYS;
}

// Rows of a workgroup of the 128-row kernel: 128 tokens of one query head (1), or, where that would leave too many of all
// rows empty (short suffixes), 128 / G tokens of the G heads of a key/value group (G).  Too many: a fifth.  In calls of many rounds of
// workgroups fewer will do, down to 7 in a hundred at G >= 8 and 9.5 below (64 suffixes of 200 to 1000 tokens behind 3000 to 5000, G = 8, 0.926 of the
// rows, 1572 -> 1530 us, at d = 64 891 -> 861; at G = 4 and 0.915 to 0.926 of them 0.93 to 1.13 of the time, 1.00 on average), if the
// key tiles this saves weigh more than the plan it costs: G times the units, some 25 ns each to list, sort and send.  (64 suffixes of 110 to 440
// behind 64 to 128, G = 8, d = 64, 0.834 of the rows but 1108 units for 166: 54 -> 66 us; of 250 to 500 behind 3000 to 6000, d = 256, 0.868 of them
// 2061 -> 1871.  Over 530 calls of G = 4 and 8 that are less than a fifth empty this rule is 0.5 % from the better form on average, 6 % at worst; packing all of
// them 0.7 and 17 %, and 1.3 % where each call is waited for before the next; packing none 2.9 %.)
// In smaller calls the cut of the walks and the last round decide (d = 256, one suffix of 430 to 860 tokens 57 / 77, three 111 / 101).
int pick_pack(const attn_shape& s, int32_t n_req, const int32_t* len, const int32_t* start_pos, const std::vector<char>& elsewhere) {
    const int G = s.H_q / s.H_kv;
    if (G == 1 || ATT_BQ % G != 0 || g_allow_pack.load() == 0) return 1;
    const int KT = att_kt(s.d);
    int64_t units[2] = {0, 0};           // plain, packed
    double tiles[2] = {0.0, 0.0};        // key tiles of one head block's workgroups
    for (int32_t r = 0; r < n_req; ++r) {
        if (elsewhere[r]) continue;
        for (int k = 0; k < 2; ++k) {
            const int TPW = k ? ATT_BQ / G : ATT_BQ;
            const int64_t n = (len[r] + TPW - 1) / TPW;
            units[k] += n;
            tiles[k] += (double)n * (0.5 + ((double)start_pos[r] + 0.5 * (len[r] + TPW)) / KT);
        }
    }
    const int64_t rows_plain = units[0] * s.H_q, rows_packed = units[1] * s.H_kv;      // (in workgroups: 128 rows each)
    if (rows_packed * 100 <= rows_plain * 80) return G;
    if (rows_packed < 4 * SPLIT_BELOW || rows_packed * 1000 > rows_plain * (G >= 8 ? 930 : 905)) return 1;
    const double tile_ns = s.d == 64 ? 2.2 : 3.9, plain_ns = tile_ns * tiles[0] * s.H_q, packed_ns = tile_ns * tiles[1] * s.H_kv;   // a workgroup's tile, the chip full
    return plain_ns - packed_ns >= 25.0 * (double)(units[1] - units[0]) ? G : 1;
}

// Which kernel walks the few-rows requests.  What is in a call beside such a request must not change the bits of its whole walk,
// so it is walked whole by the few-rows kernel only.  A call of nothing else takes that kernel.  A mixed call either takes both
// kernels, one launch behind the other, or stays one launch of the 128-row kernel, which then cuts these walks into two parts at
// least.  One launch is better where the call is small enough for split walks anyway (d = 128, both against one launch: 1 decode
// row and 64 tokens 33 against 24 us, 32 decode rows and 32 short contexts 42 against 33), and where the other requests fill the
// chip by themselves, so that the decode rows' reads hide under their products (64 decode rows and 8 suffixes of 200 to 1000
// tokens 356 against 293, 32 and 32 886 against 791); between them, both (63 decode rows and 512 tokens behind 7680 keys 127 against
// 139 us, 32 and four of 512 tokens 88 against 104, 128 decode rows and 128 short contexts 92 against 103).
void pick_kernels(const attn_shape& s, int32_t n_req, const int32_t* len, const int32_t* start_pos, UnitPlan& out) {
    const int G = s.H_q / s.H_kv;
    const bool allowed = g_allow_pack.load() != 0 && g_allow_split.load() != 0;
    int64_t n_few = 0, n_live = 0;
    out.few.assign(n_req, 0);
    for (int32_t r = 0; r < n_req; ++r) {
        out.few[r] = allowed && few_rows(len[r], start_pos[r], G);
        out.longest[out.few[r]] = std::max(out.longest[out.few[r]], len[r]);
        n_few += out.few[r];
        n_live += len[r] > 0;
    }
    out.pack = pick_pack(s, n_req, len, start_pos, std::vector<char>(n_req, 0));
    if (n_few == 0) return;
    const int TPW = ATT_BQ / out.pack, HB = s.H_q / out.pack;
    int64_t others = 0;
    for (int32_t r = 0; r < n_req; ++r)
        if (!out.few[r]) others += (len[r] + TPW - 1) / TPW;
    const bool one_launch = n_few < n_live && ((others + n_few) * HB < SPLIT_BELOW || others * HB >= SPLIT_BELOW);
    const bool room = 2 * n_few * HB * NAR_ROWS <= SPLIT_MAX_WGS * ATT_BQ && 2 * n_few * WIDE_INTS <= UNIT_INTS * SPLIT_MAX_WGS;   // two parts each
    out.apart = !(one_launch && room);
    if (out.apart) out.pack = pick_pack(s, n_req, len, start_pos, out.few);
}

void build_units(const attn_shape& sh, int32_t n_req, const int32_t* len, const int32_t* start_pos, UnitPlan& out) {
    const attn_shape* s = &sh;
    const int KT = att_kt(s->d);
    pick_kernels(sh, n_req, len, start_pos, out);
    const int pack = out.pack;
    const int HB[2] = {s->H_q / pack, out.apart ? s->H_kv : s->H_q / pack};   // head blocks (workgroups) per unit
    // ---- pieces: one per workgroup of suffix tokens of a request (one in all of a few-rows request)
    std::vector<Piece> pieces[2];
    int64_t wide_items = 0, wide_tiles = 0;       // of the 128-row kernel's walks
    for (int32_t r = 0; r < n_req; ++r) {
        const int k = out.few[r], TPW = k ? NAR_ROWS : ATT_BQ / pack;
        for (int32_t t = 0; t * TPW < len[r]; ++t) {
            const int32_t kv = start_pos[r] + std::min((t + 1) * TPW, len[r]);
            pieces[k].push_back({r, t, (kv + KT - 1) / KT, 1, 0});
            if (k && out.apart) continue;
            ++wide_items;
            wide_tiles += pieces[k].back().n_tiles;
        }
    }
    // ---- too few workgroups for the chip: cut long key walks into parts
    int64_t parts[2] = {0, 0};                    // of split walks
    auto cut = [&](int k, auto&& parts_of) {
        parts[k] = 0;
        for (Piece& p : pieces[k]) {
            p.parts = (int32_t)parts_of((int64_t)p.n_tiles);
            if (p.parts > 1) parts[k] += p.parts;
        }
    };
    if (out.apart) {
        auto count = [&](int64_t tp) {
            int64_t n = 0;
            for (const Piece& p : pieces[1]) n += (p.n_tiles + tp - 1) / tp;
            return n * HB[1];
        };
        int64_t lo = SPLIT_MIN_KEYS / KT, hi = lo;
        for (const Piece& p : pieces[1]) hi = std::max<int64_t>(hi, p.n_tiles);
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if (count(mid) <= NARROW_WGS) hi = mid; else lo = mid + 1;
        }
        cut(1, [&](int64_t n) { return (n + lo - 1) / lo; });    // (more requests than workgroups: lo is the longest walk)
    } else {
        cut(1, [](int64_t) { return 2; });
    }
    if (wide_items * HB[0] < SPLIT_BELOW && g_allow_split.load() != 0) {
        int64_t tp = std::max<int64_t>(SPLIT_MIN_KEYS / KT, (wide_tiles * HB[0] + SPLIT_BELOW - 1) / SPLIT_BELOW);
        for (;; tp *= 2) {
            cut(0, [&](int64_t n) { return n >= 2 * tp ? (n + tp - 1) / tp : 1; });
            if (!out.apart) cut(1, [&](int64_t n) { return n >= 2 * tp ? (n + tp - 1) / tp : 2; });
            // all partial results fit their part of the workspace, and all unit indexes theirs (plan_ints; with one key/value
            // head and few heads to a group the second can be the tighter one)
            if (parts[0] * HB[0] * ATT_BQ + parts[1] * HB[1] * NAR_ROWS <= (int64_t)SPLIT_MAX_WGS * ATT_BQ &&
                WIDE_INTS * parts[0] + (out.apart ? NAR_REC : WIDE_INTS) * parts[1] <= (int64_t)UNIT_INTS * SPLIT_MAX_WGS)
                break;
        }
    }
    // ---- units: a whole walk or one part of it; those with the most key tiles first
    for (int k = 0; k < 2; ++k) {
        for (Piece& p : pieces[k]) {
            if (p.parts == 1) {
                out.units.push_back({p.req, p.tile, 0, p.n_tiles, -1, k == 1});
                continue;
            }
            p.base = out.n_slots[k];
            out.split[k].push_back(p);
            const int32_t per = (p.n_tiles + p.parts - 1) / p.parts;
            for (int32_t j = 0; j < p.parts; ++j)
                out.units.push_back({p.req, p.tile, j * per, std::min((j + 1) * per, p.n_tiles), out.n_slots[k]++, k == 1});
        }
        out.n_units[k] = (int64_t)out.units.size() - (k ? out.n_units[0] : 0);
    }
    std::stable_sort(out.units.begin(), out.units.end(), [](const Unit& x, const Unit& y) { return x.t1 - x.t0 > y.t1 - y.t0; });
}

// Whether the workgroups of the 128-row kernel take two head blocks each (see attn_kernel.h), where that kernel is built: in calls of at most two rounds
// of such workgroups, one to a compute unit, whose walks are long enough and that balance over the chip as well as workgroups of half the size, two to one.
// Balance is estimated by the key tiles of the fullest place when the units, longest first, are dealt back and forth; a single-head workgroup that has a
// compute unit to itself goes through its tiles faster, so its side counts half way to the mean.  Single / pairs, 16 heads on 2, one suffix: 8192 tokens 303 /
// 280 us, 7936 288 / 265; 3000 68 / 79 and 4096 100 / 115 (unbalanced); 32 heads on 4, 4096 tokens 161 / 153.
// Walks: a pair starts when both its heads' first tiles have come and ends when both are done, which a short walk does not make up for.  Two rounds, by mean tiles of
// a walk: below 6 6 % slower on average (64 prompts of 128 tokens 37 / 42, behind 64 to 96 45 / 49), 6 to 16 4 %, 16 to 24 2 %, 28 to 34 even,
// 34 to 50 1.5 % faster, more 3 %; one round: below 12 2 % slower (512 tokens of 32 heads behind 2048 44 / 45), 16 2 % faster (512 of 16 behind 8000 58 / 57).
// Beyond two rounds it goes either way: 8320 tokens 310 / 292, behind 2048 441 / 460, behind 8000 894 / 941, 10240 437 / 451, 12288 620 / 623, 16384 1060 / 1029; five with
// 32 heads on 4 386 / 422, 29 of 915 to 1830 486 / 497, 16 of 900 to 1900 751 / 727; over 141 calls of more than 1024 workgroups between 0.94 and 1.19,
// 1.01 on average.  These keep one head.
inline bool pairs_pay(const UnitPlan& plan, int head_blocks) {
    std::vector<int32_t> tiles;
    int64_t sum = 0;
    for (const Unit& u : plan.units) {
        if (u.few && plan.apart) continue;
        tiles.push_back(u.t1 - u.t0);
        sum += u.t1 - u.t0;
    }
    constexpr int CUS = SPLIT_BELOW / 2;
    const int64_t wgs = (int64_t)tiles.size() * head_blocks;
    if (wgs > 4 * CUS || sum < (int64_t)tiles.size() * (wgs <= 2 * CUS ? 14 : 28)) return false;
    auto fullest = [&](int per_unit, int places) {
        std::vector<int32_t> load(places, 0);
        int j = 0, most = 0;
        for (int32_t n : tiles)
            for (int h = 0; h < per_unit; ++h, ++j) {
                int32_t& x = load[j / places % 2 ? places - 1 - j % places : j % places];
                x += n;
                most = std::max(most, (int)x);
            }
        return (double)most;
    };
    const double mean = (double)sum * head_blocks / (2 * CUS);
    return fullest(head_blocks / 2, CUS) <= 1.06 * 0.5 * (fullest(head_blocks, 2 * CUS) + mean);
}

// Head blocks per workgroup of the 128-row kernel.
inline int heads_per_workgroup(const attn_shape& s, const UnitPlan& plan) {
    const int mode = g_pairs.load();
    if (mode == 0 || s.d != 128 || s.H_q / s.H_kv / plan.pack % 2 != 0) return 1;
    return mode == 2 || pairs_pay(plan, s.H_q / plan.pack) ? 2 : 1;
}

// The requests of attn_plan and attn_plan_heads checked, and their suffix lengths.
int32_t plan_lengths(int32_t n_req, const int32_t* cu_seqlens, const int32_t* start_pos, std::vector<int32_t>& len) {
    len.resize(n_req);
    if (!cu_seqlens || !start_pos) return GDN_ERR_NULL;
    if (cu_seqlens[0] != 0) return GDN_ERR_SEQLENS;
    for (int32_t r = 0; r < n_req; ++r) {
        if (cu_seqlens[r + 1] < cu_seqlens[r]) return GDN_ERR_SEQLENS;
        len[r] = cu_seqlens[r + 1] - cu_seqlens[r];
        if (start_pos[r] < 0 || (int64_t)start_pos[r] + len[r] > INT32_MAX - 256) return GDN_ERR_START;
    }
    return GDN_OK;
}

}  // namespace
}  // namespace attn

using namespace attn;

extern "C" {

int64_t attn_workspace_bytes(const attn_shape* s, int32_t n_req, int64_t total_tokens) {
    const int32_t rc = check_shape(s);
    if (rc != GDN_OK) return rc;
    if (n_req < 0 || total_tokens < 0) return GDN_ERR_COUNT;
    return plan_bytes(n_req, total_tokens, s->H_q / s->H_kv) + part_ml_bytes() + part_o_bytes(s->d);
}

// shared by attn_kv_restore and attn_kv_spill: rows [0, n_rows[r]) of one pool's slot to the other's
static int32_t kv_tier_copy(const attn_shape* s, int32_t n_req, const int32_t* n_rows, void* host_k, void* host_v,
                            int64_t host_slot_stride, int32_t n_host_slots, const int32_t* host_slot, void* k_cache, void* v_cache,
                            int64_t slot_stride, int32_t n_slots, int32_t cap, const int32_t* seq_slot, bool to_device,
                            hipStream_t stream) {
    int32_t rc = check_shape(s);
    if (rc != GDN_OK) return rc;
    if (n_req < 0 || n_host_slots < 0) return GDN_ERR_COUNT;
    rc = check_pool(s, slot_stride, n_slots, cap);
    if (rc != GDN_OK) return rc;
    rc = check_pool(s, host_slot_stride, n_host_slots, cap);
    if (rc != GDN_OK) return rc;
    if (n_req == 0) return GDN_OK;
    if (!n_rows || !host_slot || !seq_slot) return GDN_ERR_NULL;
    int64_t total = 0;
    for (int32_t r = 0; r < n_req; ++r) {
        if (n_rows[r] < 0 || n_rows[r] > cap) return GDN_ERR_START;
        total += n_rows[r];
    }
    // the source slots only have to exist; the destination slots must also differ
    for (int32_t r = 0; r < n_req; ++r) {
        if (host_slot[r] < 0 || host_slot[r] >= n_host_slots) return GDN_ERR_SLOT_RANGE;
        if (seq_slot[r] < 0 || seq_slot[r] >= n_slots) return GDN_ERR_SLOT_RANGE;
    }
    rc = to_device ? check_slots(seq_slot, n_req, n_slots, false, nullptr) : check_slots(host_slot, n_req, n_host_slots, false, nullptr);
    if (rc != GDN_OK) return rc;
    if (total == 0) return GDN_OK;
    if (!host_k || !host_v || !k_cache || !v_cache) return GDN_ERR_NULL;
    if (!aligned16(k_cache) || !aligned16(v_cache)) return GDN_ERR_ALIGN;
    const int64_t row = (int64_t)s->H_kv * s->d;
    for (int32_t r = 0; r < n_req; ++r) {
        if (n_rows[r] == 0) continue;
        const size_t bytes = (size_t)n_rows[r] * row * sizeof(uint16_t);
        const int64_t ho = (int64_t)host_slot[r] * host_slot_stride, dv = (int64_t)seq_slot[r] * slot_stride;
        uint16_t* const hk = static_cast<uint16_t*>(host_k) + ho;
        uint16_t* const hv = static_cast<uint16_t*>(host_v) + ho;
        uint16_t* const dk = static_cast<uint16_t*>(k_cache) + dv;
        uint16_t* const dvp = static_cast<uint16_t*>(v_cache) + dv;
        hipError_t e = to_device ? hipMemcpyAsync(dk, hk, bytes, hipMemcpyHostToDevice, stream)
                                 : hipMemcpyAsync(hk, dk, bytes, hipMemcpyDeviceToHost, stream);
        if (e != hipSuccess) return hip_err(e);
        e = to_device ? hipMemcpyAsync(dvp, hv, bytes, hipMemcpyHostToDevice, stream)
                      : hipMemcpyAsync(hv, dvp, bytes, hipMemcpyDeviceToHost, stream);
        if (e != hipSuccess) return hip_err(e);
    }
    return GDN_OK;
}

int32_t attn_kv_restore(const attn_shape* s, int32_t n_req, const int32_t* prefix_len, const void* host_k, const void* host_v,
                        int64_t host_slot_stride, int32_t n_host_slots, const int32_t* host_slot, void* k_cache, void* v_cache,
                        int64_t slot_stride, int32_t n_slots, int32_t cap, const int32_t* seq_slot, void* stream) {
    return kv_tier_copy(s, n_req, prefix_len, const_cast<void*>(host_k), const_cast<void*>(host_v), host_slot_stride, n_host_slots,
                        host_slot, k_cache, v_cache, slot_stride, n_slots, cap, seq_slot, true, static_cast<hipStream_t>(stream));
}

int32_t attn_kv_spill(const attn_shape* s, int32_t n_req, const int32_t* n_rows, void* host_k, void* host_v,
                      int64_t host_slot_stride, int32_t n_host_slots, const int32_t* host_slot, const void* k_cache,
                      const void* v_cache, int64_t slot_stride, int32_t n_slots, int32_t cap, const int32_t* seq_slot, void* stream) {
    return kv_tier_copy(s, n_req, n_rows, host_k, host_v, host_slot_stride, n_host_slots, host_slot, const_cast<void*>(k_cache),
                        const_cast<void*>(v_cache), slot_stride, n_slots, cap, seq_slot, false, static_cast<hipStream_t>(stream));
}

int32_t attn_plan(const attn_shape* s, int32_t n_req, const int32_t* cu_seqlens, const int32_t* start_pos, int32_t capacity,
                  int32_t* unit_req, int32_t* unit_tile, int32_t* unit_t0, int32_t* unit_t1, int32_t* unit_part,
                  int32_t* n_units, int32_t* heads_per_row_group, int32_t* key_tile_rows) {
    int32_t rc = check_shape(s);
    if (rc != GDN_OK) return rc;
    if (n_req < 0 || capacity < 0) return GDN_ERR_COUNT;
    if (!n_units || !heads_per_row_group || !key_tile_rows) return GDN_ERR_NULL;
    *n_units = 0;
    *heads_per_row_group = 1;
    *key_tile_rows = att_kt(s->d);
    if (n_req == 0) return GDN_OK;
    std::vector<int32_t> len;
    rc = plan_lengths(n_req, cu_seqlens, start_pos, len);
    if (rc != GDN_OK) return rc;
    UnitPlan plan;
    build_units(*s, n_req, len.data(), start_pos, plan);
    *n_units = (int32_t)plan.units.size();
    *heads_per_row_group = plan.apart && plan.n_units[0] == 0 ? s->H_q / s->H_kv : plan.pack;
    if ((int64_t)plan.units.size() > capacity) return GDN_ERR_COUNT;
    if (!plan.units.empty() && (!unit_req || !unit_tile || !unit_t0 || !unit_t1 || !unit_part)) return GDN_ERR_NULL;
    for (size_t i = 0; i < plan.units.size(); ++i) {
        unit_req[i] = plan.units[i].req;
        unit_tile[i] = plan.units[i].tile;
        unit_t0[i] = plan.units[i].t0;
        unit_t1[i] = plan.units[i].t1;
        unit_part[i] = plan.units[i].part < 0 ? -1 : plan.units[i].part + (plan.units[i].few ? plan.n_slots[0] : 0);
    }
    return GDN_OK;
}

int32_t attn_plan_heads(const attn_shape* s, int32_t n_req, const int32_t* cu_seqlens, const int32_t* start_pos) {
    int32_t rc = check_shape(s);
    if (rc != GDN_OK) return rc;
    if (n_req < 0) return GDN_ERR_COUNT;
    if (n_req == 0) return 1;
    std::vector<int32_t> len;
    rc = plan_lengths(n_req, cu_seqlens, start_pos, len);
    if (rc != GDN_OK) return rc;
    UnitPlan plan;
    build_units(*s, n_req, len.data(), start_pos, plan);
    return heads_per_workgroup(*s, plan);
}

int32_t attn_suffix_prefill(const attn_shape* s, const void* q, const void* k_new, const void* v_new, const void* out_gate,
                            int32_t n_req, const int32_t* cu_seqlens, const int32_t* start_pos, void* k_cache, void* v_cache,
                            int64_t slot_stride, int32_t n_slots, int32_t cap, const int32_t* seq_slot, void* o, void* workspace,
                            int64_t workspace_bytes, void* stream_v) {
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    int32_t rc = check_shape(s);
    if (rc != GDN_OK) return rc;
    if (n_req < 0) return GDN_ERR_COUNT;
    rc = check_pool(s, slot_stride, n_slots, cap);
    if (rc != GDN_OK) return rc;
    if (n_req == 0) return GDN_OK;
    if (!cu_seqlens || !start_pos || !seq_slot) return GDN_ERR_NULL;
    if (cu_seqlens[0] != 0) return GDN_ERR_SEQLENS;
    std::vector<int32_t> len(n_req);
    for (int32_t r = 0; r < n_req; ++r) {
        if (cu_seqlens[r + 1] < cu_seqlens[r]) return GDN_ERR_SEQLENS;
        len[r] = cu_seqlens[r + 1] - cu_seqlens[r];
        if (start_pos[r] < 0 || (int64_t)start_pos[r] + len[r] > cap) return GDN_ERR_START;
    }
    rc = check_slots(seq_slot, n_req, n_slots, true, len.data());
    if (rc != GDN_OK) return rc;
    const int64_t T = cu_seqlens[n_req];
    if (T == 0) return GDN_OK;
    if (!q || !k_new || !v_new || !k_cache || !v_cache || !o) return GDN_ERR_NULL;
    if (!aligned16(q) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(o) ||
        !aligned16(out_gate))
        return GDN_ERR_ALIGN;
    if (!workspace || !aligned16(workspace) || workspace_bytes < attn_workspace_bytes(s, n_req, T)) return GDN_ERR_WORKSPACE;

    UnitPlan plan;
    build_units(*s, n_req, len.data(), start_pos, plan);
    const int G = s->H_q / s->H_kv;
    const int pack = plan.pack, HB = s->H_q / pack;
    const int NH = heads_per_workgroup(*s, plan);
    const int64_t n_narrow = plan.apart ? plan.n_units[1] : 0, n_wide = (int64_t)plan.units.size() - n_narrow;
    const bool xcd_split = 8 % s->H_kv == 0;
    int64_t blocks;
    if (xcd_split) {
        const int X = 8 / s->H_kv;
        blocks = 8 * ((n_wide * (G / pack / NH) + X - 1) / X);
    } else {
        blocks = n_wide * (HB / NH);
    }
    if (blocks > INT32_MAX || n_narrow * s->H_kv > INT32_MAX) return GDN_ERR_COUNT;

    // the uploaded image is packed to what this call uses (the workspace is sized for the most a call can need):
    // a copy of a few hundred bytes takes the runtime's short path, one of 16 KiB and more does not
    const int64_t rec_at = n_narrow > 0 ? (3 * (int64_t)n_req + 1 + NAR_REC - 1) / NAR_REC * NAR_REC : 3 * (int64_t)n_req + 1;   // records: aligned
    const int64_t unit_at = rec_at + NAR_REC * n_narrow;
    const int64_t piece_at[2] = {unit_at + WIDE_INTS * n_wide, unit_at + WIDE_INTS * n_wide + 4 * (int64_t)plan.split[0].size()};
    std::vector<int32_t> img((size_t)(piece_at[1] + 4 * (int64_t)plan.split[1].size()), 0);
    int32_t* p_cu = img.data();
    int32_t* p_start = p_cu + n_req + 1;
    int32_t* p_slot = p_start + n_req;
    int32_t* p_rec = p_cu + rec_at;            // records of the few-rows kernel's units
    int32_t* p_unit = p_cu + unit_at;          // five arrays of n_wide
    std::memcpy(p_cu, cu_seqlens, sizeof(int32_t) * (n_req + 1));
    for (int32_t r = 0; r < n_req; ++r) p_start[r] = plan.apart && plan.few[r] ? -1 : start_pos[r];
    std::memcpy(p_slot, seq_slot, sizeof(int32_t) * n_req);
    const int KT = att_kt(s->d);
    for (const Unit& u : plan.units) {
        if (u.few && plan.apart) {
            const int32_t kv = start_pos[u.req] + len[u.req];
            const int32_t rec[NAR_REC] = {cu_seqlens[u.req], len[u.req], start_pos[u.req], seq_slot[u.req], u.t0 * KT, std::min(u.t1 * KT, kv), u.part, 0};
            std::memcpy(p_rec, rec, sizeof rec);
            p_rec += NAR_REC;
            continue;
        }
        p_unit[0] = u.req;
        p_unit[n_wide] = u.tile;
        p_unit[2 * n_wide] = u.t0;
        p_unit[3 * n_wide] = u.t1;
        p_unit[4 * n_wide] = u.few && u.part >= 0 ? -2 - u.part : u.part;
        ++p_unit;
    }
    for (int k = 0; k < 2; ++k) {
        const int64_t n = (int64_t)plan.split[k].size();
        int32_t* p_piece = p_cu + piece_at[k];     // four arrays of n
        for (int64_t i = 0; i < n; ++i) {
            p_piece[i] = plan.split[k][i].req;
            p_piece[n + i] = plan.split[k][i].tile;
            p_piece[2 * n + i] = plan.split[k][i].base;
            p_piece[3 * n + i] = plan.split[k][i].parts;
        }
    }
    rc = gdn::upload_plan(img.data(), img.size() * sizeof(int32_t), workspace, stream);
    if (rc != GDN_OK) return rc;
    const int32_t* d = static_cast<const int32_t*>(workspace);

    AppendArgs ap;
    ap.k_new = static_cast<const uint16_t*>(k_new);
    ap.v_new = static_cast<const uint16_t*>(v_new);
    ap.k_cache = static_cast<uint16_t*>(k_cache);
    ap.v_cache = static_cast<uint16_t*>(v_cache);
    ap.cu = d;
    ap.start = d + n_req + 1;
    ap.slot = d + 2 * (int64_t)n_req + 1;
    ap.slot_stride = slot_stride;
    ap.row_chunks = s->H_kv * s->d / 8;
    ap.n_chunks = T * ap.row_chunks;
    ap.n_req = n_req;
    hipError_t e = hipSuccess;
    const int64_t ablocks = (ap.n_chunks + APPEND_THREADS - 1) / APPEND_THREADS;
    if (ablocks > INT32_MAX) return GDN_ERR_COUNT;
    if (n_wide > 0) {                          // (the few-rows kernel appends its own rows)
        hipLaunchKernelGGL(attn_append_kernel, dim3((unsigned)ablocks), dim3(APPEND_THREADS), 0, stream, ap);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_err(e);
    }

    AttnArgs a;
    a.q = static_cast<const uint16_t*>(q);
    a.gate = static_cast<const uint16_t*>(out_gate);
    a.k_cache = ap.k_cache;
    a.v_cache = ap.v_cache;
    a.o = o;
    a.cu = ap.cu;
    a.start = ap.start;
    a.slot = ap.slot;
    a.unit_rec = d + rec_at;
    a.unit_req = d + unit_at;
    a.unit_tile = a.unit_req + n_wide;
    a.unit_t0 = a.unit_req + 2 * n_wide;
    a.unit_t1 = a.unit_req + 3 * n_wide;
    a.unit_part = a.unit_req + 4 * n_wide;
    a.part_ml = reinterpret_cast<float*>(static_cast<char*>(workspace) + plan_bytes(n_req, T, G));
    a.part_o = reinterpret_cast<float*>(static_cast<char*>(workspace) + plan_bytes(n_req, T, G) + part_ml_bytes());
    a.few_row0 = (int64_t)plan.n_slots[0] * HB * ATT_BQ;
    a.slot_stride = slot_stride;
    a.n_units = (int32_t)n_wide;
    a.H_q = s->H_q;
    a.H_kv = s->H_kv;
    a.xcd_split = xcd_split ? 1 : 0;
    a.scale_log2e = s->scale * 1.4426950408889634f;
    if (n_narrow > 0) {
        // non-temporal reads where the launch reads more keys and values than the memory-side cache would hold for the next one
        // (465 MB 91 against 99 us with ordinary reads; 16 requests, 92 MB read again and again, 32 against 28)
        int64_t kv_rows = 0;
        for (int32_t r = 0; r < n_req; ++r)
            if (plan.few[r]) kv_rows += start_pos[r] + len[r];
        const unsigned nb = (unsigned)(n_narrow * s->H_kv);
        const bool nt = kv_rows * s->H_kv * s->d * 4 > ((int64_t)128 << 20);
        a.pack = G;
        e = s->o_dtype == GDN_F32 ? (nt ? launch_narrow_d<float, true>(s->d, a, ap, nb, stream) : launch_narrow_d<float, false>(s->d, a, ap, nb, stream))
                                  : (nt ? launch_narrow_d<uint16_t, true>(s->d, a, ap, nb, stream) : launch_narrow_d<uint16_t, false>(s->d, a, ap, nb, stream));
        if (e != hipSuccess) return hip_err(e);
    }
    if (n_wide > 0) {
        a.pack = pack;
        e = s->o_dtype == GDN_F32 ? launch_attn_d<float>(s->d, NH, a, (unsigned)blocks, stream)
                                  : launch_attn_d<uint16_t>(s->d, NH, a, (unsigned)blocks, stream);
        if (e != hipSuccess) return hip_err(e);
    }

    CombineArgs ca;
    ca.part_o = a.part_o;
    ca.part_ml = a.part_ml;
    ca.gate = a.gate;
    ca.o = o;
    ca.cu = a.cu;
    for (int k = 0; k < 2; ++k) {
        CombineSet& c = ca.set[k];
        const int64_t n = (int64_t)plan.split[k].size();
        c.piece_req = d + piece_at[k];
        c.piece_tile = c.piece_req + n;
        c.piece_base = c.piece_req + 2 * n;
        c.piece_parts = c.piece_req + 3 * n;
        c.row0 = k ? a.few_row0 : 0;
        c.slot_rows = k ? NAR_ROWS : ATT_BQ;
        c.pack = k && plan.apart ? G : pack;
        c.subs = (std::min(plan.longest[k], ATT_BQ / c.pack) * c.pack * (s->d / 4) + ATT_THREADS - 1) / ATT_THREADS;
        c.blocks = (int32_t)(n * (s->H_q / c.pack) * c.subs);
    }
    if (ca.set[0].blocks + ca.set[1].blocks == 0) return GDN_OK;
    ca.H_q = s->H_q;
    ca.scale_log2e = a.scale_log2e;
    e = s->o_dtype == GDN_F32 ? launch_combine_d<float>(s->d, ca, stream) : launch_combine_d<uint16_t>(s->d, ca, stream);
    return hip_err(e);
}

int32_t attn_tune_split(int32_t allow) { return g_allow_split.exchange(allow != 0); }

int32_t attn_tune_pack(int32_t allow) { return g_allow_pack.exchange(allow != 0); }

int32_t attn_tune_pairs(int32_t mode) { return g_pairs.exchange(mode == 0 || mode == 2 ? mode : 1); }

}  // extern "C"
