// k_plits.hip -- PLITS, the two-phase tabu search of Section 3.3 (Alg. 3),
// one wave64 per individual on gfx950.
//
// Conflict counts in factored form.  In the Latin square graph the neighbours
// of a cell are exactly the other cells of its row and of its column
// (Section 2.1), so the incremental evaluation table of Section 3.3,
// conf[v][k] = #neighbours of v coloured k, equals
//     rowcnt[r(v)][k] + colcnt[c(v)][k] - 2 [S(v) = k]
// with rowcnt/colcnt the number of vertices of each colour per row and per
// column.  These 2 n (n+1) byte counters replace the sum_v |D*(v)| table, live
// in LDS, and a move updates four of them instead of every neighbour's entry.
//
// Candidate rows.  The moves of vertex v are the colours of {0} u D*(v)
// (0: uncolour), kept ascending at cand[v][0 .. d] with d = |D*(v)|, TS
// positions per vertex; the tabu expiry of each move sits at the same
// position of tabu[v].  The rows are cut into chunks of CH consecutive
// positions; one lane evaluates one chunk.
//
// Two forms of an iteration.
//   Listed: the chunks of the eligible vertices V_0 u C(S) stay with their
//   lanes from one iteration to the next, one chunk per lane in up to
//   kPlitsSlots slots: vertex, row, column, colour and candidate colours in
//   registers, in no order (a move's id decides ties, not where it is found).
//   A move frees the lanes of the vertices that leave and gives the first free
//   lanes to those that join, about one each, so an iteration neither scans
//   for eligible vertices nor deals chunks nor loads candidates.  Conflict
//   counts and expiries are read afresh: keeping them with the chunks too
//   makes every move update all slots, which costs more than the reads.
//   Dealt: while the chunks do not fit (the first descent from an offspring,
//   mostly) and while iterations are idle beside vertices in conflict, they are
//   dealt to the lanes round by round from the eligibility bitmap, which both
//   forms keep.
//   Six slots hold the chunks in 97 % of the iterations at n = 50, half
//   prefilled (24 eligible vertices of 13 colours).  With four, 22 % of the
//   iterations at n = 70, 70 % (145 vertices of 6), and 34 % at n = 61, 65 %
//   were dealt: 2.93 -> 2.72 ns an iteration there, 5.58 -> 5.17 us; eight gain
//   no more and leave no registers over.
//
// Per wave (LDS): S[stride] colours, rowcnt|colcnt, the eligibility bitmap of
//   V_0 u C(S), tm8[|V|] (per vertex: whether this phase wrote its tabu row,
//   and its latest tabu expiry relative to a base advanced by 128 iterations
//   at a time, 255 = "treat as live"; a vertex not live has no tabu move),
//   the colour halves of the iteration's tie values; for the dealt form the
//   eligible vertices being dealt, a ring of chunk descriptors and bit planes
//   of the vertices' chunk counts.
// Per individual (HBM): tabu[|V|][TS] "allowed from" iteration of every move,
//   read only for vertices with a live entry; all zero between phases (each
//   phase clears the rows it wrote).
//
// One iteration:
//   1. the chunks (listed, or dealt from the bitmap): move value from the
//      row/column counts, admissibility from tabu and aspiration, best key per
//      lane: (value, tie value) above the move id (v, k), the tie value being
//      the top half of fmix32(w1 ^ v) ^ fmix32(w2 ^ k) for the iteration's
//      random words w1, w2;
//   2. a DPP wave minimum of the keys, then (only when several lanes hold it)
//      of their move ids, picks the unique best admissible move;
//   3. counts, colour, eligibility of the row/column vertices holding the old
//      or new colour (and the list), tenure, tabu entry, best-solution
//      snapshot.
//
// Bound by instruction issue: a lone wave takes about 7 cycles an instruction
// of any kind, and 16 waves per CU keep the VALU busy for two thirds of the
// time.  Per iteration at n = 50, half prefilled, |P| = 4096: 387 VALU, 279
// scalar, 53 LDS instructions and 41 branches; with every iteration dealt 502,
// 273, 68 and 55.  ns per iteration over the device (4096 searches) and us per
// iteration of a lone search, all dealt -> now:
//   n = 50, 50 % prefilled: 1.31 -> 1.15 ns, 2.74 -> 2.23 us
//   n = 70, 70 %:           4.06 -> 2.72 ns, 6.38 -> 4.31 us
//   n = 70, 80 %, PartialCol (chunks of 4): 2.94 -> 1.67 ns
//   n = 100, 50 %:          8.72 -> 7.45 us;   n = 10: 2.58 -> 1.78 us
// What keeps the scalar side small: wave-uniform values are made uniform for
// the compiler (readfirst, scalar loads of arguments and tables), and each loop
// has one exit, so that the list's registers are not copied at its joins.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace plse {

namespace {

struct WaveState {
    uint8_t *S;
    uint8_t *H;        // rowcnt [n][n+1] then colcnt [n][n+1]
    uint32_t *bm;
    uint8_t *tm8;      // [|V|] 0: no tabu entry this phase; 1: entries, all expired;
                       // m in 2..254: latest expiry = base + m - 1; 255: treat as live
    uint16_t *stage;   // [kPlitsStage] eligible vertices of consecutive ranks
    uint32_t *ring;    // chunk descriptors: vertex | chunk index << 16 | live << 31
    uint32_t *hk;      // [n+1] colour halves of the iteration's tie values
    uint32_t *planes;  // [B][W] bit b of floor(|D*(v)| / CH) (chunks per row - 1)
    int nplanes;
};

// Per-individual counters of one launch (moves = iterations - idle ones).
// Iterations per phase are at most 2^31 - 1, so the per-iteration ones fit 32
// bits; eligible-vertex and update sums take 64.
struct Cnt {
    uint32_t iters, idle, snaps, repairs;
    uint64_t elig, nupd, cupd;
};

struct Scal {
    int32_t f, c, nC;  // uncoloured, conflicting edges, conflicting vertices
    int32_t fbest, cbest;
};

// The lane id for code that seldom runs: addresses formed from it are not kept
// in registers around the search's loops.
__device__ __forceinline__ int rare_lane() {
    int lane = lane_id();
    asm volatile("" : "+v"(lane));
    return lane;
}

// Position of colour k in a candidate row with 128-bit domain mask a: 0 for
// k = 0, else 1 + the number of domain colours below k.
__device__ __forceinline__ uint32_t position_in(const u32x4 a, int k) {
    if (k == 0) return 0u;
    const uint64_t m0 = ((uint64_t)a.y << 32) | a.x;
    const uint64_t m1 = ((uint64_t)a.w << 32) | a.z;
    if (k < 64) return 1u + (uint32_t)__popcll(m0 & ((1ull << k) - 1ull));
    return 1u + (uint32_t)__popcll(m0) + (uint32_t)__popcll(m1 & ((1ull << (k - 64)) - 1ull));
}

// S from `src`; row/column colour counts; eligibility bitmap; f, c, |C(S)|.
__device__ void setup_state(const DevInstance &I, const uint8_t *src, const WaveState &ws,
                            Scal &sc) {
    const int lane = rare_lane();
    const int n = I.n, nv = I.nv, np1 = n + 1;
    for (int q = lane; q < (I.stride >> 4); q += 64)
        reinterpret_cast<u32x4 *>(ws.S)[q] = gload4(reinterpret_cast<const u32x4 *>(src) + q);
    const int hbytes = 2 * n * np1;
    uint32_t *h32 = reinterpret_cast<uint32_t *>(ws.H);
    for (int q = lane; q < (hbytes + 3) / 4; q += 64) h32[q] = 0u;
    PLSE_WAVE_SYNC();
    for (int v = lane; v < nv; v += 64) {
        const int s = ws.S[v];
        if (s) {
            const uint32_t rc = gptr(I.vrc)[v];
            const int a = (int)(rc & 0xFFu) * np1 + s;
            const int b = n * np1 + (int)(rc >> 8) * np1 + s;
            atomicAdd(&h32[a >> 2], 1u << ((a & 3) * 8));
            atomicAdd(&h32[b >> 2], 1u << ((b & 3) * 8));
        }
    }
    PLSE_WAVE_SYNC();
    const uint8_t *rowH = ws.H, *colH = ws.H + n * np1;
    const int W = (nv + 31) >> 5;
    uint32_t f = 0, c2 = 0, nC = 0;
    for (int w = lane; w < W; w += 64) {
        uint32_t bits = 0u;
        const int vend = min(nv, (w + 1) * 32);
        for (int v = w * 32; v < vend; ++v) {
            const int s = ws.S[v];
            int own = 0;
            if (s) {
                const uint32_t rc = gptr(I.vrc)[v];
                own = (int)rowH[(rc & 0xFFu) * np1 + s] + (int)colH[(rc >> 8) * np1 + s] - 2;
            }
            if (s == 0 || own > 0) bits |= 1u << (v & 31);
            f += (s == 0);
            c2 += (uint32_t)own;
            nC += (s != 0 && own > 0);
        }
        ws.bm[w] = bits;
    }
    for (int q = lane; q < (nv + 3) >> 2; q += 64) reinterpret_cast<uint32_t *>(ws.tm8)[q] = 0u;
    PLSE_WAVE_SYNC();
    sc.f = (int32_t)wave_sum_u32_dpp(f);
    sc.c = (int32_t)(wave_sum_u32_dpp(c2) >> 1);  // each conflicting edge seen twice
    sc.nC = (int32_t)wave_sum_u32_dpp(nC);
}

__device__ __forceinline__ void snapshot(const DevInstance &I, const uint8_t *S, uint8_t *dst) {
    for (int q = rare_lane(); q < (I.stride >> 4); q += 64)
        gstore4(reinterpret_cast<u32x4 *>(dst) + q, reinterpret_cast<const u32x4 *>(S)[q]);
}

// Zero the tabu rows this phase wrote (vertices with a nonzero mark).
__device__ void clear_tabu(const DevInstance &I, uint32_t *tabu, const WaveState &ws) {
    const int q4 = I.ts >> 2;
    for (int v = rare_lane(); v < I.nv; v += 64) {
        if (ws.tm8[v] != 0) {
            u32x4 *tb = reinterpret_cast<u32x4 *>(tabu + (size_t)v * I.ts);
            for (int t = 0; t < q4; ++t) gstore4(tb + t, u32x4{0u, 0u, 0u, 0u});
        }
    }
}

// base + off: a 32-bit offset from a uniform base needs no 64-bit address
// arithmetic per lane.
template <typename T>
__device__ __forceinline__ const T *at_byte(const void *base, uint32_t off) {
    return reinterpret_cast<const T *>(static_cast<const uint8_t *>(base) + off);
}

// CH consecutive candidate colours (bytes) and their tabu expiries.
template <int CH>
struct Chunk;

template <>
struct Chunk<2> {
    static __device__ __forceinline__ uint32_t colours(const uint8_t *p) {
        return *gptr(reinterpret_cast<const uint16_t *>(p));
    }
    static __device__ __forceinline__ void tabu(const uint32_t *p, uint32_t *t) {
        const u32x2 a = gload2(p);
        t[0] = a.x;
        t[1] = a.y;
    }
};

template <>
struct Chunk<4> {
    static __device__ __forceinline__ uint32_t colours(const uint8_t *p) {
        return *gptr(reinterpret_cast<const uint32_t *>(p));
    }
    static __device__ __forceinline__ void tabu(const uint32_t *p, uint32_t *t) {
        const u32x4 a = gload4(p);
        t[0] = a.x;
        t[1] = a.y;
        t[2] = a.z;
        t[3] = a.w;
    }
};

template <>
struct Chunk<8> {
    static __device__ __forceinline__ uint64_t colours(const uint8_t *p) {
        return *gptr(reinterpret_cast<const uint64_t *>(p));
    }
    static __device__ __forceinline__ void tabu(const uint32_t *p, uint32_t *t) {
        const u32x4 a = gload4(p);
        const u32x4 b = gload4(p + 4);
        t[0] = a.x;
        t[1] = a.y;
        t[2] = a.z;
        t[3] = a.w;
        t[4] = b.x;
        t[5] = b.y;
        t[6] = b.z;
        t[7] = b.w;
    }
};

// Slots of the chunk list, and the mark of a free lane (no vertex has it).
constexpr int kPlitsSlots = 6;
constexpr uint32_t kFreeLane = 0xFFFFFFFFu;
constexpr int32_t kZeroMove = 0x1000;       // e of a move that changes nothing
constexpr int32_t kOwnUncoloured = 0x1FFF;  // above every move's
constexpr uint32_t kNoMove = 0xFFFFFFFFu >> 3;
// Dealt iterations after the list is left, and after each idle one beside
// vertices in conflict.  There the list would find only a vertex's own colour,
// then be left and made again: with tenures that outlast the moves (n = 10,
// 40 %, alpha = 100, idle in nearly every iteration) 1.87 times as long as
// dealing, now 1.03; 16 instead of 8: n = 10, 80 %, 5 % longer.
constexpr uint32_t kCalm = 8u;

// Byte t of a chunk's colours.
__device__ __forceinline__ uint32_t colour_at(uint64_t cw, uint32_t t) {
    return __builtin_amdgcn_perm((uint32_t)(cw >> 32), (uint32_t)cw, t | 0x0C0C0C00u);
}
__device__ __forceinline__ uint32_t colour_at(uint32_t cw, uint32_t t) {
    return __builtin_amdgcn_perm(0u, cw, t | 0x0C0C0C00u);
}

// A lane's best move: value and tie value, its id (vertex << 7 | colour) and
// its vertex's payload.
struct Best {
    uint32_t hi, id, pay;
};

// v * u of 24-bit factors, u uniform (a full 32-bit product takes four times
// as long).
__device__ __forceinline__ uint32_t mul24(uint32_t v, uint32_t u) {
    uint32_t x;
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(x) : "s"(u), "v"(v));
    return x;
}

// A structure at a wave-uniform address, into scalar registers (read through
// an ordinary pointer it would be held in vector registers).
template <typename T>
__device__ __forceinline__ T cload(const void *p) {
    struct Words {
        uint32_t w[sizeof(T) / 4];
    } x;
    static_assert(sizeof(T) % 4 == 0, "whole words");
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) x.w[i] = cptr(static_cast<const uint32_t *>(p))[i];
    return __builtin_bit_cast(T, x);
}

// PH 1, 2: the two phases of Section 3.3.  PH 3: PartialCol (Section 3.7),
// the search of Partial-MPMA over legal partial colourings: the eligible
// vertices are the uncoloured ones (a legal colouring has no conflicts), a
// move colours one of them and uncolours its neighbours holding the colour,
// which then may not take it back for T iterations.
template <int CH, int PH>
__device__ void run_phase(const PlitsArgs &a, int64_t iters, uint32_t slot,
                          uint32_t gen, const uint8_t *src, uint8_t *out, uint32_t *tabu,
                          const WaveState &ws, Scal &sc, Cnt &ucnt, uint32_t &lane_cands) {
    const DevInstance &I = a.I;
    const int lane = lane_id();
    const int n = I.n, nv = I.nv, np1 = n + 1, TS = I.ts;
    // F = f + phi c: phase 1 phi = 1/2 (compared as 2 f + c), phase 2 phi = |V|;
    // PartialCol: F = f (c stays 0)
    const uint32_t tag = PH == 1 ? TAG_PLITS1 : (PH == 2 ? TAG_PLITS2 : TAG_PARTIAL);
    // Move values on a 13-bit scale e ordered like delta: e = delta, but in
    // phase 2 e = 4 dc + df, which orders moves as |V| dc + df does since
    // |df| <= 1 (with fewer than three vertices no two moves at a time differ).
    // Keys carry e + 2^12 over the 16-bit tie value over the move's position in
    // its chunk.
    constexpr int kShift = PH == 2 ? 2 : 0;
    constexpr int32_t eA = 1 << kShift;        // per unit of dc
    constexpr int32_t eB = PH == 1 ? 2 : 1;    // per unit of df
    const uint32_t alpha_n = (uint32_t)a.P.alpha_num, alpha_d = (uint32_t)a.P.alpha_den;
    const uint32_t m_alpha = 0xFFFFFFFFu / alpha_d;
    uint8_t *rowH = ws.H;
    uint8_t *colH = ws.H + n * np1;

    setup_state(I, src, ws, sc);
    if (src != out) snapshot(I, ws.S, out);
    sc.fbest = sc.f;
    sc.cbest = sc.c;
    const int W = (nv + 31) >> 5;
    uint32_t wx = 0u, wy = 0u, wz = 0u;  // random words of iterations (it & ~63) + lane
    // The tabu entry of a move is written at the start of the next
    // iteration's candidate loads (lane 0 holds it; the others hold ~0): its
    // completion then overlaps those loads instead of stalling the move.
    uint32_t pend_off = 0xFFFFFFFFu, pend_val = 0u;
    // likewise the expiry mark of the moved vertex, raised at the start of
    // the next iteration (under the eligibility scan)
    uint32_t pend_tv = 0xFFFFFFFFu, pend_tu = 0u;
    uint32_t tbase = 0u;  // base of the relative expiry marks
    // lane roles of the count updates
    const bool ln_new = (lane & 2) != 0;  // entering colour
    const bool ln_odd = (lane & 1) != 0;  // column count
    PLSE_WAVE_SYNC();

    // The chunk list: one chunk per lane and slot (vertex | chunk << 16 and, in
    // the vertex's first chunk, |D*(v)| << 24; the vertex's payload and the
    // chunk's colours), in any order.
    constexpr int R = kPlitsSlots;
    using Colours = decltype(Chunk<CH>::colours(nullptr));
    uint32_t sent[R], spay[R];
    Colours scw[R];
    uint32_t slots = 1u;  // slots in use
    // Free the lanes of vertex u.
    auto drop = [&](uint32_t u) {
#pragma unroll
        for (int q = 0; q < R; ++q)
            sent[q] = (sent[q] & 0xFFFFu) == u ? kFreeLane : sent[q];
    };
    // Give the chunks of vertex u the first free lanes; false if too few.
    auto enlist = [&](uint32_t u, uint32_t colour) -> bool {
        const uint32_t vi = *cptr(I.vinfo + u);
        const uint8_t *row = I.cand + (size_t)u * TS;
        const uint32_t d = (vi >> 16) & 0xFFu, pay = (vi & 0xFF00FFFFu) | (colour << 16);
        uint32_t need = d / CH + 1u, first = 0u;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if (need == 0u) break;
            const uint64_t room = ballot(sent[q] == kFreeLane);
            const uint32_t at = rank_below(room);
            const bool me = sent[q] == kFreeLane && at < need;
            const uint32_t ci = first + at;
            if (me) scw[q] = Chunk<CH>::colours(row + ci * CH);
            sent[q] = me ? u | (ci << 16) | (ci == 0u ? d << 24 : 0u) : sent[q];
            spay[q] = me ? pay : spay[q];
            const uint32_t got = min(need, (uint32_t)__popcll(room));
            first += got;
            need -= got;
            slots = max(slots, (uint32_t)q + 1u);
        }
        return need == 0u;
    };

    // Counters of the last 64 iterations.
    uint32_t n_elig = 0u, n_nupd = 0u, n_ends = 0u;
    auto tally = [&]() {
        ucnt.elig += n_elig;
        ucnt.nupd += n_nupd;
        ucnt.cupd += 2u * n_ends;
        n_elig = n_nupd = n_ends = 0u;
    };
    // iterations of a phase: below 2^31
    const uint32_t end = (uint32_t)iters;
    uint32_t itu = 0u, w0 = 0u, w1 = 0u, w2 = 0u;
    // Random words, expiry marks, the last move's tabu entry and the colour
    // halves of the tie values (nothing counts twice where an iteration is
    // begun again in the dealt form).
    auto begin = [&]() {
        if ((itu & 63u) == 0u) {
            const U4 rw = draw(a.seed_lo, a.seed_hi, slot, gen, tag, itu + (uint32_t)rare_lane());
            tally();
            wx = rw.x;
            wy = rw.y;
            wz = rw.z;
        }
        if ((itu & 127u) == 0u && tbase != itu) {
            // advance the base: marks drop by 128 (expired ones to 1), 255 stays
            tbase += 128u;
            PLSE_WAVE_SYNC();
            for (int q = rare_lane(); q < (nv + 3) >> 2; q += 64) {
                const uint32_t x = reinterpret_cast<uint32_t *>(ws.tm8)[q];
                uint32_t y = 0u;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t b = (x >> (8 * t)) & 0xFFu;
                    y |= (b == 255u ? 255u : (b > 128u ? b - 128u : (b != 0u ? 1u : 0u))) << (8 * t);
                }
                reinterpret_cast<uint32_t *>(ws.tm8)[q] = y;
            }
            PLSE_WAVE_SYNC();
        }
        if (lane == 0 && pend_tv != 0xFFFFFFFFu) {
            const uint32_t rel = pend_tu - tbase;  // >= 0
            const uint32_t mark = rel > 253u ? 255u : rel + 1u;
            if (mark > ws.tm8[pend_tv]) ws.tm8[pend_tv] = (uint8_t)mark;
        }
        if (pend_off != 0xFFFFFFFFu) gptr(tabu)[pend_off] = pend_val;
        w0 = readlane_u32(wx, (int)(itu & 63u));
        w1 = readlane_u32(wy, (int)(itu & 63u));
        w2 = readlane_u32(wz, (int)(itu & 63u));
        if (lane <= n) ws.hk[lane] = fmix32(w2 ^ (uint32_t)lane) >> 16 << 3;
        if (n >= 64 && lane + 64 <= n)
            ws.hk[lane + 64] = fmix32(w2 ^ (uint32_t)(lane + 64)) >> 16 << 3;
        PLSE_WAVE_SYNC();
    };
    // Aspiration F + delta < F*: keys below this.
    auto bound = [&]() -> uint32_t {
        const int32_t te = PH == 2 ? squeezed_bound(sc.fbest - sc.f, sc.cbest - sc.c, nv)
                         : (PH == 1 ? 2 * (sc.fbest - sc.f) + (sc.cbest - sc.c) : sc.fbest - sc.f);
        return (uint32_t)max(te + kZeroMove, 0) << 19;
    };
    // Wave-uniform flags as 0 or 1 in scalar registers (as conditions they
    // would be kept as lane masks); the 1 is opaque, or min became a compare.
    uint32_t one = 1u;
    asm("" : "+s"(one));
    auto nonzero = [&](uint32_t x) -> uint32_t { return min(x, one); };
    auto eligible = [&]() -> uint32_t { return (uint32_t)(PH == 3 ? sc.f : sc.f + sc.nC); };
    // The best move of chunk ci of vertex v (pay: row | column << 8 |
    // colour << 16 | degree << 24) against the lane's best so far.  Without
    // `exact` the vertex's own colour is no exception: it then counts two
    // conflicts more than the vertex has (kOwnUncoloured if uncoloured).
    auto look = [&](auto exact, Best &b, uint32_t teb, uint32_t v, uint32_t ci, bool live, uint32_t pay, Colours cw) {
        uint32_t tv[CH];
#pragma unroll
        for (int t = 0; t < CH; ++t) tv[t] = 0u;
        if (live)
            Chunk<CH>::tabu(at_byte<uint32_t>(tabu, (mul24(v, (uint32_t)TS) + ci * CH) * 4u), tv);
        const uint32_t s = (pay >> 16) & 0xFFu;
        const uint8_t *rH = rowH + __umul24(pay & 0xFFu, (uint32_t)np1);
        const uint8_t *cH = colH + __umul24((pay >> 8) & 0xFFu, (uint32_t)np1);
        // Up to four moves at a time.  Their LDS reads are issued together, the
        // second four's between the keys and the comparisons of the first
        // (the scheduler, saving registers, would wait for each pair).
        constexpr int kG = CH < 4 ? CH : 4;
        uint32_t kk[kG], ra[kG], ca[kG], hkv[kG], key[kG];
        auto fetch = [&](int g) {
#pragma unroll
            for (int t = 0; t < kG; ++t) kk[t] = (uint32_t)(cw >> (8 * (g + t))) & 0xFFu;
#pragma unroll
            for (int t = 0; t < kG; ++t) ra[t] = rH[kk[t]], ca[t] = cH[kk[t]];
#pragma unroll
            for (int t = 0; t < kG; ++t) hkv[t] = ws.hk[kk[t]];
            __builtin_amdgcn_sched_barrier(0);
        };
        const uint32_t sr = rH[s], sc_ = cH[s];
        fetch(0);
        // e = eB df + eA (conf(v,k) - conf(v,s)), df = -1 when v was
        // uncoloured (the counts of colour 0 are 0), +1 for the uncolour
        // move (k = 0, position 0)
        const uint32_t hv = fmix32(w1 ^ v) >> 16 << 3;
        const int32_t base = kZeroMove + (s ? 2 * eA : -eB) - eA * (int32_t)(sr + sc_);
        const int32_t base0 = ci != 0u ? base
                              : (!decltype(exact)::value && s == 0u ? kOwnUncoloured : base + eB);
        // the parts of the keys that do not depend on the colour
        const uint32_t kv = ((uint32_t)base << 19) + hv, kv0 = ((uint32_t)base0 << 19) + hv;
        uint32_t best = 0xFFFFFFFFu;
#pragma unroll
        for (int g = 0; g < CH; g += kG) {
            bool own[kG];
#pragma unroll
            for (int t = 0; t < kG; ++t) {
                const uint32_t x = __builtin_amdgcn_bitop3_b32(
                    g + t == 0 ? kv0 : kv, hkv[t], (uint32_t)(g + t), 0xBE);  // (a ^ b) | c
                key[t] = ((ra[t] + ca[t]) << (19 + kShift)) + x;
                own[t] = decltype(exact)::value && kk[t] == s;
            }
            if (g + kG < CH) {
                __builtin_amdgcn_sched_barrier(0);
                fetch(g + kG);
            }
            // keeps the compares of the expiries out of the branch that loads
            // them, where their results would wait in scalar registers
#pragma unroll
            for (int t = 0; t < kG; ++t) asm volatile("" : "+v"(tv[g + t]));
#pragma unroll
            for (int t = 0; t < kG; ++t) {
                // positions past the domain repeat its last colour and that
                // colour's tabu entry: they never beat the original, which
                // has a smaller position
                const bool ok = !own[t] & ((itu >= tv[g + t]) | (key[t] < teb));
                best = min(best, ok ? key[t] : 0xFFFFFFFFu);
            }
            if (g + kG < CH) __builtin_amdgcn_sched_barrier(0);
        }
        // positions ascend with colours: (value, tie value, id) of the
        // chunk's best decides against another chunk
        const uint32_t hi = best >> 3;
        const uint32_t id = (v << 7) | colour_at(cw, best & 7u);
        const bool take = hi < b.hi || (hi == b.hi && id < b.id);
        b.hi = take ? hi : b.hi;
        b.id = take ? id : b.id;
        b.pay = take ? pay : b.pay;
    };
    // Unique best over the wave: minimum of value and tie value, then of the
    // move ids among the lanes holding it; 0: no admissible move.
    auto choose = [&](const Best &b, uint32_t &id, uint32_t &pay) -> uint32_t {
        const uint32_t ghi = wave_min_u32_dpp(b.hi);
        uint64_t who = ballot(b.hi == ghi);
        if (__popcll(who) != 1) {
            const uint32_t gid = wave_min_u32_dpp(b.hi == ghi ? b.id : 0xFFFFFFFFu);
            who = ballot(b.hi == ghi && b.id == gid);
        }
        const int wl = (int)__builtin_ctzll(who);
        id = readlane_u32(b.id, wl);
        pay = readlane_u32(b.pay, wl);
        // (an uncoloured vertex's own colour is no move and comes after all)
        return nonzero(((uint32_t)kOwnUncoloured << 16) & ~ghi);
    };
    // Apply move (v, k); with `keep`, also to the list.  False: the list could
    // not take a vertex that joined.
    auto apply = [&](auto keep, uint32_t id, uint32_t pay) -> bool {
        bool list_ok = decltype(keep)::value;
        const int v = (int)(id >> 7), k = (int)(id & 0x7Fu);
        const int r = (int)(pay & 0xFFu);
        const int c = (int)((pay >> 8) & 0xFFu);
        const int old = (int)((pay >> 16) & 0xFFu);
        const int deg = (int)(pay >> 24);
        // the counts of the two colours in v's row and column, then the memory
        // the apply needs, fetched together: v's first 64 neighbours and its
        // domain mask (the tabu position of the colour it leaves)
        // (read through one address per lane: 0-1 old's row and column count,
        // 2-3 k's, where the move's updates go too)
        const uint32_t hcol = (uint32_t)(ln_new ? k : old);
        const uint32_t hb = (uint32_t)(ln_odd ? (n + c) * np1 : r * np1) + hcol;
        const uint32_t hval = ws.H[hb];
        const int32_t ho_r = (int32_t)readlane_u32(hval, 0), ho_c = (int32_t)readlane_u32(hval, 1);
        const int32_t hk_r = (int32_t)readlane_u32(hval, 2), hk_c = (int32_t)readlane_u32(hval, 3);
        const uint32_t *nb = I.nbr + (size_t)v * I.nl;
        const uint32_t ent0 = lane < deg ? gptr(nb)[lane] : 0u;
        u32x4 dmask{0u, 0u, 0u, 0u};
        if constexpr (PH != 3) dmask = *cptr(reinterpret_cast<const u32x4 *>(I.vrec) + 2 * v);
        const int32_t cvk = k ? hk_r + hk_c : 0;
        const int32_t cvo = old ? ho_r + ho_c - 2 : 0;
        const uint32_t is_k = nonzero((uint32_t)k), is_old = nonzero((uint32_t)old);
        const uint32_t vC = nonzero((uint32_t)cvk);  // v in conflict
        const uint32_t stays = vC | (1u ^ is_k);      // v in V_0 u C(S)
        PLSE_WAVE_SYNC();
        if constexpr (PH == 3) {
            // PartialCol: v (uncoloured) takes k; its cvk neighbours holding k
            // (at most one per row and column) are uncoloured and may not take
            // k back before `until`
            if (lane < 4) {
                const uint32_t add = hcol != 0u ? (ln_new ? 1u : ~0u) << ((hb & 3u) * 8u) : 0u;
                atomicAdd(reinterpret_cast<uint32_t *>(ws.H) + (hb >> 2), add);
            }
            if (lane == 0) {
                ws.S[v] = (uint8_t)k;
                atomicAdd(&ws.bm[v >> 5], 0u - (1u << (v & 31)));
            }
            sc.f += cvk - 1;
            n_ends += 1u + (uint32_t)cvk;
            const uint32_t mp = (uint32_t)sc.f;
            const uint32_t T = scale32(w0, 10u) + udiv_by(alpha_n * mp, alpha_d, m_alpha);
            const uint32_t until = itu + 1u + T;
            PLSE_WAVE_SYNC();
            // conflict-table entries: v's neighbours, then each uncoloured
            // vertex's neighbours
            uint32_t nupd_l = 0u;
            if (list_ok) drop((uint32_t)v);
            for (int t0 = 0; t0 < deg; t0 += 64) {
                const int t = t0 + lane;
                const uint32_t ent = t0 == 0 ? ent0 : (t < deg ? gptr(nb)[t] : 0u);
                const int u = (int)(ent & 0xFFFFu), other = (int)((ent >> 16) & 0x7FFFu);
                const bool freed = t < deg && ws.S[u] == k;
                uint64_t joins = list_ok ? ballot(freed) : 0ull;
                while (joins) {
                    const int L = (int)__ffsll((unsigned long long)joins) - 1;
                    joins &= joins - 1ull;
                    list_ok = enlist(readlane_u32((uint32_t)u, L), 0u) && list_ok;
                }
                if (freed) {
                    nupd_l += gptr(I.vinfo)[u] >> 24;
                    const bool inrow = (ent >> 31) == 0;
                    const int ur = inrow ? r : other, uc = inrow ? other : c;
                    const int rb = ur * np1 + k, cb = n * np1 + uc * np1 + k;
                    uint32_t *H32 = reinterpret_cast<uint32_t *>(ws.H);
                    ws.S[u] = 0;
                    atomicAdd(H32 + (rb >> 2), 0u - (1u << ((rb & 3) * 8)));
                    atomicAdd(H32 + (cb >> 2), 0u - (1u << ((cb & 3) * 8)));
                    atomicOr(&ws.bm[u >> 5], 1u << (u & 31));
                    // tabu entry (u, k), repeated over the rest of the chunk
                    // when k is u's last domain colour
                    const u32x4 dm = gload4(reinterpret_cast<const u32x4 *>(I.vrec) + 2 * u);
                    const uint32_t po = position_in(dm, k);
                    const uint32_t du = (uint32_t)(__popcll(((uint64_t)dm.y << 32) | dm.x) +
                                                   __popcll(((uint64_t)dm.w << 32) | dm.z));
                    const uint32_t nrep = po == du ? (uint32_t)CH - du % (uint32_t)CH : 1u;
                    for (uint32_t q = 0; q < nrep; ++q)
                        gptr(tabu)[(size_t)u * TS + po + q] = until;
                    const uint32_t rel = until - tbase;
                    const uint32_t mark = rel > 253u ? 255u : rel + 1u;
                    if (mark > ws.tm8[u]) ws.tm8[u] = (uint8_t)mark;
                }
            }
            n_nupd += (uint32_t)deg + wave_sum_u32_dpp(nupd_l);
        } else {
            // 4. apply.  Counts: lanes 0-1 the leaving colour's row and column
            //    count (-1), lanes 2-3 the entering colour's (+1), as LDS adds on
            //    the bytes of u32 words (exact: counts stay within 0..n, nothing
            //    carries), an add of 0 for colour 0.  Lane 0: v's colour, and v's
            //    eligibility bit cleared (an exact add: v was eligible) unless v
            //    stays in V_0 u C.
            if (lane < 4) {
                const uint32_t add = hcol != 0u ? (ln_new ? 1u : ~0u) << ((hb & 3u) * 8u) : 0u;
                atomicAdd(reinterpret_cast<uint32_t *>(ws.H) + (hb >> 2), add);
            }
            if (lane == 0) {
                ws.S[v] = (uint8_t)k;
                atomicAdd(&ws.bm[v >> 5], (stays - 1u) & (0u - (1u << (v & 31))));
            }
            PLSE_WAVE_SYNC();
            // eligibility of the row/column vertices holding the old or new colour:
            // all reads unconditional, one toggle where it changes
            int32_t dC = 0;
            if constexpr (decltype(keep)::value) {
                // v's chunks: its new colour, or free
                if (stays) {
                    const uint32_t npay = (pay & 0xFF00FFFFu) | ((uint32_t)k << 16);
#pragma unroll
                    for (int q = 0; q < R; ++q)
                        spay[q] = (sent[q] & 0xFFFFu) == (uint32_t)v ? npay : spay[q];
                } else {
                    drop((uint32_t)v);
                }
            }
            // those that hold k are in conflict now; those that hold old stay
            // so unless it was with v alone: the count of the shared line
            // without v is known, that of their other line read
            const uint32_t kx = k ? (uint32_t)k : 256u, ox = old ? (uint32_t)old : 256u;
            for (int t0 = 0; t0 < deg; t0 += 64) {
                const int t = t0 + lane;
                const uint32_t ent = t0 == 0 ? ent0 : (t < deg ? gptr(nb)[t] : 0u);
                const bool inrow = (ent >> 31) == 0;
                const int u = (int)(ent & 0xFFFFu), other = (int)((ent >> 16) & 0x7FFFu);
                const uint32_t su = ws.S[u];
                const uint32_t bw = ws.bm[u >> 5];
                const uint32_t other_n = ws.H[(other + (inrow ? n : 0)) * np1 + (int)su];
                const uint32_t shared = (uint32_t)(inrow ? ho_r : ho_c);
                const bool hit = (t < deg) & ((su == ox) | (su == kx));
                const bool was = (bw >> (u & 31)) & 1u;
                const bool now = (su == kx) | (shared + other_n > 3u);
                const bool flip = hit && (now != was);
                if (flip) atomicXor(&ws.bm[u >> 5], 1u << (u & 31));
                uint64_t joins = ballot(flip && now), leaves = ballot(flip && !now);
                dC += (int32_t)__popcll(joins) - (int32_t)__popcll(leaves);
                if (list_ok) {
                    while (leaves) {
                        const int L = (int)__ffsll((unsigned long long)leaves) - 1;
                        leaves &= leaves - 1ull;
                        drop(readlane_u32((uint32_t)u, L));
                    }
                    while (joins) {
                        const int L = (int)__ffsll((unsigned long long)joins) - 1;
                        joins &= joins - 1ull;
                        list_ok = enlist(readlane_u32((uint32_t)u, L), (uint32_t)k) && list_ok;
                    }
                }
            }
            sc.nC += dC + (int32_t)vC - (int32_t)is_old;
            sc.f += (int32_t)is_old - (int32_t)is_k;
            sc.c += cvk - cvo;
            const uint32_t ends = is_old + is_k;
            n_ends += ends;
            n_nupd += (uint32_t)deg * ends;
            // tenure T = L + alpha (|V_0| + |C|) after the move; moving v back to
            // `old` is tabu for T iterations
            const uint32_t mp = (uint32_t)(sc.f + sc.nC);
            const uint32_t T = scale32(w0, 10u) + udiv_by(alpha_n * mp, alpha_d, m_alpha);
            const uint32_t until = itu + 1u + T;
            pend_tv = (uint32_t)v;
            pend_tu = until;
            {
                // the entry of the last domain colour is repeated over the rest
                // of its chunk, where the candidate row repeats that colour
                const uint32_t po = position_in(dmask, old);
                const uint32_t dv = (uint32_t)(__popcll(((uint64_t)dmask.y << 32) | dmask.x) +
                                               __popcll(((uint64_t)dmask.w << 32) | dmask.z));
                const uint32_t nrep = po == dv ? (uint32_t)CH - dv % (uint32_t)CH : 1u;
                pend_off = (uint32_t)lane < nrep ? (uint32_t)v * (uint32_t)TS + po + (uint32_t)lane
                                                 : 0xFFFFFFFFu;
                pend_val = until;
            }
        }
        PLSE_WAVE_SYNC();
        // F < F*: in phase 2 the conflicts decide, except one conflict more
        // against |V| uncoloured vertices fewer, which is equal
        const int32_t gf = sc.f - sc.fbest, gc = sc.c - sc.cbest;
        if (PH == 1 ? 2 * gf + gc < 0
                    : (PH == 3 ? gf < 0 : (gc < -1 || (gc == -1 && gf < nv) || (gc == 0 && gf < 0)))) {
            sc.fbest = sc.f;
            sc.cbest = sc.c;
            snapshot(I, ws.S, out);
            ucnt.snaps++;
        }
        return list_ok;
    };
    // Stage the eligible vertices of rank g .. g + kPlitsStage - 1, ascending.
    auto stage_from = [&](uint32_t g) {
        const int lane = rare_lane();
        const uint32_t gend = g + (uint32_t)kPlitsStage;
        uint32_t base = 0;
        for (int wb = 0; wb < W && base < gend; wb += 64) {
            const int w = wb + lane;
            uint32_t bits = (w < W) ? ws.bm[w] : 0u;
            uint32_t total;
            uint32_t pos = base + wave_excl_scan_dpp((uint32_t)__popc(bits), &total);
#pragma unroll 1
            while (bits && pos < gend) {
                const int b = __ffs(bits) - 1;
                bits &= bits - 1u;
                if (pos >= g) ws.stage[pos - g] = (uint16_t)(w * 32 + b);
                ++pos;
            }
            base += total;
        }
        PLSE_WAVE_SYNC();
    };
    // Make the list of the staged eligible vertices; false if they do not fit.
    auto build = [&]() -> bool {
        const int lane = rare_lane();
        const uint32_t m = eligible();
        if (m > (uint32_t)kPlitsStage) return false;
        stage_from(0u);
#pragma unroll
        for (int q = 0; q < R; ++q) sent[q] = kFreeLane, spay[q] = 0u, scw[q] = 0;
        uint32_t chunks = 0u;
        for (uint32_t g = 0u; g < m; g += 64u) {
            const uint32_t e = g + (uint32_t)lane;
            uint32_t v = 0u, nch = 0u, d = 0u;
            if (e < m) {
                v = ws.stage[e];
                d = (*gptr(at_byte<uint32_t>(I.vinfo, v * 4u)) >> 16) & 0xFFu;
                nch = d / CH + 1u;
            }
            uint32_t total;
            const uint32_t at = wave_excl_scan_dpp(nch, &total);
#pragma unroll 1
            for (uint32_t t = 0; t < nch; ++t)
                ws.ring[at + t] = v | (t << 16) | (t == 0u ? d << 24 : 0u);
            PLSE_WAVE_SYNC();
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const uint32_t y = 64u * (uint32_t)q + (uint32_t)lane - chunks;
                if (y < total) sent[q] = ws.ring[y];
            }
            PLSE_WAVE_SYNC();
            chunks += total;
        }
        if (chunks > 64u * (uint32_t)R) return false;
        slots = max(1u, (chunks + 63u) >> 6);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if (sent[q] != kFreeLane) {
                const uint32_t v = sent[q] & 0xFFFFu, ci = (sent[q] >> 16) & 0xFFu;
                const uint32_t vi = *gptr(at_byte<uint32_t>(I.vinfo, v * 4u));
                spay[q] = (vi & 0xFF00FFFFu) | ((uint32_t)ws.S[v] << 16);
                scw[q] = Chunk<CH>::colours(at_byte<uint8_t>(I.cand, v * (uint32_t)TS + ci * CH));
            }
        }
        return true;
    };

    // One exit per loop: the list's registers then stay where they are.
    bool done = end == 0u || eligible() == 0u;
    uint32_t deal = 1u;  // dealt iterations to come, at the least
    while (!done) {
        if (deal) {
            // dealt iterations, until the chunks fit the list
            do {
                begin();
                stage_from(0u);
                const uint32_t m = eligible();
                n_elig += m;
                const int lane = rare_lane();
                const uint32_t teb = bound();
                Best b{kNoMove, 0u, 0u};
                uint32_t chunks = 0u;
                uint32_t head = 0u, tail = 0u, g = 0u;
                uint32_t sbase = 0u;  // rank of stage[0]
                for (;;) {
                    // once the ring is empty, deal the rows of the next 64 eligible
                    // vertices into it
                    if (head == tail && g < m) {
                        head = tail = 0u;
                        if (g >= sbase + (uint32_t)kPlitsStage) {
                            // the bitmap does not change within the iteration
                            PLSE_WAVE_SYNC();
                            sbase = g;
                            stage_from(g);
                        }
                        const uint32_t e = g + (uint32_t)lane;
                        uint32_t v = 0u, nch = 0u, ent = 0u;
                        if (e < m) {
                            v = ws.stage[e - sbase];
                            // chunk count and liveness of v, read together: planes 0
                            // and 1 (or 0 twice), further planes only when present
                            const int vw = (int)(v >> 5);
                            const bool p0ok = ws.nplanes > 0, p1ok = ws.nplanes > 1;
                            const uint32_t q0 = p0ok ? ws.planes[vw] : 0u;
                            const uint32_t q1 = p1ok ? ws.planes[W + vw] : 0u;
                            const uint32_t tm = ws.tm8[v];
                            uint32_t code = ((q0 >> (v & 31u)) & 1u) | (((q1 >> (v & 31u)) & 1u) << 1);
                            if (ws.nplanes > 2) {
#pragma unroll
                                for (int b = 2; b < 6; ++b)
                                    if (b < ws.nplanes)
                                        code |= ((ws.planes[b * W + vw] >> (v & 31u)) & 1u) << b;
                            }
                            nch = code + 1u;  // ceil((d + 1) / CH)
                            // a vertex not live has no tabu move this iteration
                            const bool live = tm > itu - tbase + 1u;
                            ent = v | ((uint32_t)live << 31);
                        }
                        uint32_t total;
                        const uint32_t at = tail + wave_excl_scan_dpp(nch, &total);
#pragma unroll 1
                        for (uint32_t t = 0; t < nch; ++t) ws.ring[at + t] = ent | (t << 16);
                        tail += total;
                        g += 64u;
                        PLSE_WAVE_SYNC();
                        chunks += total;
                    }
                    if (head == tail) break;
                    const uint32_t x = head + (uint32_t)lane;
                    head = min(head + 64u, tail);
                    if (x < tail) {
                        // ring entry: vertex | chunk index << 16 | live << 31
                        const uint32_t ent = ws.ring[x];
                        const uint32_t v = ent & 0xFFFFu, ci = (ent >> 16) & 0x7FFFu;
                        const uint32_t vi = *gptr(at_byte<uint32_t>(I.vinfo, v * 4u));
                        if (ci == 0u) lane_cands += (vi >> 16) & 0xFFu;
                        look(std::true_type{}, b, teb, v, ci, (ent >> 31) != 0u, (vi & 0xFF00FFFFu) | ((uint32_t)ws.S[v] << 16),
                             Chunk<CH>::colours(at_byte<uint8_t>(I.cand, v * (uint32_t)TS + ci * CH)));
                    }
                    PLSE_WAVE_SYNC();
                }
                uint32_t id, pay;
                const uint32_t any = choose(b, id, pay);
                --deal;
                if (any) {
                    (void)apply(std::false_type{}, id, pay);
                } else {
                    ucnt.idle++;
                    if (PH != 3 && sc.nC != 0) deal = kCalm;  // (no conflicts in PartialCol)
                }
                ++itu;
                done = itu >= end || eligible() == 0u;  // none: complete legal colouring
                if (chunks + 32u > 64u * (uint32_t)R) deal = max(deal, 1u);
            } while (deal && !done);
        }
        if (!done) {
            deal = build() ? 0u : 1u;
            if (deal == 0u) {
                // iterations on the list
                bool relist = false, leave;
                do {
                    begin();
                    const uint32_t m = eligible(), teb = bound(), cands0 = lane_cands;
                    Best b{kNoMove, 0u, 0u};
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        if ((uint32_t)q >= slots) break;
                        if (sent[q] != kFreeLane) {
                            const uint32_t v = sent[q] & 0xFFFFu;
                            const uint32_t tm = ws.tm8[v];
                            lane_cands += sent[q] >> 24;
                            look(std::false_type{}, b, teb, v, (sent[q] >> 16) & 0xFFu,
                                 tm > itu - tbase + 1u, spay[q], scw[q]);
                        }
                    }
                    PLSE_WAVE_SYNC();
                    uint32_t id, pay;
                    const uint32_t any = choose(b, id, pay);
                    // no move is better than the own colour of a vertex in
                    // conflict: such moves have to be told apart, which the
                    // dealt form does
                    const uint32_t own = any & (1u ^ nonzero((id & 0x7Fu) ^ ((pay >> 16) & 0xFFu)));
                    bool room = true;
                    if (any > own) room = apply(std::true_type{}, id, pay);
                    ucnt.idle += 1u ^ any;
                    n_elig += m & (own - 1u);
                    itu += 1u - own;
                    if (own) lane_cands = cands0;
                    if ((itu & 15u) == 0u && slots > 1u) {
                        // fewer chunks than the slots in use are there for
                        uint32_t chunks = 0u;
#pragma unroll
                        for (int q = 0; q < R; ++q)
                            chunks += (uint32_t)__popcll(ballot(sent[q] != kFreeLane));
                        relist = chunks + 8u <= 64u * (slots - 1u);
                    }
                    leave = own || !room;
                    done = itu >= end || eligible() == 0u;
                } while (!leave && !relist && !done);
                deal = leave ? kCalm : 0u;
            }
        }
    }
    ucnt.iters += itu;
    tally();
    // the last move's tabu entry and mark: the mark tells clear_tabu the row
    // was written
    if (pend_off != 0xFFFFFFFFu) gptr(tabu)[pend_off] = pend_val;
    if (lane == 0 && pend_tv != 0xFFFFFFFFu && ws.tm8[pend_tv] == 0) ws.tm8[pend_tv] = 1;
    PLSE_WAVE_SYNC();
    clear_tabu(I, tabu, ws);
    PLSE_WAVE_SYNC();
}

// Greedy conflict removal (Section 3.7): uncolour the vertex with the most
// conflicts (ties: lowest id) until the colouring is legal; `from` -> `out`.
__device__ void repair(const PlitsArgs &a, const uint8_t *from, uint8_t *out, const WaveState &ws,
                       Scal &sc, Cnt &ucnt) {
    const DevInstance &I = a.I;
    const int lane = rare_lane();
    const int n = I.n, nv = I.nv, np1 = n + 1;
    setup_state(I, from, ws, sc);
    uint8_t *rowH = ws.H, *colH = ws.H + n * np1;
    for (;;) {
        uint32_t lkey = 0u;
        for (int v = lane; v < nv; v += 64) {
            const int s = ws.S[v];
            if (s) {
                const uint32_t rc = gptr(I.vrc)[v];
                const int own =
                    (int)rowH[(rc & 0xFFu) * np1 + s] + (int)colH[(rc >> 8) * np1 + s] - 2;
                if (own > 0) {
                    const uint32_t key = ((uint32_t)own << 16) | (0xFFFFu - (uint32_t)v);
                    lkey = key > lkey ? key : lkey;
                }
            }
        }
        const uint32_t g = wave_max_u32(lkey);
        if (g == 0u) break;
        const int v = (int)(0xFFFFu - (g & 0xFFFFu));
        if (lane == 0) {
            const uint32_t rc = gptr(I.vrc)[v];
            const int old = ws.S[v];
            rowH[(rc & 0xFFu) * np1 + old] -= 1;
            colH[(rc >> 8) * np1 + old] -= 1;
            ws.S[v] = 0;
        }
        ucnt.repairs++;
        PLSE_WAVE_SYNC();
    }
    snapshot(I, ws.S, out);
    PLSE_WAVE_SYNC();
}

// The search of individual `ind` of one instance in generation `gen`, by one
// wave whose LDS starts at `base`.
template <int CH, bool PARTIAL>
__device__ __forceinline__ void plits_individual(const PlitsArgs &a, int ind, int gen, uint8_t *base) {
    WaveState ws;
    ws.S = base;
    ws.H = base + a.off_h;
    ws.bm = reinterpret_cast<uint32_t *>(base + a.off_bm);
    ws.tm8 = base + a.off_tm;
    ws.stage = reinterpret_cast<uint16_t *>(base + a.off_el);
    ws.ring = reinterpret_cast<uint32_t *>(base + a.off_ring);
    ws.hk = reinterpret_cast<uint32_t *>(base + a.off_hk);
    ws.planes = reinterpret_cast<uint32_t *>(base + a.off_planes);
    ws.nplanes = a.nplanes;
    {
        // chunk-count planes: bit b of floor(|D*(v)| / CH) per vertex
        const int W = (a.I.nv + 31) >> 5;
        for (int w = lane_id(); w < W; w += 64) {
            uint32_t pl[6] = {0u, 0u, 0u, 0u, 0u, 0u};
            const int vend = min(a.I.nv, (w + 1) * 32);
            for (int v = w * 32; v < vend; ++v) {
                const uint32_t code = ((gptr(a.I.vinfo)[v] >> 16) & 0xFFu) / CH;
#pragma unroll
                for (int b = 0; b < 6; ++b) pl[b] |= ((code >> b) & 1u) << (v & 31);
            }
            for (int b = 0; b < a.nplanes; ++b) ws.planes[b * W + w] = pl[b];
        }
    }
    const DevInstance &I = a.I;
    ind = readfirst(ind);
    uint32_t *tabu = a.tabu + (size_t)ind * I.nv * I.ts;
    const uint8_t *src = a.S_in + (size_t)ind * I.stride;
    uint8_t *out = a.S_out + (size_t)ind * I.stride;

    Cnt ucnt{0u, 0u, 0u, 0u, 0ull, 0ull, 0ull};
    uint32_t lane_cands = 0;
    Scal sc;
    const uint32_t slot = (uint32_t)ind;
    int32_t f_final;
    if constexpr (PARTIAL) {
        // Partial-MPMA (Section 3.7): the offspring repaired into a legal
        // partial colouring, then PartialCol for the whole depth
        repair(a, src, out, ws, sc, ucnt);
        run_phase<CH, 3>(a, a.P.depth1 + a.P.depth2, slot, (uint32_t)gen, out, out, tabu, ws,
                         sc, ucnt, lane_cands);
        f_final = sc.fbest;
    } else {
        // phase 1 from the offspring, phase 2 from phase 1's best (both write
        // their best into `out`)
        run_phase<CH, 1>(a, a.P.depth1, slot, (uint32_t)gen, src, out, tabu, ws, sc, ucnt,
                         lane_cands);
        run_phase<CH, 2>(a, a.P.depth2, slot, (uint32_t)gen, out, out, tabu, ws, sc, ucnt,
                         lane_cands);
        f_final = sc.fbest;
        if (sc.cbest > 0) {
            repair(a, out, out, ws, sc, ucnt);
            f_final = sc.f + (int32_t)ucnt.repairs;
        }
    }
    const uint64_t cands = wave_sum_u64(lane_cands);
    const int lane = lane_id();
    if (lane < kCounters) {
        uint64_t v = 0;
        switch (lane) {
            case C_ITERS: v = ucnt.iters; break;
            case C_MOVES: v = ucnt.iters - ucnt.idle; break;
            case C_IDLE: v = ucnt.idle; break;
            case C_CANDS: v = cands; break;
            case C_ELIG: v = ucnt.elig; break;
            case C_NUPD: v = ucnt.nupd; break;
            case C_SNAPS: v = ucnt.snaps; break;
            case C_REPAIRS: v = ucnt.repairs; break;
            default: v = ucnt.cupd; break;
        }
        gptr(a.cnt_out)[(size_t)ind * kCounters + lane] = v;
    }
    if (lane == 0) gptr(a.f_out)[ind] = f_final;
}

}  // namespace

template <int CH, bool PARTIAL>
__global__ __launch_bounds__(256, 4) void plits_kernel(const ArgList L) {
    extern __shared__ __align__(16) uint8_t lds[];
    const PlitsArgs a = cload<PlitsArgs>(L.p[blockIdx.y]);
    const int wv = (int)(threadIdx.x >> 6);
    const int ind = (int)blockIdx.x * (int)(blockDim.x >> 6) + wv;
    if (ind >= a.p) return;
    int gen = a.gen_fixed;
    if (gen == 0) {
        if (gptr(a.ctl)->stop) return;
        gen = gptr(a.ctl)->gen;
    }
    plits_individual<CH, PARTIAL>(a, ind, gen, lds + (size_t)wv * a.lds_per_wave);
}

// Persistent form for many instances: every wave takes (instance,
// individual) items from a queue until it runs dry.  Items run instance by
// instance in the order of the argument list (longest estimated work first),
// individuals in order within an instance; stopped instances are skipped.
// Every wave of the launch uses `lds_per_wave` bytes (the largest instance's).
template <int CH, bool PARTIAL>
__global__ __launch_bounds__(256, 4) void plits_persistent_kernel(const ArgList L, int count, int p,
                                                                  int lds_per_wave,
                                                                  uint32_t *queue) {
    extern __shared__ __align__(16) uint8_t lds[];
    uint8_t *base = lds + (size_t)(threadIdx.x >> 6) * lds_per_wave;
    const uint32_t total = (uint32_t)count * (uint32_t)p;
    for (;;) {
        uint32_t item = 0u;
        if (lane_id() == 0) item = atomicAdd(queue, 1u);
        item = readlane_u32(item, 0);
        if (item >= total) break;
        const uint32_t inst = item / (uint32_t)p, ind = item - inst * (uint32_t)p;
        const PlitsArgs a = cload<PlitsArgs>(L.p[inst]);
        int gen = a.gen_fixed;
        if (gen == 0) {
            if (gptr(a.ctl)->stop) continue;
            gen = gptr(a.ctl)->gen;
        }
        plits_individual<CH, PARTIAL>(a, (int)ind, gen, base);
        PLSE_WAVE_SYNC();
    }
}

__global__ void queue_reset_kernel(uint32_t *queue) {
    if (threadIdx.x == 0) *gptr(queue) = 0u;
}

// The PLITS kernel of a chunk size, MPMA or Partial-MPMA; null for other sizes.
const void *plits_fn(int slots_per_lane, bool partial) {
    switch (slots_per_lane) {
        case 2: return partial ? (const void *)plits_kernel<2, true> : (const void *)plits_kernel<2, false>;
        case 4: return partial ? (const void *)plits_kernel<4, true> : (const void *)plits_kernel<4, false>;
        case 8: return partial ? (const void *)plits_kernel<8, true> : (const void *)plits_kernel<8, false>;
        default: return nullptr;
    }
}

// Zero a tabu region (a fresh workspace, before the first phase uses it).
__global__ void fill_zero_kernel(const ArgList L) {
    const FillArgs a = arg_of<FillArgs>(L);
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t nq = a.n / 4;
    for (size_t i = t; i < nq; i += (size_t)gridDim.x * blockDim.x)
        gstore4(reinterpret_cast<u32x4 *>(a.p) + i, u32x4{0u, 0u, 0u, 0u});
    for (size_t i = nq * 4 + t; i < a.n; i += (size_t)gridDim.x * blockDim.x) gptr(a.p)[i] = 0u;
}

hipError_t launch_plits(const ArgList &L, int count, int p, int lds_per_wave,
                        int slots_per_lane, int waves_per_block, bool partial, bool lean,
                        hipStream_t stream) {
    const int blocks = (p + waves_per_block - 1) / waves_per_block;
    const size_t lds = (size_t)lds_per_wave * waves_per_block;
    const dim3 grid(blocks, count), block(64 * waves_per_block);
    const void *fn = lean ? plits_lean_fn(slots_per_lane) : plits_fn(slots_per_lane, partial);
    if (!fn) return hipErrorInvalidValue;
    void *args[] = {const_cast<ArgList *>(&L)};
    return hipLaunchKernel(fn, grid, block, args, lds, stream);
}

const void *plits_persistent_fn(int slots_per_lane, bool partial) {
    switch (slots_per_lane) {
        case 2: return partial ? (const void *)plits_persistent_kernel<2, true>
                               : (const void *)plits_persistent_kernel<2, false>;
        case 4: return partial ? (const void *)plits_persistent_kernel<4, true>
                               : (const void *)plits_persistent_kernel<4, false>;
        case 8: return partial ? (const void *)plits_persistent_kernel<8, true>
                               : (const void *)plits_persistent_kernel<8, false>;
        default: return nullptr;
    }
}

hipError_t launch_plits_persistent(const ArgList &L, int count, int p, int lds_per_wave,
                                   int slots_per_lane, int waves_per_block, bool partial,
                                   int blocks, uint32_t *queue, hipStream_t stream) {
    const void *fn = plits_persistent_fn(slots_per_lane, partial);
    if (!fn || blocks < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(queue_reset_kernel, dim3(1), dim3(64), 0, stream, queue);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds = (size_t)lds_per_wave * waves_per_block;
    ArgList Lc = L;
    void *args[] = {&Lc, &count, &p, &lds_per_wave, &queue};
    return hipLaunchKernel(fn, dim3(blocks), dim3(64 * waves_per_block), args, lds, stream);
}

hipError_t launch_fill_zero(const ArgList &L, int count, hipStream_t stream) {
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1024, count), dim3(256), 0, stream, L);
    return hipGetLastError();
}

// Resident waves per CU of a PLITS launch shape (the runtime's occupancy
// calculation: registers, LDS and workgroup limits).
int plits_waves_per_cu(int slots_per_lane, int waves_per_block, int lds_per_wave, bool partial,
                       bool lean, bool persistent) {
    const void *fn = lean ? plits_lean_fn(slots_per_lane)
                          : (persistent ? plits_persistent_fn(slots_per_lane, partial)
                                        : plits_fn(slots_per_lane, partial));
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, 64 * waves_per_block,
                                                     (size_t)lds_per_wave * waves_per_block) !=
        hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return blocks * waves_per_block;
}

hipError_t plits_set_lds_limit(int bytes) {
    hipError_t e = hipSuccess;
    for (int spl : {2, 4, 8}) {
        for (bool partial : {false, true})
            if (e == hipSuccess) e = set_dynamic_lds_limit(plits_fn(spl, partial), bytes);
        if (e == hipSuccess) e = set_dynamic_lds_limit(plits_lean_fn(spl), bytes);
        for (bool partial : {false, true})
            if (e == hipSuccess) e = set_dynamic_lds_limit(plits_persistent_fn(spl, partial), bytes);
    }
    return e;
}

}  // namespace plse
