// k_evo.hip -- the per-generation kernels around the tabu search on gfx950:
// best-solution saving, bit-sliced Hamming distances (Eq. 8), the
// population update (Alg. 4), nearest-neighbour parent matching
// (Section 3.5.1) and the AUX crossover (Alg. 5, Eq. 9), plus the small
// control kernels of the generation graph.
#include "device_common.h"
#include "kernels.h"

namespace plse {

// ---------------------------------------------------------------------------
// control
// ---------------------------------------------------------------------------
__global__ void ctl_reset_kernel(const ArgList L) {
    Ctl *ctl = static_cast<Ctl *>(const_cast<void *>(L.p[blockIdx.y]));
    if (threadIdx.x == 0) {
        ctl->gen = 0;
        ctl->stop = 0;
        ctl->fstar = INT32_MAX;
        ctl->best_gen = 0;
        ctl->gens_run = 0;
        ctl->stop_reason = 0;
        ctl->iters = 0;
    }
}

__global__ void gen_begin_kernel(const ArgList L) {
    Ctl *ctl = static_cast<Ctl *>(const_cast<void *>(L.p[blockIdx.y]));
    if (threadIdx.x == 0 && !ctl->stop) ctl->gen += 1;
}

// Fresh population bookkeeping: uid = slot, empty partner history, and the
// first offspring population is the initial population itself (Alg. 2).
__global__ void pop_setup_kernel(const ArgList L) {
    const PopSetupArgs a = arg_of<PopSetupArgs>(L);
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (size_t)a.p) {
        a.uid[i] = i;
        a.hc[i] = 0;
    }
    const size_t nq = (size_t)a.p * (a.stride >> 4);
    for (size_t q = i; q < nq; q += (size_t)gridDim.x * blockDim.x)
        reinterpret_cast<uint4 *>(a.S_off)[q] = reinterpret_cast<const uint4 *>(a.S)[q];
}

// ---------------------------------------------------------------------------
// best-solution saving (Alg. 2): argmin f over the improved offspring, ties to
// the lowest slot; S* replaced only on strict improvement.  Also sums the
// per-individual counters of the generation and sets the bound stop flag.
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(1024) void best_kernel(const ArgList L) {
    const BestArgs a = arg_of<BestArgs>(L);
    if (a.ctl->stop) return;
    const int g = a.ctl->gen;
    __shared__ uint64_t kmin[16];
    __shared__ uint64_t csum[16][kCounters];
    __shared__ int improved;
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint64_t key = ~0ull;
    uint64_t c[kCounters];
#pragma unroll
    for (int q = 0; q < kCounters; ++q) c[q] = 0;
    for (int i = tid; i < a.p; i += blockDim.x) {
        const uint64_t k = ((uint64_t)(uint32_t)a.f_new[i] << 32) | (uint32_t)i;
        key = k < key ? k : key;
#pragma unroll
        for (int q = 0; q < kCounters; ++q) c[q] += a.cnt[(size_t)i * kCounters + q];
    }
    key = wave_min_u64(key);
#pragma unroll
    for (int q = 0; q < kCounters; ++q) c[q] = wave_sum_u64(c[q]);
    if (lane == 0) {
        kmin[wv] = key;
#pragma unroll
        for (int q = 0; q < kCounters; ++q) csum[wv][q] = c[q];
    }
    __syncthreads();
    if (tid == 0) {
        uint64_t k = ~0ull;
        uint64_t s[kCounters] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            k = kmin[w] < k ? kmin[w] : k;
            for (int q = 0; q < kCounters; ++q) s[q] += csum[w][q];
        }
        const int32_t fb = (int32_t)(k >> 32);
        improved = 0;
        if (fb < a.ctl->fstar) {
            a.ctl->fstar = fb;
            a.ctl->best_gen = g;
            improved = 1 + (int)(uint32_t)k;  // slot + 1
        }
        GenStat &gs = a.stats[g - 1];
        gs.best_f = a.ctl->fstar;
        for (int q = 0; q < kCounters; ++q) gs.cnt[q] = s[q];
        a.ctl->gens_run = g;
        a.ctl->iters += s[0];
        if (a.stop_at_ub && a.nsq_minus_l - a.ctl->fstar == a.ub) {
            a.ctl->stop = 1;
            a.ctl->stop_reason = 1;
        } else if (a.max_iters > 0 && a.ctl->iters >= (uint64_t)a.max_iters) {
            // iteration budget (Section 4.3), known at generation ends only
            a.ctl->stop = 1;
            a.ctl->stop_reason = 2;
        }
    }
    __syncthreads();
    if (improved) {
        const uint8_t *src = a.S_new + (size_t)(improved - 1) * a.stride;
        for (int q = tid; q < (a.stride >> 4); q += blockDim.x)
            reinterpret_cast<uint4 *>(a.Sstar)[q] = reinterpret_cast<const uint4 *>(src)[q];
    }
}

// ---------------------------------------------------------------------------
// Hamming distances (Eq. 8), bit-sliced.  pack: colour bit b of vertices
// 32w..32w+31 of row x -> planes[(w*pitch + x)*B + b].  A pair differs at v iff
// some plane differs, so D = sum_w popcount(OR_b (a_b XOR c_b)).
// ---------------------------------------------------------------------------

// One thread per row and word: 32 colours as eight u32 words; the bits b of a
// word's four bytes are brought together by a multiplication.  32768 rows of
// n = 50: 45 us (byte by byte: 95), of which 41 MB in and 31 MB out take 14.
__global__ __launch_bounds__(256) void pack_kernel(const ArgList L) {
    const PackArgs a = arg_of<PackArgs>(L);
    if (a.ctl && a.ctl->stop) return;
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (size_t)a.m * a.W) return;
    const int x = a.row0 + (int)(t / a.W), w = (int)(t % a.W);
    const uint8_t *row = a.S + (size_t)x * a.stride + 32 * w;
    const u32x4 lo = gload4_any(row);
    u32x4 hi = {0u, 0u, 0u, 0u};
    if (32 * w + 16 < a.stride) hi = gload4_any(row + 16);
    const uint32_t s[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    const int left = a.nv - 32 * w;  // vertices in the word
    const uint32_t valid = left >= 32 ? 0xFFFFFFFFu : (1u << left) - 1u;
    uint32_t *dst = a.planes + ((size_t)w * a.pitch + x) * a.B;
    for (int b = 0; b < a.B; ++b) {
        uint32_t pl = 0u;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            pl |= ((((s[q] >> b) & 0x01010101u) * 0x01020408u) >> 24) << (4 * q);
        gptr(dst)[b] = pl & valid;
    }
}

// The planes of a lane's two adjacent columns, as they are loaded.
template <int B>
struct Columns {
    u32x4 four[B / 2 > 0 ? B / 2 : 1];
    u32x2 two;
    __device__ uint32_t at(int i) const { return i < B / 2 * 4 ? four[i / 4][i % 4] : two[i % 2]; }
};

// One wave per unit of R rows x 128 columns, two adjacent columns a lane.  The
// rows' planes are wave-uniform: scalar loads, and the scalar operand of the
// XOR-OR; the columns' planes and the sums are in registers.  So nothing passes
// through LDS and nearly all issued instructions are the B + 1 of a pair and
// word.  The next group of rows and the next word's columns are loaded ahead
// (without: 5.1 ms in the case below, the waves waiting for scalar loads).  Units
// of a column block j cover the rows up to its last column, so every pair is in
// one; D[row][column] and its mirror are both written.
//
// Bound by the VALU: 32768 rows of n = 50, half prefilled (40 words of 6
// planes), take 3.6 ms: the 7 operations of every pair and word run at 41 T/s.  (One
// instruction a SIMD every four cycles of 2.4 GHz is 39.3; loops of independent
// operations on this card run v_bitop3 and v_bcnt at 33 T/s, v_add at 55.)  Tiles
// of 64 x 64 staged through LDS, 4 x 4 pairs a thread, took 5.06 ms (1024 rows: 70
// us more).
template <int B, int R>
__global__ __launch_bounds__(256) void dist_kernel(const ArgList L) {
    const DistArgs a = arg_of<DistArgs>(L);
    if (a.ctl && a.ctl->stop) return;
    const int t = readfirst((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6)) + a.unit0;
    if (t >= a.unit1) return;
    // unit -> column block j, and the row block within it
    constexpr int kHalf = kDistCols / R / 2;  // kHalf j (j + 1) units before block j
    int j = (int)((sqrtf(4.0f / kHalf * (float)t + 1.0f) - 1.0f) * 0.5f);
    while (kHalf * (j + 1) * (j + 2) <= t) ++j;
    while (kHalf * j * (j + 1) > t) --j;
    j = readfirst(j);
    const int r0 = R * (t - kHalf * j * (j + 1)), c = kDistCols * j + 2 * lane_id();
    if (r0 >= a.m) return;
    // (the pitch is even, so either both of a lane's columns lie within or none is used)
    const uint32_t oc = (uint32_t)min(c, a.pitch - 2) * B;
    constexpr int kG = 4;  // rows per group of scalar loads
    constexpr int kGroups = R / kG;
    const uint32_t wstep = (uint32_t)a.pitch * B;
    uint32_t acc[R][2];
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i][0] = acc[i][1] = 0u;
    Columns<B> col[2];
    uint32_t row[2][kG * B];
    auto columns = [&](Columns<B> &x, const uint32_t *planes) {
        const uint32_t *base = planes + oc;
#pragma unroll
        for (int q = 0; q < B / 2; ++q) x.four[q] = gload4_any(base + 4 * q);
        if constexpr (B & 1)
            x.two = *gptr(reinterpret_cast<const u32x2_any *>(base + 2 * B - 2));
    };
    auto rows = [&](uint32_t (&x)[kG * B], const uint32_t *planes, int g) {
        // (the last rows of the planes again, past the end)
        const auto *pr = cptr(planes + (uint32_t)min(r0 + kG * g, a.pitch - kG) * B);
#pragma unroll
        for (int i = 0; i < kG * B; ++i) x[i] = pr[i];
    };
    // one word; the next group of rows and the next word's columns are on their way
    const uint32_t *at = a.planes;
    auto word = [&](int w, const Columns<B> &now, Columns<B> &next) {
        const uint32_t *const here = at;
        if (w + 1 < a.W) at += wstep;
        columns(next, at);
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            uint32_t(&cur)[kG * B] = row[g & 1];
            // scalar loads return in any order: wait for these before the next are issued
            asm volatile("" ::"s"(cur[0]), "s"(cur[kG * B - 1]));
            if (g + 1 < kGroups)
                rows(row[(g + 1) & 1], here, g + 1);
            else
                rows(row[(g + 1) & 1], at, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < kG; ++i) {
                uint32_t x = cur[i * B] ^ now.at(0), y = cur[i * B] ^ now.at(B);
#pragma unroll
                for (int b = 1; b < B; ++b) {
                    // v_bitop3 with table 0xBE = (s0 ^ s1) | s2
                    x = __builtin_amdgcn_bitop3_b32(cur[i * B + b], now.at(b), x, 0xBE);
                    y = __builtin_amdgcn_bitop3_b32(cur[i * B + b], now.at(B + b), y, 0xBE);
                }
                acc[kG * g + i][0] += (uint32_t)__popc(x);
                acc[kG * g + i][1] += (uint32_t)__popc(y);
                // (v_bcnt adds to its sum; regrouped, two words' counts would need a
                // third addition)
                asm volatile("" : "+v"(acc[kG * g + i][0]), "+v"(acc[kG * g + i][1]));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (a.W > 0) rows(row[0], at, 0);
    if (a.W & 1) {
        columns(col[1], at);
        word(0, col[1], col[0]);
    } else if (a.W > 0) {
        columns(col[0], at);
    }
    for (int w = a.W & 1; w < a.W; w += 2) {
        word(w, col[0], col[1]);
        word(w + 1, col[1], col[0]);
    }
    // rows: two columns a lane, 256 bytes a row and wave
    const bool two = c + 1 < a.m, one = c < a.m;
    const bool whole = r0 + R <= a.m;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int g = i / kG, r = min(r0 + kG * g, a.pitch - kG) + i % kG;
        if (r >= a.m) continue;
        int16_t *d = a.D + (size_t)r * a.ld + c;
        if (two)
            *gptr(reinterpret_cast<u32_any *>(d)) = acc[i][0] | (acc[i][1] << 16);
        else if (one)
            *gptr(d) = (int16_t)acc[i][0];
    }
    // mirror: the R rows of a column are adjacent in its row
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        if (z == 0 ? !one : !two) continue;
        int16_t *d = a.D + (size_t)(c + z) * a.ld + r0;
        if (whole) {
#pragma unroll
            for (int q = 0; q < R / 8; ++q) {
                u32x4 v;
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    v[h] = acc[8 * q + 2 * h][z] | (acc[8 * q + 2 * h + 1][z] << 16);
                *gptr(reinterpret_cast<u32x4_any *>(d) + q) = v;
            }
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int g = i / kG, r = min(r0 + kG * g, a.pitch - kG) + i % kG;
                if (r < a.m) *gptr(a.D + (size_t)(c + z) * a.ld + r) = (int16_t)acc[i][z];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Population update (Alg. 4)
// ---------------------------------------------------------------------------
// close lists: for candidate x, the candidates y != x with spacing*D(x,y) <= |V|
// (those x excludes once accepted); deg[x] counts them, adj keeps the first kAdj.

__global__ __launch_bounds__(256) void close_kernel(const ArgList L) {
    const CloseArgs a = arg_of<CloseArgs>(L);
    if (a.ctl && a.ctl->stop) return;
    const int x = (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (x >= a.m) return;
    const int lane = lane_id();
    const int16_t *row = a.D + (size_t)x * a.ld;
    // spacing * d <= |V| for d up to this (spacing >= 1)
    const int32_t dmax = readfirst((int32_t)min((int64_t)INT16_MAX, (int64_t)a.nv / a.spacing));
    uint32_t cnt = 0;
    // Eight distances per lane and load, four loads in flight.  Few are close:
    // the minimum of the eight decides for the wave whether any has to be
    // looked at.  32768 rows: 376 us, 5.7 TB/s of D (413 us with each distance
    // tested; rows of no multiple of eight were read two bytes at a time).
    auto scan = [&](int y0, const u32x4 &q) {
        typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        i16x2 m2 = __builtin_bit_cast(i16x2, w[0]);
#pragma unroll
        for (int t = 1; t < 4; ++t)
            m2 = __builtin_elementwise_min(m2, __builtin_bit_cast(i16x2, w[t]));
        const int yb = y0 + lane * 8;
        const bool in = yb + 8 <= a.m;
        if (ballot(in && min((int32_t)m2.x, (int32_t)m2.y) <= dmax) == 0ull) return;
        uint32_t fl = 0u;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int32_t d = (int16_t)((w[t >> 1] >> (16 * (t & 1))) & 0xFFFFu);
            fl |= (uint32_t)(in && yb + t != x && d <= dmax) << t;
        }
        // ascending order: lanes in order, then the lane's eight
        uint32_t total;
        uint32_t pos = cnt + wave_excl_scan_dpp((uint32_t)__popc(fl), &total);
        while (fl) {
            const int t = __ffs(fl) - 1;
            fl &= fl - 1u;
            if (pos < (uint32_t)kAdj) *gptr(a.adj + (size_t)x * kAdj + pos) = (uint16_t)(yb + t);
            ++pos;
        }
        cnt += total;
    };
    constexpr int kAhead = 4;  // loads in flight per lane
    const int full = a.m & ~7;
    for (int y0 = 0; y0 < full; y0 += 512 * kAhead) {
        u32x4 q[kAhead];
#pragma unroll
        for (int h = 0; h < kAhead; ++h)
            q[h] = gload4_any(row + min(y0 + 512 * h + lane * 8, full - 8));
#pragma unroll
        for (int h = 0; h < kAhead; ++h) scan(y0 + 512 * h, q[h]);
    }
    const int y = full + lane;
    const bool cl = y < a.m && y != x && (int32_t)*gptr(row + min(y, a.m - 1)) <= dmax;
    const uint64_t msk = ballot(cl);
    const uint32_t pos = cnt + rank_below(msk);
    if (cl && pos < (uint32_t)kAdj) *gptr(a.adj + (size_t)x * kAdj + pos) = (uint16_t)y;
    cnt += (uint32_t)__popcll(msk);
    if (lane == 0) *gptr(a.deg + x) = (int32_t)cnt;
}

// Selection keys of P^all: f << 48 | SELECT draw << 16 | index (the order of
// Alg. 4: e, then a random key, then the index), ~0 beyond m: the four from 4q on.
__device__ __forceinline__ void select_keys(const SelectArgs &a, uint32_t gen, int q,
                                            uint64_t *K) {
    const int x0 = q * 4;
    U4 w{0, 0, 0, 0};
    if (x0 < a.m) w = draw(a.seed_lo, a.seed_hi, 0u, gen, TAG_SELECT, (uint32_t)q);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int x = x0 + t;
        K[t] = (x < a.m) ? (((uint64_t)(uint32_t)a.f_all[x] << 48) |
                            ((uint64_t)word_of(w, t) << 16) | (uint32_t)x)
                         : ~0ull;
    }
}

__device__ __forceinline__ bool select_gen(const SelectArgs &a, uint32_t *gen) {
    int g = a.gen_fixed;
    if (g == 0) {
        if (a.ctl->stop) return false;
        g = a.ctl->gen;
    }
    *gen = (uint32_t)g;
    return true;
}

// Pair i of a bitonic step with partner distance j: lower index.
__device__ __forceinline__ int bitonic_lo(int i, int j) { return ((i & ~(j - 1)) << 1) | (i & (j - 1)); }

// Key sort for populations whose keys exceed LDS: tiles sorted in LDS, then each
// key's place is the sum of its place in every tile (binary searches; the keys
// differ).  Bound by latency: the 66 steps of a tile, then 24 dependent reads.
// 32768 keys: 35 us; a bitonic network over the whole array, tile-local
// steps in LDS, took 95 in ten launches.
constexpr int kSortTile = 2048;

__global__ __launch_bounds__(1024) void sort_tile_kernel(const ArgList L) {
    __shared__ uint64_t t[kSortTile];
    const SelectArgs a = arg_of<SelectArgs>(L);
    uint32_t gen;
    if (!select_gen(a, &gen)) return;
    const int base = (int)blockIdx.x * kSortTile;
    for (int q = (int)threadIdx.x; q < (kSortTile >> 2); q += (int)blockDim.x)
        select_keys(a, gen, (base >> 2) + q, t + 4 * q);
    __syncthreads();
    for (int k = 2; k <= kSortTile; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = (int)threadIdx.x; i < (kSortTile >> 1); i += (int)blockDim.x) {
                const int lo = bitonic_lo(i, j), hi = lo + j;
                const uint64_t x = t[lo], y = t[hi];
                if ((x > y) == ((lo & k) == 0)) {
                    t[lo] = y;
                    t[hi] = x;
                }
            }
            __syncthreads();
        }
    }
    for (int q = (int)threadIdx.x; q < kSortTile; q += (int)blockDim.x) a.keys_g[base + q] = t[q];
}

__global__ __launch_bounds__(256) void sort_rank_kernel(const ArgList L, int tiles) {
    const SelectArgs a = arg_of<SelectArgs>(L);
    uint32_t gen;
    if (!select_gen(a, &gen)) return;
    const int q = (int)(blockIdx.x * blockDim.x + threadIdx.x);  // < tiles * kSortTile
    const uint64_t key = *gptr(a.keys_g + q);
    const int own = q / kSortTile;
    int place = q % kSortTile;
    constexpr int kAhead = 8;  // searches side by side
    for (int t0 = 0; t0 < tiles; t0 += kAhead) {
        int lo[kAhead];
#pragma unroll
        for (int h = 0; h < kAhead; ++h) lo[h] = 0;
        auto tile = [&](int h) { return a.keys_g + (size_t)min(t0 + h, tiles - 1) * kSortTile; };
        for (int step = kSortTile >> 1; step > 0; step >>= 1) {
#pragma unroll
            for (int h = 0; h < kAhead; ++h)
                lo[h] += *gptr(tile(h) + lo[h] + step - 1) < key ? step : 0;
        }
#pragma unroll
        for (int h = 0; h < kAhead; ++h) {
            const int below = lo[h] + (*gptr(tile(h) + lo[h]) < key ? 1 : 0);
            place += t0 + h < tiles && t0 + h != own ? below : 0;
        }
    }
    // (the fill of the last tile ranks past all keys)
    if (place < a.m) *gptr(a.order + place) = (uint16_t)key;
}

// One workgroup: keys (f, SELECT draw, index) sorted (here by a bitonic network
// when they fit LDS), then scanned in that order.  A candidate is accepted iff
// no accepted candidate before it is close to it and the population is not
// full.  The scan takes a window of candidates, one per thread, and decides it
// in rounds: the undecided mark the later ones of the window in their close
// lists; who stays unmarked is accepted and blocks its list; who is blocked
// drops out.  The result is that of deciding one by one: a candidate is only
// accepted once all before it that could block it are decided.  A window ends
// before an unblocked candidate whose close list exceeds kAdj; that one is
// decided alone, its row of D read by all threads.  Rounds are as many as the
// longest chain of candidates each close to the next, about log of the window
// where the draws order them; where f does, they may be all of it.  After
// kRounds one wave decides the rest, 64 at a time on masks: 8192 candidates in
// one chain by f 0.41 ms, by rounds alone 4.4.  (8 rounds before: 0.50; each
// close to the next 13: 1.35, 8 rounds 1.56.)
//
// Bound by the latency of a window's rounds, 5 us each.  32768 candidates in
// families of about eight: 178 us with the keys sorted before; one wave that
// decided 64 candidates at a time, one after the other in a scalar loop, took
// 2.92 ms.  128 candidates: 11.5 us with their sort, from 17.5.
__host__ __device__ inline size_t select_head_bytes(int m, int pow2, bool keys, bool ranks) {
    return ((keys ? (size_t)pow2 * 8 : ranks ? (size_t)m * 2 : 0) + 15) & ~(size_t)15;
}

__device__ __forceinline__ bool is_close(const SelectArgs &a, int16_t d) {
    return a.spacing * (int64_t)d <= (int64_t)a.nv;
}

// Each candidate's place is read per member of a close list: from LDS, or from
// the workspace where LDS is limited to 64 KiB and more than 27900 candidates
// leave no room for them.
constexpr int kRounds = 6;

template <bool RANK_LDS>
__global__ __launch_bounds__(1024) void select_kernel(const ArgList L) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ int s_stop[2], s_any[2], s_na;
    __shared__ uint32_t s_wait[2][32], s_part[16];
    __shared__ uint64_t s_left[16];
    const SelectArgs a = arg_of<SelectArgs>(L);
    uint32_t gen;
    if (!select_gen(a, &gen)) return;
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x, lane = lane_id();
    const int m = a.m, P2 = a.pow2;
    const int nbw = (m + 31) / 32;
    const bool klds = a.keys_in_lds != 0;
    // keys (then the candidates in order, and each candidate's place in it);
    // with the order in global memory the places alone, or nothing
    uint64_t *K = reinterpret_cast<uint64_t *>(lds);
    uint16_t *rank = reinterpret_cast<uint16_t *>(lds);
    uint16_t *order = rank + P2;
    uint32_t *blocked = reinterpret_cast<uint32_t *>(lds + select_head_bytes(m, P2, klds, RANK_LDS));
    auto rank_at = [&](int y) -> int { return RANK_LDS ? (int)rank[y] : (int)*gptr(a.rank_g + y); };
    uint32_t *accb = blocked + nbw;  // accepted, by place
    uint32_t *gpre = accb + nbw;     // accepted before each group of 64 places

    if (klds)
        for (int q = tid; q < (P2 >> 2); q += nthr) select_keys(a, gen, q, K + 4 * q);
    for (int q = tid; q < 2 * nbw; q += nthr) blocked[q] = 0u;
    for (int q = tid; q < m; q += nthr) *gptr(a.pos + q) = -1;
    if (tid < 32) s_wait[0][tid] = s_wait[1][tid] = 0u;
    if (tid < 2) s_stop[tid] = m, s_any[tid] = 0;
    if (tid == 0) s_na = 0;
    __syncthreads();
    if (klds) {
        for (int k = 2; k <= P2; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int i = tid; i < (P2 >> 1); i += nthr) {
                    const int lo = bitonic_lo(i, j), hi = lo + j;
                    const uint64_t x = K[lo], y = K[hi];
                    if ((x > y) == ((lo & k) == 0)) {
                        K[lo] = y;
                        K[hi] = x;
                    }
                }
                __syncthreads();
            }
        }
        constexpr int kPer = 16;  // keys per thread: at most 2^14 keys fit LDS
        uint32_t own[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int r = tid + q * nthr;
            own[q] = r < m ? (uint32_t)(K[r] & 0xFFFFull) : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int r = tid + q * nthr;
            if (r < m) {
                order[r] = (uint16_t)own[q];
                rank[own[q]] = (uint16_t)r;
            }
        }
    } else {
        for (int r = tid; r < m; r += nthr) {
            const int x = *gptr(a.order + r);
            if constexpr (RANK_LDS)
                rank[x] = (uint16_t)r;
            else
                *gptr(a.rank_g + x) = (uint16_t)r;
        }
    }
    __syncthreads();
    auto order_at = [&](int r) -> int {
        return klds ? (int)order[r] : (int)*gptr(a.order + r);
    };
    auto is_blocked = [&](int x) -> bool { return (blocked[x >> 5] >> (x & 31)) & 1u; };

    int w0 = 0, par = 0, b = 0;
    while (w0 < m) {
        const int r = w0 + tid;
        const bool valid = r < m;
        const int x = valid ? order_at(r) : 0;
        const int d = valid ? *gptr(a.deg + x) : 0;
        u32x4 first = {0u, 0u, 0u, 0u};  // the close list's first eight
        const uint8_t *list = reinterpret_cast<const uint8_t *>(a.adj + (size_t)x * kAdj);
        if (d > 0) first = gload4(list);
        bool und = valid && !is_blocked(x);
        const uint64_t lng = ballot(und && d > kAdj);
        if (lane == 0 && lng)
            atomicMin(&s_stop[par], r + (int)__ffsll((unsigned long long)lng) - 1);
        __syncthreads();
        if (s_na >= a.p) break;
        const int end = min(min(w0 + nthr, m), s_stop[par]);
        par ^= 1;
        if (tid == 0) s_stop[par] = m;
        if (end == w0) {
            const int x0 = order_at(w0);
            const int16_t *row = a.D + (size_t)x0 * a.ld;
            auto mark = [&](int y, int16_t dist) {
                if (y != x0 && is_close(a, dist)) atomicOr(&blocked[y >> 5], 1u << (y & 31));
            };
            if ((m & 7) == 0) {
                for (int y = 8 * tid; y < m; y += 8 * nthr) {
                    const u32x4 q = gload4_any(row + y);
                    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                    for (int t = 0; t < 8; ++t)
                        mark(y + t, (int16_t)((w[t >> 1] >> (16 * (t & 1))) & 0xFFFFu));
                }
            } else {
                for (int y = tid; y < m; y += nthr) mark(y, *gptr(row + y));
            }
            __syncthreads();  // all have read s_na
            if (tid == 0) {
                accb[w0 >> 5] |= 1u << (w0 & 31);
                ++s_na;
            }
            ++w0;
            continue;
        }
        und = und && r < end;
        // fn(candidate, place) for the members of a close list after place r
        auto later_of = [&](const uint8_t *list, u32x4 first, int d, int r, auto fn) {
            for (int q0 = 0; q0 < d; q0 += 8) {
                const u32x4 e = q0 ? gload4(list + 2 * q0) : first;
                const uint32_t ew[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int y = (int)((ew[t >> 1] >> (16 * (t & 1))) & 0xFFFFu);
                    if (q0 + t < d) {
                        const int ry = rank_at(y);
                        if (ry > r) fn(y, ry);
                    }
                }
            }
        };
        auto later = [&](auto fn) { later_of(list, first, d, r, fn); };
        bool accepted = false, marks = true;
        for (int round = 0;; ++round) {
            if (und && marks) {
                marks = false;
                later([&](int, int ry) {
                    if (ry < end) {
                        marks = true;
                        atomicOr(&s_wait[b][(ry - w0) >> 5], 1u << ((ry - w0) & 31));
                    }
                });
            }
            if (ballot(und) && lane == 0) s_any[b] = 1;
            __syncthreads();
            if (!s_any[b]) break;
            if (round == kRounds) {
                const uint64_t left = ballot(und);
                if (lane == 0) s_left[tid >> 6] = left;
                __syncthreads();
                if (tid < 32) s_wait[b][tid] = 0u;
                if (tid == 0) s_any[b] = 0;
                for (int w = 0; tid < 64 && w < (nthr >> 6); ++w) {
                    const uint64_t u = s_left[w];
                    if (u == 0ull) continue;
                    const int base = w0 + 64 * w, r2 = base + lane;
                    const bool in = (u >> lane) & 1ull;
                    const int x2 = in ? order_at(r2) : 0, d2 = in ? *gptr(a.deg + x2) : 0;
                    const uint8_t *list2 = reinterpret_cast<const uint8_t *>(a.adj + (size_t)x2 * kAdj);
                    const u32x4 first2 = d2 > 0 ? gload4(list2) : u32x4{0u, 0u, 0u, 0u};
                    // the later ones of the 64 that this one is close to, and
                    // whether there are any beyond
                    uint64_t mk = 0ull;
                    bool far = false;
                    later_of(list2, first2, d2, r2, [&](int, int ry) {
                        if (ry < base + 64)
                            mk |= 1ull << (ry - base);
                        else
                            far = true;
                    });
                    uint64_t todo = ballot(in && !is_blocked(x2)), acc = 0ull;
                    while (todo) {
                        const int i = (int)__builtin_ctzll(todo);
                        acc |= 1ull << i;
                        const uint64_t out = ((uint64_t)readlane_u32((uint32_t)(mk >> 32), i) << 32) |
                                             readlane_u32((uint32_t)mk, i);
                        todo &= ~(out | (1ull << i));
                    }
                    if (far && ((acc >> lane) & 1ull))
                        later_of(list2, first2, d2, r2,
                                 [&](int y, int) { atomicOr(&blocked[y >> 5], 1u << (y & 31)); });
                    if (lane == 0) s_left[w] = acc;
                    PLSE_WAVE_SYNC();
                }
                __syncthreads();
                accepted = accepted || ((s_left[tid >> 6] >> lane) & 1ull);
                break;
            }
            const bool ready = und && !((s_wait[b][tid >> 5] >> (tid & 31)) & 1u);
            if (ready) later([&](int y, int) { atomicOr(&blocked[y >> 5], 1u << (y & 31)); });
            accepted = accepted || ready;
            b ^= 1;
            if (tid < 32) s_wait[b][tid] = 0u;
            if (tid == 0) s_any[b] = 0;
            __syncthreads();
            und = und && !ready && !is_blocked(x);
        }
        const uint64_t accm = ballot(accepted);
        if (accepted) atomicOr(&accb[r >> 5], 1u << (r & 31));
        if (lane == 0 && accm) atomicAdd(&s_na, (int)__popcll(accm));
        w0 = end;
    }
    __syncthreads();
    // accepted candidates in order; the rejected in order complete a short
    // population (all candidates have been scanned then)
    const int ng = (m + 63) / 64;
    auto word = [&](int w) -> uint32_t { return w < nbw ? accb[w] : 0u; };
    uint32_t c = tid < ng ? (uint32_t)(__popc(word(2 * tid)) + __popc(word(2 * tid + 1))) : 0u;
    uint32_t total;
    c = wave_excl_scan_dpp(c, &total);
    if (lane == 0) s_part[tid >> 6] = total;
    __syncthreads();
    for (int w = 0; w < (tid >> 6); ++w) c += s_part[w];
    if (tid < ng) gpre[tid] = c;
    __syncthreads();
    const int na = s_na;
    for (int g = tid >> 6; g < ng; g += nthr >> 6) {
        const int r = 64 * g + lane;
        if (r >= m) continue;
        const uint64_t bits = ((uint64_t)word(2 * g + 1) << 32) | word(2 * g);
        const int before = (int)gpre[g] + (int)rank_below(bits);
        const bool am = (bits >> lane) & 1ull;
        const int at = am ? before : na + r - before;
        if (at < a.p) *gptr(a.acc + at) = order_at(r);
    }
}

// Threads: a window each, and half the keys of the sort.
static int select_threads(int pow2) { return std::min(1024, std::max(64, pow2 / 2)); }

size_t select_lds_bytes(int m, int pow2, bool keys_in_lds, bool ranks_in_lds) {
    return select_head_bytes(m, pow2, keys_in_lds, ranks_in_lds) +
           ((size_t)2 * ((m + 31) / 32) + (size_t)(m + 63) / 64) * 4;
}

// New population P_{t+1} = accepted candidates in acceptance order: rows,
// f, uid ((gen << 32) | slot for members of P'), partner history (empty for
// members of P').  Written to the tmp arrays, then copied back.

__global__ __launch_bounds__(256) void gather_kernel(const ArgList L) {
    const GatherArgs a = arg_of<GatherArgs>(L);
    if (a.ctl->stop) return;
    const int r = (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (r >= a.p) return;
    const int lane = lane_id();
    const int x = min(max(a.acc[r], 0), 2 * a.p - 1);
    const uint4 *src = reinterpret_cast<const uint4 *>(a.S_all + (size_t)x * a.stride);
    uint4 *dst = reinterpret_cast<uint4 *>(a.S_tmp + (size_t)r * a.stride);
    for (int q = lane; q < (a.stride >> 4); q += 64) dst[q] = src[q];
    const bool old = x < a.p;
    if (lane == 0) {
        a.f_tmp[r] = a.f_all[x];
        a.uid_tmp[r] = old ? a.uid[x] : (((uint64_t)(uint32_t)a.ctl->gen << 32) | (uint32_t)(x - a.p));
        a.hc_tmp[r] = old ? a.hc[x] : 0;
        *gptr(a.pos + x) = r;
    }
    if (old) a.hist_tmp[(size_t)r * kHist + lane] = a.hist[(size_t)x * kHist + lane];
}

__global__ __launch_bounds__(256) void copyback_kernel(const ArgList L) {
    const GatherArgs a = arg_of<GatherArgs>(L);
    if (a.ctl->stop) return;
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t nq = (size_t)a.p * (a.stride >> 4);
    uint4 *S = reinterpret_cast<uint4 *>(const_cast<uint8_t *>(a.S_all));
    for (size_t q = t; q < nq; q += (size_t)gridDim.x * blockDim.x)
        S[q] = reinterpret_cast<const uint4 *>(a.S_tmp)[q];
    uint64_t *hist = const_cast<uint64_t *>(a.hist);
    for (size_t q = t; q < (size_t)a.p * kHist; q += (size_t)gridDim.x * blockDim.x)
        hist[q] = a.hist_tmp[q];
    if (t < (size_t)a.p) {
        const_cast<int32_t *>(a.f_all)[t] = a.f_tmp[t];
        const_cast<uint64_t *>(a.uid)[t] = a.uid_tmp[t];
        const_cast<int32_t *>(a.hc)[t] = a.hc_tmp[t];
    }
}

// ---------------------------------------------------------------------------
// Parent matching (Section 3.5.1): nearest neighbour (D, then slot) among the
// individuals not yet crossed with S_i; plain nearest neighbour when all are.
// uid -> slot through an open-addressing table rebuilt every generation.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t hash_uid(uint64_t u) {
    u ^= u >> 33;
    u *= 0xFF51AFD7ED558CCDull;
    u ^= u >> 33;
    return (uint32_t)u;
}

// Words of an individual's bits of excluded entries of its row.
__host__ __device__ inline int match_words(int cnt) { return (cnt + 31) / 32; }

__global__ void hash_clear_kernel(const ArgList L) {
    const HashArgs a = arg_of<HashArgs>(L);
    if (a.ctl && a.ctl->stop) return;
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    for (int q = t; q < a.hsize; q += gridDim.x * blockDim.x) a.hkeys[q] = ~0ull;
}

__global__ void hash_insert_kernel(const ArgList L) {
    const HashArgs a = arg_of<HashArgs>(L);
    if (a.ctl && a.ctl->stop) return;
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= a.p) return;
    const uint64_t u = a.uid[i];
    uint32_t h = hash_uid(u) & (uint32_t)(a.hsize - 1);
    for (;;) {
        const unsigned long long prev =
            atomicCAS((unsigned long long *)&a.hkeys[h], ~0ull, (unsigned long long)u);
        if (prev == ~0ull || prev == u) {
            a.hvals[h] = i;
            return;
        }
        h = (h + 1) & (uint32_t)(a.hsize - 1);
    }
}

// One wave per individual.  Its row of D is read eight distances a lane and
// load, each made the key d << 16 | j (j < 2^15) whose minimum names the
// partner.  Excluded entries (the history, and the individual itself) are bits
// in the row's order, one byte per load, so that the loop has four operations
// an entry and no further lookup.  Bound by the reads of D, four loads of a lane
// in flight: 16384 rows of 16384 take 106 us (5.1 TB/s), one load after another
// 125; two-byte loads, 64-bit keys and a lookup per entry took 410.
template <bool IDX>
__device__ __forceinline__ uint32_t nearest(const MatchArgs &a, const int16_t *row,
                                            const uint32_t *excl) {
    const int lane = lane_id();
    const int cnt = IDX ? a.m : a.p;
    const uint8_t *ex8 = reinterpret_cast<const uint8_t *>(excl);
    uint32_t lb = 0xFFFFFFFFu;
    struct Eight {
        u32x4 d, pa, pb;
        uint32_t ex;
    };
    auto load = [&](int x0) {
        Eight e{gload4_any(row + x0), {0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}, ex8[x0 >> 3]};
        if constexpr (IDX) e.pa = gload4(a.pos + x0), e.pb = gload4(a.pos + x0 + 4);
        return e;
    };
    auto scan = [&](int x0, const Eight &e) {
        const uint32_t w[4] = {e.d.x, e.d.y, e.d.z, e.d.w};
        const uint32_t js[8] = {e.pa.x, e.pa.y, e.pa.z, e.pa.w, e.pb.x, e.pb.y, e.pb.z, e.pb.w};
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            // pos is -1 for candidates not selected: a key of ~0
            const uint32_t j = IDX ? js[t] : (uint32_t)(x0 + t);
            const uint32_t d = (t & 1) ? w[t >> 1] & 0xFFFF0000u : w[t >> 1] << 16;
            const uint32_t out = (uint32_t)((int32_t)(e.ex << (31 - t)) >> 31);
            lb = min(lb, d | j | out);
        }
    };
    // loads of D in flight per lane (two beside the map's: with four, 122 registers
    // leave too few waves, and short rows lose 6 %)
    constexpr int kAhead = IDX ? 2 : 4;
    int x0 = lane * 8;
    for (; x0 - lane * 8 + 512 * kAhead <= cnt; x0 += 512 * kAhead) {
        Eight e[kAhead];
#pragma unroll
        for (int h = 0; h < kAhead; ++h) e[h] = load(x0 + 512 * h);
#pragma unroll
        for (int h = 0; h < kAhead; ++h) scan(x0 + 512 * h, e[h]);
    }
#pragma unroll 4
    for (; x0 + 8 <= cnt; x0 += 512) scan(x0, load(x0));
    const int x = (cnt & ~7) + lane;
    if (x < cnt && !((excl[x >> 5] >> (x & 31)) & 1u)) {
        const uint32_t j = IDX ? (uint32_t)*gptr(a.pos + x) : (uint32_t)x;
        lb = min(lb, ((uint32_t)(uint16_t)*gptr(row + x) << 16) | j);
    }
    return wave_min_u32_dpp(lb);
}

__global__ __launch_bounds__(256) void match_kernel(const ArgList L) {
    extern __shared__ __align__(16) uint8_t lds[];
    const MatchArgs a = arg_of<MatchArgs>(L);
    if (a.ctl && a.ctl->stop) return;
    const int wv = (int)(threadIdx.x >> 6), lane = lane_id();
    const int i = (int)blockIdx.x * 4 + wv;
    const int nbw = match_words(a.idx ? a.m : a.p);
    uint32_t *excl = reinterpret_cast<uint32_t *>(lds) + (size_t)wv * nbw;
    if (i >= a.p) return;
    const int hcount = max(*gptr(a.hc + i), 0);
    const int ai = a.idx ? *gptr(a.idx + i) : i;
    const int16_t *row = a.D + (size_t)ai * a.ld;
    uint32_t best = 0xFFFFFFFFu;
    if (a.mode == 1) {
        // random matching (Section 5.3): uniform over the other p - 1
        int gen = a.gen_fixed;
        if (gen == 0) gen = a.ctl->gen;
        const U4 w = draw(a.seed_lo, a.seed_hi, (uint32_t)i, (uint32_t)gen, TAG_MATCH, 0u);
        int j = (int)(((uint64_t)w.x * (uint64_t)(uint32_t)(a.p - 1)) >> 32);
        j += (j >= i) ? 1 : 0;
        const int aj = a.idx ? *gptr(a.idx + j) : j;
        best = ((uint32_t)(uint16_t)*gptr(row + aj) << 16) | (uint32_t)j;
    } else {
        for (int pass = 0; pass < 2 && best == 0xFFFFFFFFu; ++pass) {
            for (int q = lane; q < nbw; q += 64) excl[q] = 0u;
            PLSE_WAVE_SYNC();
            const int nh = pass == 0 ? min(hcount, a.hist_len) : 0;
            for (int t = lane; t < nh; t += 64) {
                const uint64_t u = *gptr(a.hist + (size_t)i * kHist + t);
                uint32_t h = hash_uid(u) & (uint32_t)(a.hsize - 1);
                for (;;) {
                    const uint64_t k = *gptr(a.hkeys + h);
                    if (k == u) {
                        const int s = *gptr(a.hvals + h);
                        const int x = a.idx ? *gptr(a.idx + s) : s;
                        atomicOr(&excl[x >> 5], 1u << (x & 31));
                        break;
                    }
                    if (k == ~0ull) break;
                    h = (h + 1) & (uint32_t)(a.hsize - 1);
                }
            }
            if (lane == 0) atomicOr(&excl[ai >> 5], 1u << (ai & 31));
            PLSE_WAVE_SYNC();
            best = a.idx ? nearest<true>(a, row, excl) : nearest<false>(a, row, excl);
        }
    }
    if (lane == 0) {
        const int j = (int)(best & 0xFFFFu);
        a.partner[i] = j;
        a.dpart[i] = (int32_t)(best >> 16);
        if (a.hist_len > 0) {
            const int pos = hcount % a.hist_len;
            a.hist[(size_t)i * kHist + pos] = a.uid[j];
            int nc = hcount + 1;
            if (nc >= 2 * a.hist_len) nc -= a.hist_len;
            a.hc[i] = nc;
        }
    }
}

// ---------------------------------------------------------------------------
// AUX crossover (Alg. 5): vertex v keeps S_i(v) when its XOVER draw is below
// thr = floor((beta*D - |V|) 2^32 / (beta*D)) (p_ij of Eq. 9 in 2^-32
// units; 0 when beta*D <= |V|), else takes S_j(v).  One wave per child, four
// vertices per lane step (one Philox block).
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void aux_kernel(const ArgList L) {
    const AuxArgs a = arg_of<AuxArgs>(L);
    int gen = a.gen_fixed;
    if (gen == 0) {
        if (a.ctl->stop) return;
        gen = a.ctl->gen;
    }
    const int i = (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (i >= a.p) return;
    const int lane = lane_id();
    int j = a.partner[i];
    if (j < 0 || j >= a.p) j = i;  // out-of-range partner: no crossover
    const uint64_t bd = (uint64_t)a.beta_num * (uint64_t)(uint32_t)a.dpart[i];
    const uint64_t bv = (uint64_t)a.beta_den * (uint64_t)a.nv;
    // UX fixes p_ij at 1/2 (Section 3.5.2); without crossover the offspring
    // copies its first parent (Section 5.2)
    const uint64_t thr = a.mode == 1   ? (1ull << 31)
                         : a.mode == 2 ? (1ull << 32)
                                       : ((bd <= bv) ? 0ull : frac_shift32(bd - bv, bd));
    const uint32_t *si = reinterpret_cast<const uint32_t *>(a.S + (size_t)i * a.stride);
    const uint32_t *sj = reinterpret_cast<const uint32_t *>(a.S + (size_t)j * a.stride);
    uint32_t *so = reinterpret_cast<uint32_t *>(a.S_off + (size_t)i * a.stride);
    const int nq = a.stride >> 2;
    for (int q = lane; q < nq; q += 64) {
        uint32_t out = 0u;
        if (4 * q < a.nv) {
            const U4 w = draw(a.seed_lo, a.seed_hi, (uint32_t)i, (uint32_t)gen, TAG_XOVER,
                              (uint32_t)q);
            const uint32_t x = si[q], y = sj[q];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (4 * q + t < a.nv) {
                    const uint32_t b = ((uint64_t)word_of(w, t) < thr) ? x : y;
                    out |= b & (0xFFu << (8 * t));
                }
            }
        }
        so[q] = out;
    }
}

hipError_t launch_ctl_reset(const ArgList &L, int count, hipStream_t stream) {
    hipLaunchKernelGGL(ctl_reset_kernel, dim3(1, count), dim3(64), 0, stream, L);
    return hipGetLastError();
}

hipError_t launch_gen_begin(const ArgList &L, int count, hipStream_t stream) {
    hipLaunchKernelGGL(gen_begin_kernel, dim3(1, count), dim3(64), 0, stream, L);
    return hipGetLastError();
}

hipError_t launch_pop_setup(const ArgList &L, int count, hipStream_t stream) {
    hipLaunchKernelGGL(pop_setup_kernel, dim3(512, count), dim3(256), 0, stream, L);
    return hipGetLastError();
}

hipError_t launch_best(const ArgList &L, int count, hipStream_t stream) {
    hipLaunchKernelGGL(best_kernel, dim3(1, count), dim3(1024), 0, stream, L);
    return hipGetLastError();
}

hipError_t launch_pack(const ArgList &L, int count, size_t max_threads, hipStream_t stream) {
    // at least one block: an instance without vertices packs nothing
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)std::max<size_t>(1, (max_threads + 255) / 256), count), dim3(256),
                       0, stream, L);
    return hipGetLastError();
}

hipError_t launch_dist(const ArgList &L, int count, long units, int B, int rows,
                       hipStream_t stream) {
    if (units <= 0) return hipSuccess;
    const dim3 grid((unsigned)((units + 3) / 4), count);
    auto go = [&](auto kernel_short, auto kernel_tall) {
        void (*k)(const ArgList) = rows == kDistShort ? kernel_short : kernel_tall;
        hipLaunchKernelGGL(k, grid, 256, 0, stream, L);
        return hipGetLastError();
    };
    switch (B) {
        case 1: return go(dist_kernel<1, kDistShort>, dist_kernel<1, kDistTall>);
        case 2: return go(dist_kernel<2, kDistShort>, dist_kernel<2, kDistTall>);
        case 3: return go(dist_kernel<3, kDistShort>, dist_kernel<3, kDistTall>);
        case 4: return go(dist_kernel<4, kDistShort>, dist_kernel<4, kDistTall>);
        case 5: return go(dist_kernel<5, kDistShort>, dist_kernel<5, kDistTall>);
        case 6: return go(dist_kernel<6, kDistShort>, dist_kernel<6, kDistTall>);
        case 7: return go(dist_kernel<7, kDistShort>, dist_kernel<7, kDistTall>);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_close(const ArgList &L, int count, int m, hipStream_t stream) {
    hipLaunchKernelGGL(close_kernel, dim3((m + 3) / 4, count), dim3(256), 0, stream, L);
    return hipGetLastError();
}

hipError_t launch_select(const ArgList &L, int count, size_t lds, int m, int pow2,
                         bool keys_in_lds, bool ranks_in_lds, hipStream_t stream) {
    if (!keys_in_lds) {
        const int tiles = (m + kSortTile - 1) / kSortTile;
        if (tiles * kSortTile > pow2) return hipErrorInvalidValue;
        hipLaunchKernelGGL(sort_tile_kernel, dim3(tiles, count), dim3(1024), 0, stream, L);
        hipLaunchKernelGGL(sort_rank_kernel, dim3(tiles * (kSortTile / 256), count), dim3(256), 0,
                           stream, L, tiles);
    }
    void (*k)(const ArgList) = ranks_in_lds ? select_kernel<true> : select_kernel<false>;
    hipLaunchKernelGGL(k, dim3(1, count), dim3(select_threads(pow2)), lds, stream, L);
    return hipGetLastError();
}

hipError_t launch_gather(const ArgList &L, int count, int p, hipStream_t stream) {
    hipLaunchKernelGGL(gather_kernel, dim3((p + 3) / 4, count), dim3(256), 0, stream, L);
    hipLaunchKernelGGL(copyback_kernel, dim3(256, count), dim3(256), 0, stream, L);
    return hipGetLastError();
}

hipError_t launch_hash(const ArgList &L, int count, int p, int hsize, hipStream_t stream) {
    hipLaunchKernelGGL(hash_clear_kernel, dim3((hsize + 255) / 256, count), dim3(256), 0, stream,
                       L);
    hipLaunchKernelGGL(hash_insert_kernel, dim3((p + 255) / 256, count), dim3(256), 0, stream, L);
    return hipGetLastError();
}

hipError_t launch_match(const ArgList &L, int count, int p, int cnt, hipStream_t stream) {
    const size_t lds = (size_t)4 * match_words(cnt) * 4;
    hipLaunchKernelGGL(match_kernel, dim3((p + 3) / 4, count), dim3(256), lds, stream, L);
    return hipGetLastError();
}

hipError_t launch_aux(const ArgList &L, int count, int p, hipStream_t stream) {
    hipLaunchKernelGGL(aux_kernel, dim3((p + 3) / 4, count), dim3(256), 0, stream, L);
    return hipGetLastError();
}

hipError_t evo_set_lds_limit(int bytes) {
    hipError_t e = set_dynamic_lds_limit((const void *)select_kernel<true>, bytes);
    if (e != hipSuccess) return e;
    return set_dynamic_lds_limit((const void *)match_kernel, bytes);
}

}  // namespace plse
