// k_init.hip -- initial population (Section 3.2: "initialized at random in
// parallel"), one wave per individual.  Reading: a randomised greedy legal
// colouring.  Vertices are visited in the order of their INIT_ORDER draws
// (ties by id), each taking a uniformly drawn colour of D*(v) not used in its
// row or column so far.
//
// The order: the draws are uniform, so a counting sort by their top bits leaves
// about one vertex per bucket; a vertex's place is its bucket's start plus the
// members with a smaller (draw, id).  The walk takes the next 64 vertices of
// the order at once, one per lane.  A lane may choose its colour when no
// earlier undone lane shares its row or column, since only those change the
// colours it may take; lanes that go together share no line, so each updates
// its two lines alone.
//
// Bound by VALU issue (about 15 instructions a vertex, a third of them the two
// Philox draws).  16384 individuals of n = 50, half prefilled (|V| = 1250):
// 500 us.  A bitonic sort of the keys and a walk of one lane, vertex by vertex,
// took 5.6 ms: 66 passes over the keys, then 1250 dependent steps of memory
// latency with 63 lanes idle.
#include "device_common.h"
#include "kernels.h"

namespace plse {

// The idx-th set bit (from 0) of w, which has more than idx of them.
__device__ __forceinline__ uint32_t nth_set_bit(uint32_t w, uint32_t idx) {
    uint32_t at = 0u;
#pragma unroll
    for (int h = 16; h >= 1; h >>= 1) {
        const uint32_t c = (uint32_t)__popc((w >> at) & ((1u << h) - 1u));
        const bool up = idx >= c;
        idx -= up ? c : 0u;
        at += up ? (uint32_t)h : 0u;
    }
    return at;
}

// Walks the order, W 32-bit words of colours per line (orders up to 31, 63 and
// 127).  `used`: W words per row, then per column, zero; `pend`: one 64-bit
// word per line.  Returns the lane's count of vertices left uncoloured.
template <int W>
__device__ __forceinline__ uint32_t greedy_walk(const InitArgs &a, int ind, const uint16_t *order,
                                                uint32_t *used, uint64_t *pend, uint8_t *S) {
    const DevInstance &I = a.I;
    const int lane = lane_id(), nv = I.nv, n = I.n;
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t zeros = 0u;
    // tables of the batch, loaded one batch ahead
    uint32_t v = 0u, rc = 0u;
    u32x4 dm = {0u, 0u, 0u, 0u};
    auto fetch = [&](int t) {
        if (t >= nv) return;
        v = order[t];
        rc = gptr(I.vrc)[v];
        dm = gload4(static_cast<const uint8_t *>(I.vrec) + 32u * v);
    };
    fetch(lane);
    for (int t0 = 0; t0 < nv; t0 += 64) {
        const bool in = t0 + lane < nv;
        const uint32_t bv = v, r = rc & 0xFFu, c = (uint32_t)n + (rc >> 8);
        const uint32_t dom[4] = {dm[0], dm[1], dm[2], dm[3]};
        fetch(t0 + 64 + lane);
        const uint32_t pw = draw(a.seed_lo, a.seed_hi, (uint32_t)ind, 0u, TAG_INIT_PICK,
                                 (uint32_t)(t0 + lane)).x;
        if (in) pend[r] = 0ull, pend[c] = 0ull;
        PLSE_WAVE_SYNC();
        if (in) {
            atomicOr(reinterpret_cast<unsigned long long *>(pend + r), 1ull << lane);
            atomicOr(reinterpret_cast<unsigned long long *>(pend + c), 1ull << lane);
        }
        PLSE_WAVE_SYNC();
        // earlier lanes of the batch in the vertex's lines
        const uint64_t pred = in ? (pend[r] | pend[c]) & below : 0ull;
        uint64_t todo = ballot(in);
        while (todo) {
            const bool go = ((todo >> lane) & 1ull) && (pred & todo) == 0ull;
            todo &= ~ballot(go);
            if (go) {
                uint32_t leg[W], cnt = 0u;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    leg[w] = dom[w] & ~(used[r * W + w] | used[c * W + w]);
                    cnt += (uint32_t)__popc(leg[w]);
                }
                uint32_t idx = scale32(pw, cnt), word = leg[0], at = 0u;
#pragma unroll
                for (int w = 0; w + 1 < W; ++w) {
                    const uint32_t k = (uint32_t)__popc(word);
                    const bool up = at == 32u * (uint32_t)w && idx >= k;
                    idx -= up ? k : 0u;
                    word = up ? leg[w + 1] : word;
                    at = up ? 32u * (uint32_t)(w + 1) : at;
                }
                const uint32_t b = nth_set_bit(word, idx);
                if (cnt != 0u) {
                    const uint32_t w = at >> 5, bit = 1u << b;
                    used[r * W + w] |= bit;
                    used[c * W + w] |= bit;
                } else {
                    ++zeros;
                }
                S[bv] = (uint8_t)(cnt != 0u ? at + b : 0u);
            }
            PLSE_WAVE_SYNC();
        }
    }
    return zeros;
}

__global__ __launch_bounds__(64) void init_kernel(const ArgList L) {
    extern __shared__ __align__(16) uint8_t lds[];
    const InitArgs a = arg_of<InitArgs>(L);
    const DevInstance &I = a.I;
    const int ind = (int)blockIdx.x;
    const int lane = lane_id();
    const int nv = I.nv, n = I.n;
    // draws (then the colours), vertices by bucket, vertices in order, and the
    // buckets' ends (then the lines' masks)
    const int nvp = I.stride;  // nv rounded up
    uint32_t *dr = reinterpret_cast<uint32_t *>(lds);
    uint8_t *S = lds;
    uint16_t *bucket = reinterpret_cast<uint16_t *>(dr + nvp);
    uint16_t *order = bucket + nvp;
    uint32_t *ends = reinterpret_cast<uint32_t *>(order + nvp);
    const int nb = 1 << a.log2_buckets, shift = 32 - a.log2_buckets;

    for (int q = lane; q < nb; q += 64) ends[q] = 0u;
    PLSE_WAVE_SYNC();
    for (int q = lane; 4 * q < nv; q += 64) {
        const U4 w = draw(a.seed_lo, a.seed_hi, (uint32_t)ind, 0u, TAG_INIT_ORDER, (uint32_t)q);
        *reinterpret_cast<uint4 *>(dr + 4 * q) = uint4{w.x, w.y, w.z, w.w};
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (4 * q + t < nv) atomicAdd(ends + (word_of(w, t) >> shift), 1u);
    }
    PLSE_WAVE_SYNC();
    // counts to starts; placing the vertices then turns starts to ends
    uint32_t carry = 0u;
    for (int q = lane; q < nb; q += 64) {
        uint32_t total;
        const uint32_t x = wave_excl_scan_dpp(ends[q], &total);
        ends[q] = carry + x;
        carry += total;
    }
    PLSE_WAVE_SYNC();
    for (int v = lane; v < nv; v += 64)
        bucket[atomicAdd(ends + (dr[v] >> shift), 1u)] = (uint16_t)v;
    PLSE_WAVE_SYNC();
    for (int i = lane; i < nv; i += 64) {
        const uint32_t v = bucket[i], d = dr[v], b = d >> shift;
        const uint32_t lo = b ? ends[b - 1u] : 0u, hi = ends[b];
        uint32_t at = lo;
        for (uint32_t j = lo; j < hi; ++j) {
            const uint32_t u = bucket[j], e = dr[u];
            at += (e < d || (e == d && u < v)) ? 1u : 0u;
        }
        order[at] = (uint16_t)v;
    }
    PLSE_WAVE_SYNC();
    // the row's padding is 0
    for (int v = nv + lane; v < nvp; v += 64) S[v] = 0u;
    uint64_t *pend = reinterpret_cast<uint64_t *>(ends);  // [2n]
    uint32_t *used = reinterpret_cast<uint32_t *>(pend + 2 * n);
    for (int q = lane; q < 8 * n; q += 64) used[q] = 0u;
    PLSE_WAVE_SYNC();
    uint32_t zeros;
    if (n < 32)
        zeros = greedy_walk<1>(a, ind, order, used, pend, S);
    else if (n < 64)
        zeros = greedy_walk<2>(a, ind, order, used, pend, S);
    else
        zeros = greedy_walk<4>(a, ind, order, used, pend, S);
    PLSE_WAVE_SYNC();
    uint8_t *dst = a.S + (size_t)ind * nvp;
    for (int q = lane; q < (nvp >> 4); q += 64)
        gstore4(dst + 16 * q, *reinterpret_cast<const u32x4 *>(S + 16 * q));
    zeros = wave_sum_u32_dpp(zeros);
    if (lane == 0) a.f[ind] = (int32_t)zeros;
}

// About one vertex per bucket; 2^10 buckets at most, so that the counters stay
// small beside the vertices' 8 bytes each (2^8 to 2^11 buckets take the same
// time within 5 % at |V| = 1250).
int init_log2_buckets(int nv) {
    int b = 6;
    while (b < 10 && (1 << b) < nv) ++b;
    return b;
}

size_t init_lds_bytes(const DevInstance &I) {
    const size_t buckets = (size_t)4 << init_log2_buckets(I.nv);
    const size_t lines = (size_t)2 * I.n * (8 + 16);
    return (size_t)8 * I.stride + (buckets > lines ? buckets : lines);
}

hipError_t launch_init(const ArgList &L, int count, int p, size_t lds, hipStream_t stream) {
    hipLaunchKernelGGL(init_kernel, dim3(p, count), dim3(64), lds, stream, L);
    return hipGetLastError();
}

hipError_t init_set_lds_limit(int bytes) {
    return set_dynamic_lds_limit((const void *)init_kernel, bytes);
}

}  // namespace plse
