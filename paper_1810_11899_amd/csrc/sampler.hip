// Graph sampling and GCN construction on the sample (Sec. IV; Alg. 1-5):
//
//   frontier_kernel  frontier sampling with the Dashboard (Sec. IV-A/IV-B,
//                    Alg. 2-4); one wavefront per sampler instance, the 64
//                    lanes are the p processors of the probing step and of
//                    the Dashboard updates (intra-subgraph parallelism), one
//                    workgroup per sampler (inter-subgraph parallelism,
//                    Sec. IV-C)
//   induce kernels   the subgraph of G induced by each sampled vertex list, as
//                    a mean-normalised CSR with local ids, for a batch of
//                    samples at once (the last step of Alg. 2 / Alg. 3)
//   gather kernel    feature (or label) rows of the sampled vertices
//
// Dashboard layout (LDS, per sampler): db[entries] holds, for every entry, the
// Index-Array slot it belongs to (16 bits); slot k holds its vertex, the start
// of its neighbour list in G and its degree, with the live flag in bit 31.
// Popping a vertex clears one flag, which invalidates all of its entries at
// once (the paper's Alg. 4 writes INV into each of them), and reads no global
// memory; a step then costs two dependent global loads (the chosen neighbour,
// then its row bounds).  Random numbers: Philox4x64-10 (Salmon et al.,
// SC 2011) keyed by (seed, sampler id); each block gives four draws.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "gcn_sampler.h"

namespace gcn {
namespace {

constexpr size_t kSamplerMaxLds = 160 * 1024;  // LDS of one gfx950 CU

constexpr int kSampThreads = 64;          // one wavefront per sampler
constexpr uint32_t kLive = 0x80000000u;
constexpr uint64_t kKindRoot = 1, kKindProbe = 2, kKindNeigh = 3;
constexpr int64_t kProbeRoundLimit = 1 << 20;

// ---------------------------------------------------------------- Philox
// One Philox4x64-10 block: counter (c0, kind, c2, 0), key (seed, sampler id).
struct Words {
    uint64_t w0, w1, w2, w3;
    __device__ __forceinline__ uint64_t get(uint32_t i) const {
        const uint64_t lo = (i & 1u) ? w1 : w0, hi = (i & 1u) ? w3 : w2;
        return (i & 2u) ? hi : lo;
    }
};
__device__ __forceinline__ Words philox(uint64_t c0, uint64_t kind, uint64_t c2, uint64_t seed, uint64_t sid) {
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
    uint64_t x0 = c0, x1 = kind, x2 = c2, x3 = 0, k0 = seed, k1 = sid;
#pragma unroll 1    // (inlined at a dozen places: unrolled, the sampler outgrows the instruction cache)
    for (int r = 0; r < 10; ++r) {
        const uint64_t lo0 = M0 * x0, hi0 = __umul64hi(M0, x0);
        const uint64_t lo1 = M1 * x2, hi1 = __umul64hi(M1, x2);
        x0 = hi1 ^ x1 ^ k0;
        x1 = lo1;
        x2 = hi0 ^ x3 ^ k1;
        x3 = lo0;
        k0 += W0;
        k1 += W1;
    }
    return Words{x0, x1, x2, x3};
}
// integer uniform on [0, n): high word of r * n
__device__ __forceinline__ int64_t below(uint64_t r, int64_t n) { return (int64_t)__umul64hi(r, (uint64_t)n); }

// the same for n < 2^32, in two 32-bit products
__device__ __forceinline__ uint32_t below32(uint64_t r, uint32_t n) {
    return (uint32_t)(((r >> 32) * n + (((r & 0xFFFFFFFFull) * n) >> 32)) >> 32);
}
// a value all lanes share, in a scalar register
__device__ __forceinline__ int32_t uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    return (uint64_t)(uint32_t)uniform((int32_t)(x >> 32)) << 32 | (uint32_t)uniform((int32_t)x);
}

__device__ __forceinline__ int32_t weight_of_deg(uint32_t d, int32_t cap) {
    return (cap > 0 && (int32_t)d > cap) ? cap : (int32_t)d;
}

// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ int64_t wave_incl_scan(int64_t x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    return x;
}

// ------------------------------------------------------- frontier sampling
struct SampArgs {
    int32_t nV;
    const int32_t *indptr;
    const int32_t *indices;
    int32_t m, n, db_cap, ia_cap, cap;
    uint64_t seed;
    int64_t first_sampler;
    int32_t *vertices;   // [S][n]
    int32_t *counts;     // [S]
    int32_t *status;     // [S]
};

// Index-Array slots in LDS: vertex, start of its neighbour list in G, and
// degree with the live flag (the slot keeps what a pop needs, so popping
// reads no global memory).
struct Slots {
    int2 *bd;        // x: start of the neighbour list, y: degree | kLive
    int32_t *v;
};

// Cleanup (Alg. 4): keep the live slots in slot order, renumber them, and
// rebuild the Dashboard from their weights.  Whole wavefront.
__device__ void dashboard_cleanup(uint16_t *db, Slots sl, int32_t cap, int32_t &s, int32_t &used) {
    const int lane = threadIdx.x;
    int32_t ns = 0;
    for (int32_t base = 0; base < s; base += 64) {
        const int32_t k = base + lane;
        const bool in = k < s;
        const int32_t v = in ? sl.v[k] : 0;
        const int2 bd = in ? sl.bd[k] : make_int2(0, 0);
        const bool live = in && ((uint32_t)bd.y & kLive);
        const uint64_t mask = __ballot(live);
        const int rank = __popcll(mask & ((1ull << lane) - 1ull));
        __syncthreads();            // every lane has read its slot before any moves
        if (live) {
            sl.v[ns + rank] = v;
            sl.bd[ns + rank] = bd;
        }
        ns += __popcll(mask);
        __syncthreads();
    }
    s = ns;
    int64_t off = 0;
    for (int32_t base = 0; base < ns; base += 64) {
        const int32_t k = base + lane;
        const int32_t w = k < ns ? weight_of_deg((uint32_t)sl.bd[k].y & ~kLive, cap) : 0;
        const int64_t incl = wave_incl_scan(w);
        const int64_t start = off + incl - w;
        for (int32_t e = 0; e < w; ++e) db[start + e] = (uint16_t)k;
        off += __shfl(incl, 63, 64);
    }
    used = uniform((int32_t)off);
    __syncthreads();
}

template <bool CAPPED>
__global__ __launch_bounds__(kSampThreads) void frontier_kernel(SampArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    Slots sl;
    sl.bd = (int2 *)lds;                                // [ia_cap]
    sl.v = (int32_t *)(sl.bd + a.ia_cap);               // [ia_cap]
    uint16_t *db = (uint16_t *)(sl.v + a.ia_cap);       // Dashboard [db_cap]
    const int lane = threadIdx.x;
    const uint64_t sid = (uint64_t)(a.first_sampler + blockIdx.x);
    int32_t *out = a.vertices + (int64_t)blockIdx.x * a.n;
    int status = GCN_SAMPLE_OK;
    int32_t count = 0;

    // ---- roots: m distinct vertices; candidate t is kept unless it repeats an
    // earlier root (the lanes of a round take candidates t = 64 r + lane in order)
    {
        const uint64_t limit = 64ull * (uint64_t)a.m + 65536ull;
        int32_t got = 0;
        for (uint64_t base = 0; got < a.m; base += 64) {
            if (base >= limit) { status = GCN_SAMPLE_ROOT_LIMIT; break; }
            const uint64_t t = base + lane;
            const int32_t c = (int32_t)below(philox(t, kKindRoot, 0, a.seed, sid).w0, a.nV);
            bool dup = t >= limit;
            for (int32_t k = 0; k < got && !dup; ++k) dup = (sl.v[k] == c);
            for (int j = 0; j < 64; ++j) {
                const int32_t cj = __shfl(c, j, 64);
                if (j < lane && cj == c) dup = true;
            }
            const uint64_t mask = __ballot(!dup);
            const int rank = __popcll(mask & ((1ull << lane) - 1ull));
            if (!dup && got + rank < a.m) {
                sl.v[got + rank] = c;
                out[got + rank] = c;
            }
            got += min(__popcll(mask), a.m - got);
            __syncthreads();
        }
        count = got;
    }

    int32_t used = 0, live_weight = 0;   // at most db_cap entries
    int32_t s = 0;
    if (status == GCN_SAMPLE_OK) {
        // ---- Dashboard from the roots (Alg. 3, initialisation)
        for (int32_t base = 0; base < a.m; base += 64) {
            const int32_t k = base + lane;
            int32_t b = 0;
            uint32_t d = 0;
            if (k < a.m) {
                const int32_t v = sl.v[k];
                b = a.indptr[v];
                d = (uint32_t)(a.indptr[v + 1] - b);
            }
            const int32_t w = weight_of_deg(d, a.cap);
            const int64_t incl = wave_incl_scan(w);
            const int64_t total = __shfl(incl, 63, 64);
            const bool over = __builtin_amdgcn_readfirstlane((int)(used + total > a.db_cap)) != 0;
            if (over) { status = GCN_SAMPLE_OVERFLOW; break; }
            const int64_t start = used + incl - w;
            if (k < a.m) {
                sl.bd[k] = make_int2(b, (int32_t)(d | kLive));
                for (int32_t e = 0; e < w; ++e) db[start + e] = (uint16_t)k;
            }
            used += uniform((int32_t)total);
        }
        live_weight = used;
        s = a.m;
        __syncthreads();
    }

    // ---- main loop: pop a frontier vertex, step to a neighbour, add it.
    //
    // A step is two dependent loads (the neighbour, then its row bounds), and
    // the next step's pop needs the second one's result: how many entries the
    // new vertex adds.  With a cap that number is nearly always the cap (the
    // walk prefers vertices of high degree), so with a cap two more steps are
    // popped on that guess: iteration i issues the neighbour load of step
    // i + 2 and the row-bound loads of step i + 1, and appends step i, whose
    // loads have had an iteration each.  An append of fewer entries takes the
    // pops behind it back (their vertices are live again) and they are drawn
    // anew from the same random words, so the run is the sequential one.
    // Where more than about a quarter of the guesses are wrong (degrees mostly
    // below the cap) a step ahead costs more than it hides, and the rest of
    // the run goes one step at a time: 256 runs, m = 300, n = 2500, on 100,000
    // vertices, with pops ahead throughout / one at a time: all guesses right
    // 1.86 / 2.60 ms, nearly none 4.38 / 2.46, about a third wrong 2.58 / 2.34.
    // The loads of the steady path are issued in every iteration, needed or
    // not, and the paths that fill it wait for theirs: each use then waits for
    // its own load and not for the later ones.
    // A step is also some hundred instructions of one wavefront, hence the
    // scalar branches, the shared Philox calls and the branch-free writes.
    // 256 runs, m = 1000, n = 8000, cap 30: 9.24 ms one step at a time (1.32 us
    // each), now 6.95 ms.
    struct Step {
        int32_t k, v, b, e;   // popped slot; its neighbour; the neighbour's row bounds (loads in flight)
        uint32_t deg;         // degree of the popped vertex
        uint64_t round;       // probing rounds used up to and with this pop
    };
    Step q[3] = {};
    uint64_t round = 0;       // ... up to the last append
    int32_t popped = 0;       // steps popped from step i on: q[phase], q[phase + 1], ...
    uint64_t pblk = ~0ull - 8;
    int32_t nblk = -64, prov = 0;   // prov: slots below it have cap entries written ahead
    Words pw{0, 0, 0, 0}, nw{0, 0, 0, 0};
    int32_t i = a.m, flushed = a.m, held = 0;   // vertices flushed .. i - 1 wait in `held`, one per lane
    // ordering of this wavefront's LDS accesses (they execute in order)
    auto lds_order = []() __attribute__((always_inline)) { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
    // Probing rounds until one hits: the lowest of the 64 processors on a live
    // entry wins.  It is nearly always among the first 16, so only their words
    // are drawn, for 16 rounds at once (lane l: processor l % 16, Philox block
    // pblk + l / 16); a round they all miss is drawn for the other 48.  One
    // step at a time (without a cap a popped hub leaves thousands of dead
    // entries, and most rounds miss) all 64 words are drawn, four rounds at
    // once: 30 roots, 2000 vertices of 20,000, no cap, 256 runs: 16 words
    // first 7.3 ms, 64 words 3.6 ms.
    auto probe = [&](auto mode, int32_t in_use, uint64_t &rnd, int32_t limit) __attribute__((always_inline)) -> int32_t {
        constexpr bool AHEAD = decltype(mode)::value;
        for (int32_t rr = 0; rr < limit; ++rr) {
            const uint64_t blk = rnd >> 2;
            if (!AHEAD) {
                if (blk != pblk) {
                    pw = philox(blk, kKindProbe, (uint64_t)lane, a.seed, sid);
                    pblk = blk;
                }
                const int32_t slot = db[below32(pw.get((uint32_t)rnd & 3u), (uint32_t)in_use)];
                ++rnd;
                const uint64_t mask = __ballot(((uint32_t)sl.bd[slot].y & kLive) != 0u);
                if (mask) return __builtin_amdgcn_readlane(slot, __ffsll((unsigned long long)mask) - 1);
                continue;
            }
            if (blk - pblk >= 4u) {
                pw = philox(blk + (lane >> 4), kKindProbe, (uint64_t)(lane & 15), a.seed, sid);
                pblk = blk;
            }
            const int g = 16 * (int)(blk - pblk);
            const uint32_t wi = (uint32_t)rnd & 3u;
            ++rnd;
            int32_t slot = db[below32(pw.get(wi), (uint32_t)in_use)];
            uint64_t mask = __ballot(((uint32_t)sl.bd[slot].y & kLive) != 0u) & (0xFFFFull << g);
            if (__builtin_expect(mask == 0, 0)) {
                const Words x = philox(blk, kKindProbe, (uint64_t)lane, a.seed, sid);
                slot = db[below32(x.get(wi), (uint32_t)in_use)];
                mask = __ballot(((uint32_t)sl.bd[slot].y & kLive) != 0u);
            }
            if (mask) return __builtin_amdgcn_readlane(slot, __ffsll((unsigned long long)mask) - 1);
        }
        return -1;
    };
    // vector loads of one word (all lanes the same): the scalar unit's loads
    // would share the LDS reads' wait counter
    auto load1 = [&](const int32_t *base, int64_t at) __attribute__((always_inline)) {
        uint32_t lo = (uint32_t)at;
        asm volatile("" : "+v"(lo));
        return base[lo];
    };
    // the loads of x are done
    auto landed = [&](Step &x) __attribute__((always_inline)) { asm volatile("" : "+v"(x.v), "+v"(x.b), "+v"(x.e)); };
    // slot k leaves the frontier as step t; returns where its neighbour is.
    // Neighbour words: lane l holds the Philox block nblk + l (four steps each).
    auto take = [&](Step &x, int32_t k, int32_t t) __attribute__((always_inline)) -> int64_t {
        const int2 bd = sl.bd[k];
        const int32_t beg = uniform(bd.x);
        x.k = k;
        x.deg = (uint32_t)uniform(bd.y) & ~kLive;   // >= 1: its weight was > 0
        lds_order();
        sl.bd[k].y = (int32_t)x.deg;                // no longer in the frontier
        lds_order();
        const int32_t blk = t >> 2;
        if ((uint32_t)(blk - nblk) >= 64u) {
            nw = philox((uint64_t)(blk + lane), kKindNeigh, 0, a.seed, sid);
            nblk = blk;
        }
        const uint64_t word = nw.get((uint32_t)(t & 3));
        const int src = (int)(blk - nblk);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)word, src);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(word >> 32), src);
        return (int64_t)beg + below32(((uint64_t)hi << 32) | lo, x.deg);
    };
    auto bounds = [&](Step &x) __attribute__((always_inline)) {
        const int32_t u = (uint32_t)x.v < (uint32_t)a.nV ? x.v : 0;
        x.b = load1(a.indptr, u);
        x.e = load1(a.indptr + 1, u);
    };
    // pop step i + j ahead (popped == j), as if steps i .. i + j - 1 append cap
    // entries each; returns where its neighbour is, or 0 without a pop
    auto ahead = [&](Step &x, const Step &prev, int32_t j) __attribute__((always_inline)) -> int64_t {
        if ((int)(popped != j) | (int)(i + j >= a.n) | (int)(used + j * a.cap > a.db_cap) | (int)(s + j > a.ia_cap))
            return 0;
        const int32_t ps = s + j - 1;               // the slot step i + j - 1 will take
        const int32_t pb = used + (j - 1) * a.cap;
        // (lanes past the end, and all lanes of a slot write, store the same
        // value again: no branch over the exec mask)
        for (int32_t e0 = 0; e0 < a.cap; e0 += 64) db[pb + min(e0 + lane, a.cap - 1)] = (uint16_t)ps;
        sl.bd[ps].y = (int32_t)kLive;
        prov = ps + 1;
        lds_order();
        uint64_t rnd = prev.round;
        const int32_t k = probe(std::true_type{}, used + j * a.cap, rnd, 8);
        if (k < 0 || k >= s) return 0;              // none, or a vertex that is not known yet
        x.round = rnd;
        popped = j + 1;
        return take(x, k, i - a.m + j);
    };
    int32_t wrong = 0;        // guesses taken back
    auto step = [&](auto mode, auto phase) __attribute__((always_inline)) -> bool {
        constexpr bool AHEAD = decltype(mode)::value;   // pops ahead, or one step at a time
        constexpr int P = decltype(phase)::value;
        Step &c = q[P], &n1 = q[(P + 1) % 3], &n2 = q[(P + 2) % 3];
        // (the same in every lane; said here so that the step's branches and
        // arithmetic are scalar)
        s = uniform(s);
        used = uniform(used);
        live_weight = uniform(live_weight);
        popped = uniform(popped);
        prov = uniform(prov);
        i = uniform(i);
        flushed = uniform(flushed);
        round = uniform64(round);
        c.round = uniform64(c.round);
        n1.round = uniform64(n1.round);
        c.k = uniform(c.k);
        n1.k = uniform(n1.k);
        c.deg = (uint32_t)uniform((int32_t)c.deg);
        pblk = uniform64(pblk);
        nblk = uniform(nblk);
        if (live_weight == 0) { status = GCN_SAMPLE_EXHAUSTED; return false; }
        if (popped < (AHEAD ? 2 : 1)) {
            if (popped == 0) {
                c.round = round;
                const int32_t k = probe(mode, used, c.round, (int32_t)kProbeRoundLimit);
                if (k < 0) { status = GCN_SAMPLE_PROBE_LIMIT; return false; }
                c.v = load1(a.indices, take(c, k, i - a.m));
                popped = 1;
                bounds(c);
            }
            if (AHEAD) n1.v = load1(a.indices, ahead(n1, c, 1));
            landed(c);
            if (AHEAD) landed(n1);
        }
        if (AHEAD) {
            n2.v = load1(a.indices, ahead(n2, n1, 2));
            bounds(n1);
        }
        // append step i
        const int32_t v = uniform(c.v), b = uniform(c.b);
        if ((uint32_t)v >= (uint32_t)a.nV) { status = GCN_SAMPLE_BAD_GRAPH; return false; }
        const uint32_t d2 = (uint32_t)(uniform(c.e) - b);
        const int32_t w = weight_of_deg(d2, a.cap);
        live_weight -= weight_of_deg(c.deg, a.cap);
        round = c.round;
        // (with pops ahead there is room for cap >= w entries and a slot)
        if ((int64_t)used + w > a.db_cap || s == a.ia_cap) {
            __syncthreads();
            dashboard_cleanup(db, sl, a.cap, s, used);
            prov = 0;
        }
        if ((int64_t)used + w > a.db_cap) { status = GCN_SAMPLE_OVERFLOW; return false; }
        if (!AHEAD || s >= prov)                    // not written ahead
            for (int32_t e0 = 0; e0 < w; e0 += 64)
                if (e0 + lane < w) db[used + e0 + lane] = (uint16_t)s;
        sl.v[s] = v;
        sl.bd[s] = make_int2(b, (int32_t)(d2 | kLive));
        if (lane == (i & 63)) held = v;
        used += w;
        live_weight += w;
        ++s;
        count = ++i;
        --popped;
        if (AHEAD && w != a.cap && popped > 0) {    // the guess was wrong
            if (lane == 0) {
                sl.bd[n1.k].y |= (int32_t)kLive;
                if (popped > 1) sl.bd[n2.k].y |= (int32_t)kLive;
            }
            popped = 0;
            prov = s;
            wrong = uniform(wrong) + 1;
        }
        lds_order();
        if (i - flushed == 64) {
            out[flushed + ((lane - flushed) & 63)] = held;
            flushed = i;
        }
        return i < a.n;
    };
    bool more = status == GCN_SAMPLE_OK && i < a.n;
    if (CAPPED && more) {
        const std::true_type ahead_mode{};
        while ((more = step(ahead_mode, std::integral_constant<int, 0>{}) &&
                       step(ahead_mode, std::integral_constant<int, 1>{}) &&
                       step(ahead_mode, std::integral_constant<int, 2>{})) &&
               wrong <= 16 + ((i - a.m) >> 2)) {
        }
        if (more) {   // the pops ahead are taken back
            if (lane == 0) {
                if (popped > 0) sl.bd[q[0].k].y |= (int32_t)kLive;
                if (popped > 1) sl.bd[q[1].k].y |= (int32_t)kLive;
            }
            lds_order();
            popped = 0;
            pblk = ~0ull - 8;
        }
    }
    if (more)
        while (step(std::false_type{}, std::integral_constant<int, 0>{})) {
        }
    if (flushed + ((lane - flushed) & 63) < i) out[flushed + ((lane - flushed) & 63)] = held;
    if (lane == 0) {
        a.counts[blockIdx.x] = count;
        a.status[blockIdx.x] = status;
    }
}

// ------------------------------------------------------- induced subgraphs
constexpr int kTB = 256;
constexpr int kItems = 8;
constexpr int kTile = kTB * kItems;   // elements per scan tile

// exclusive scan of one value per thread over the block; returns the total
__device__ __forceinline__ int64_t block_excl_scan(int64_t x, int64_t &total) {
    __shared__ int64_t wsum[kTB / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t incl = wave_incl_scan(x);
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int64_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kTB / 64; ++w) {
        if (w < wid) before += wsum[w];
        total += wsum[w];
    }
    __syncthreads();
    return before + incl - x;
}

__global__ __launch_bounds__(kTB) void fill_i32_kernel(int32_t *__restrict__ x, int64_t n, int32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * kTB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kTB) x[i] = v;
}

// The sample sets are membership bitmaps, one bit per vertex of G per list:
// bits[s][v / 32] bit v % 32.  With wpre[s][k], the number of sampled
// vertices in words 0 .. k-1, the local id of a sampled vertex v (its rank
// among the list's distinct vertices in ascending order) is
// wpre[s][v / 32] + popcount of the bits of word v / 32 below v.  A list's
// bitmap and prefix take 8 bytes per 32 vertices of G, so the row kernels
// hold them in LDS and look each neighbour up there (the neighbour lists of
// G stream from memory coalesced; nothing else is read per neighbour).

// bits[s][v / 32] |= bit v % 32 for every sampled v of list s (duplicates collapse)
__global__ __launch_bounds__(kTB) void mark_kernel(int32_t nV, int32_t n, int32_t W,
                                                   const int32_t *__restrict__ vertices,
                                                   const int32_t *__restrict__ counts, uint32_t *__restrict__ bits) {
    const int s = blockIdx.y;
    const int32_t cnt = min(counts[s], n);
    for (int32_t i = blockIdx.x * kTB + threadIdx.x; i < cnt; i += gridDim.x * kTB) {
        const int32_t v = vertices[(int64_t)s * n + i];
        if ((uint32_t)v < (uint32_t)nV) atomicOr(&bits[(int64_t)s * W + (v >> 5)], 1u << (v & 31));
    }
}

// per (list, tile of kTile words): the number of set bits in the tile
__global__ __launch_bounds__(kTB) void popc_tile_sum_kernel(const uint32_t *__restrict__ bits, int32_t W,
                                                            int64_t *__restrict__ tsum, int32_t tiles) {
    const int s = blockIdx.y;
    const int64_t t0 = (int64_t)blockIdx.x * kTile;
    const uint32_t *bs = bits + (int64_t)s * W;
    int64_t acc = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t i = t0 + (int64_t)threadIdx.x * kItems + j;
        if (i < W) acc += __popc(bs[i]);
    }
    int64_t total;
    block_excl_scan(acc, total);
    if (threadIdx.x == 0) tsum[(int64_t)s * tiles + blockIdx.x] = total;
}

// per segment: exclusive scan of its tile sums (in place), segment total
__global__ __launch_bounds__(kTB) void seg_tile_scan_kernel(int64_t *__restrict__ tsum, int32_t tiles,
                                                            int64_t *__restrict__ seg_total) {
    const int s = blockIdx.x;
    int64_t *t = tsum + (int64_t)s * tiles;
    int64_t carry = 0;
    for (int32_t base = 0; base < tiles; base += kTB) {
        const int32_t i = base + threadIdx.x;
        const int64_t v = i < tiles ? t[i] : 0;
        int64_t total;
        const int64_t ex = block_excl_scan(v, total);
        if (i < tiles) t[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) seg_total[s] = carry;
}

// wpre[s][k] = sampled vertices in words 0 .. k-1;  vsub[s][local id] = v
__global__ __launch_bounds__(kTB) void rank_kernel(int32_t n, int32_t W, const uint32_t *__restrict__ bits,
                                                   const int64_t *__restrict__ toff, int32_t tiles,
                                                   int32_t *__restrict__ wpre, int32_t *__restrict__ vsub) {
    const int s = blockIdx.y;
    const int64_t t0 = (int64_t)blockIdx.x * kTile;
    const uint32_t *bs = bits + (int64_t)s * W;
    uint32_t words[kItems];
    int64_t acc = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t i = t0 + (int64_t)threadIdx.x * kItems + j;
        words[j] = i < W ? bs[i] : 0u;
        acc += __popc(words[j]);
    }
    int64_t total;
    int64_t r = toff[(int64_t)s * tiles + blockIdx.x] + block_excl_scan(acc, total);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t i = t0 + (int64_t)threadIdx.x * kItems + j;
        if (i < W) wpre[(int64_t)s * W + i] = (int32_t)r;
        for (uint32_t b = words[j]; b; b &= b - 1u) {
            if (r < n) vsub[(int64_t)s * n + r] = (int32_t)(32 * i + __builtin_ctz(b));
            ++r;
        }
    }
}

// Row kernels: one block of kRowThreads takes rows [b R, (b+1) R) of list s
// (R = kRowsPerBlock), clipped to the list's distinct vertices; its
// wavefronts take the next row from an LDS counter (hub rows of G are
// hundreds of times longer than the median one).  TABLE_LDS: the list's
// bitmap (and prefix) copied into LDS first; otherwise read where they are.
// The neighbour lists (4 bytes a neighbour, from the Infinity Cache or HBM)
// are what these passes read, and with one 256-byte piece in flight per
// wavefront their latency bounded them (count 2.14 ms, fill 6.58 ms for 256
// lists of the Reddit-shaped graph, 1.1 x 10^9 neighbours).  So a wavefront
// loads kRowChunks pieces at once (2 / 4 / 8 pieces: count 1.39 / 1.24 / 1.15
// ms), and the rows' bounds are read by the whole block up front instead of as
// two dependent loads a row.
constexpr int kRowThreads = 1024;
constexpr int kRowsPerBlock = 256;
constexpr int kRowChunks = 8;
constexpr size_t kInduceMaxLds = 128 * 1024;

__device__ __forceinline__ int32_t next_row(int32_t *ctr, int lane) {
    int32_t r = 0;
    if (lane == 0) r = atomicAdd(ctr, 1);
    return __shfl(r, 0);
}

// the bounds in G of rows r0 .. r1 - 1 of a list (whole block; r1 - r0 <= kRowsPerBlock)
__device__ __forceinline__ void load_row_bounds(int2 *rb, const int32_t *indptr, const int32_t *vs, int32_t r0,
                                                int32_t r1) {
    for (int32_t r = r0 + (int32_t)threadIdx.x; r < r1; r += kRowThreads) {
        const int32_t u = vs[r];
        rb[r - r0] = make_int2(indptr[u], indptr[u + 1]);
    }
}

// Calls f(w) for the row's neighbours, 64 at a time in order (lane l of a
// piece has its l-th neighbour; w = -1 past the row's end), with up to
// kRowChunks pieces loaded ahead of their use.  Loads past the end are clamped
// to the row's last neighbour.  (Unsigned offsets within the row: they pass its
// end by up to a round of pieces, and rows end at up to 2^31 - 1.)
template <class F>
__device__ __forceinline__ void for_row(const int32_t *__restrict__ indices, int2 b, int lane, F f) {
    const uint32_t len = b.y > b.x ? (uint32_t)b.y - (uint32_t)b.x : 0u, l = (uint32_t)lane;
    const int32_t *__restrict__ row = indices + b.x;
    uint32_t o = 0;
    for (; o + 64 < len; o += 64 * kRowChunks) {
        int32_t w[kRowChunks];
#pragma unroll
        for (int c = 0; c < kRowChunks; ++c) w[c] = row[min(o + 64 * c + l, len - 1)];
#pragma unroll
        for (int c = 0; c < kRowChunks; ++c)
            if (o + 64 * c < len) f(o + 64 * c + l < len ? w[c] : -1);
    }
    if (o < len) {
        const int32_t w = row[min(o + l, len - 1)];
        f(o + l < len ? w : -1);
    }
}

// row length of every local row: neighbours of vsub[s][i] that are in the list
template <bool TABLE_LDS>
__global__ __launch_bounds__(kRowThreads) void row_count_kernel(int32_t nV, int32_t n, int32_t W,
                                                                const int32_t *__restrict__ indptr,
                                                                const int32_t *__restrict__ indices,
                                                                const uint32_t *__restrict__ bits,
                                                                const int64_t *__restrict__ n_sub,
                                                                const int32_t *__restrict__ vsub,
                                                                int32_t *__restrict__ rowlen) {
    extern __shared__ __attribute__((aligned(8))) uint32_t tab[];
    __shared__ int2 rb[kRowsPerBlock];
    __shared__ int32_t ctr;
    const int s = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int32_t r0 = blockIdx.x * kRowsPerBlock;
    const int32_t r1 = (int32_t)min<int64_t>((int64_t)r0 + kRowsPerBlock, min<int64_t>(n_sub[s], n));
    if (r0 >= r1) return;
    const uint32_t *bs = bits + (int64_t)s * W;
    load_row_bounds(rb, indptr, vsub + (int64_t)s * n, r0, r1);
    if (TABLE_LDS) {
        for (int32_t k = threadIdx.x; k < W; k += kRowThreads) tab[k] = bs[k];
        bs = tab;
    }
    if (threadIdx.x == 0) ctr = r0;
    __syncthreads();
    for (int32_t i = next_row(&ctr, lane); i < r1; i = next_row(&ctr, lane)) {
        int32_t cnt = 0;
        for_row(indices, rb[i - r0], lane, [&](int32_t w) {
            cnt += ((uint32_t)w < (uint32_t)nV) ? (int32_t)((bs[w >> 5] >> (w & 31)) & 1u) : 0;
        });
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
        if (lane == 0) rowlen[(int64_t)s * n + i] = cnt;
    }
}

// per subgraph: indptr = exclusive scan of the row lengths (one block each);
// rows past the list's distinct vertices are empty.  Each length is replaced
// by the row's mean weight 1 / length (float bits), for the fill pass.
__global__ __launch_bounds__(kTB) void row_scan_kernel(int32_t n, int32_t *__restrict__ rowlen,
                                                       const int64_t *__restrict__ n_sub,
                                                       int32_t *__restrict__ indptr_sub,
                                                       int64_t *__restrict__ nnz_sub) {
    const int s = blockIdx.x;
    int32_t *rl = rowlen + (int64_t)s * n;
    int32_t *ip = indptr_sub + (int64_t)s * (n + 1);
    const int64_t ns = n_sub[s];
    int64_t carry = 0;
    for (int32_t base = 0; base < n; base += kTB) {
        const int32_t i = base + threadIdx.x;
        const int64_t v = i < ns ? rl[i] : 0;
        int64_t total;
        const int64_t ex = block_excl_scan(v, total);
        if (i < n) ip[i] = (int32_t)(carry + ex);
        if (i < ns) rl[i] = __float_as_int(1.0f / (float)(int32_t)v);
        carry += total;
    }
    if (threadIdx.x == 0) {
        ip[n] = (int32_t)carry;
        nnz_sub[s] = carry;
    }
}

// edge offsets of the subgraphs in the packed edge arrays; overflow flag
__global__ __launch_bounds__(kTB) void edge_offsets_kernel(int32_t S, const int64_t *__restrict__ nnz_sub,
                                                           int64_t *__restrict__ off, int64_t e_cap,
                                                           int32_t *__restrict__ status) {
    int64_t carry = 0;
    for (int32_t base = 0; base < S; base += kTB) {
        const int32_t i = base + threadIdx.x;
        const int64_t v = i < S ? nnz_sub[i] : 0;
        int64_t total;
        const int64_t ex = block_excl_scan(v, total);
        if (i < S) off[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) {
        off[S] = carry;
        *status = carry > e_cap ? 1 : 0;
    }
}

// local column ids and mean weights of every row, in neighbour order; rinv:
// the rows' mean weights (row_scan_kernel).  About a third of the neighbours
// are in the list, so a wavefront collects the ids it finds in an LDS ring and
// writes them 64 at a time as whole 256-byte pieces of the outputs (a store
// per 64 neighbours with a third of its lanes active: 4.5 ms, now 3.0 ms
// for the 351 million edges of 256 lists of the Reddit-shaped graph).
constexpr int kRing = 128;   // ids per wavefront: fewer than 64 held, up to 64 added
template <bool TABLE_LDS>
__global__ __launch_bounds__(kRowThreads) void fill_rows_kernel(int32_t nV, int32_t n, int32_t W,
                                                                const int32_t *__restrict__ indptr,
                                                                const int32_t *__restrict__ indices,
                                                                const uint32_t *__restrict__ bits,
                                                                const int32_t *__restrict__ wpre,
                                                                const int64_t *__restrict__ n_sub,
                                                                const int32_t *__restrict__ vsub,
                                                                const int32_t *__restrict__ indptr_sub,
                                                                const float *__restrict__ rinv,
                                                                const int64_t *__restrict__ off,
                                                                const int32_t *__restrict__ status,
                                                                int32_t *__restrict__ sub_indices,
                                                                float *__restrict__ sub_vals,
                                                                float *__restrict__ sub_vals_t) {
    extern __shared__ __attribute__((aligned(8))) uint32_t tab[];
    __shared__ int2 rb[kRowsPerBlock];
    __shared__ int32_t rp[kRowsPerBlock];
    __shared__ int32_t rings[kRowThreads / 64 * kRing];
    __shared__ int32_t ctr;
    const int s = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int32_t r0 = blockIdx.x * kRowsPerBlock;
    const int32_t r1 = (int32_t)min<int64_t>((int64_t)r0 + kRowsPerBlock, min<int64_t>(n_sub[s], n));
    if (*status != 0 || r0 >= r1) return;
    const uint32_t *bs = bits + (int64_t)s * W;
    const int32_t *ps = wpre + (int64_t)s * W;
    const int32_t *ip = indptr_sub + (int64_t)s * (n + 1);
    const float *ri = rinv + (int64_t)s * n;
    load_row_bounds(rb, indptr, vsub + (int64_t)s * n, r0, r1);
    for (int32_t r = r0 + (int32_t)threadIdx.x; r < r1; r += kRowThreads) rp[r - r0] = ip[r];
    if (TABLE_LDS) {
        for (int32_t k = threadIdx.x; k < W; k += kRowThreads) ((uint2 *)tab)[k] = make_uint2(bs[k], (uint32_t)ps[k]);
    }
    if (threadIdx.x == 0) ctr = r0;
    __syncthreads();
    const int64_t base = off[s];
    int32_t *const ring = rings + (threadIdx.x >> 6) * kRing;
    for (int32_t i = next_row(&ctr, lane); i < r1; i = next_row(&ctr, lane)) {
        const float val = ri[i];
        int64_t pos = base + rp[i - r0];   // where the ring's first id goes
        int32_t head = 0, held = 0;        // the ring holds ids head .. head + held - 1
        // lanes read what others stored: the stores come before, and the next
        // ones after (a wavefront's LDS accesses execute in order, so the
        // fences only keep the compiler from moving them)
        auto flush = [&](int32_t cnt) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane < cnt) {
                const int32_t loc = ring[(head + lane) & (kRing - 1)];
                const int64_t q = pos + lane;
                sub_indices[q] = loc;
                sub_vals[q] = val;
                if (sub_vals_t) sub_vals_t[q] = ri[loc];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            head = (head + cnt) & (kRing - 1);
            held -= cnt;
            pos += cnt;
        };
        for_row(indices, rb[i - r0], lane, [&](int32_t w) {
            int32_t loc = -1;
            if constexpr (TABLE_LDS) {
                const bool in = (uint32_t)w < (uint32_t)nV;
                const uint2 e = ((const uint2 *)tab)[in ? w >> 5 : 0];
                if (in && ((e.x >> (w & 31)) & 1u)) loc = (int32_t)e.y + __popc(e.x & ((1u << (w & 31)) - 1u));
            } else if ((uint32_t)w < (uint32_t)nV) {
                const uint32_t word = bs[w >> 5], below = word & ((1u << (w & 31)) - 1u);
                if ((word >> (w & 31)) & 1u) loc = ps[w >> 5] + __popc(below);
            }
            const uint64_t mask = __ballot(loc >= 0);
            const int32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (loc >= 0) ring[(head + held + rank) & (kRing - 1)] = loc;
            held += __popcll(mask);
            if (held >= 64) flush(64);
        });
        while (held > 0) flush(min(held, 64));
    }
}

__global__ __launch_bounds__(kTB) void copy_n_sub_kernel(int32_t S, const int64_t *__restrict__ a,
                                                         int32_t *__restrict__ b) {
    const int32_t i = blockIdx.x * kTB + threadIdx.x;
    if (i < S) b[i] = (int32_t)a[i];
}

// ------------------------------------------------------------------ gather
// out[i, :] = X[rows[i], :] for 4-byte elements; a row index outside
// [0, n_rows_X) gives a row of zeros.  VEC: 16-byte moves.
template <bool VEC>
__global__ __launch_bounds__(kTB) void gather_kernel(const uint32_t *__restrict__ X, int32_t n_rows_X,
                                                     int32_t width, int64_t ldx, const int32_t *__restrict__ rows,
                                                     int32_t count, uint32_t *__restrict__ out, int64_t ldo) {
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * (kTB / 64) + (threadIdx.x >> 6);
    if (i >= count) return;
    const int32_t r = rows[i];
    const bool ok = (uint32_t)r < (uint32_t)n_rows_X;
    const uint32_t *src = X + (int64_t)(ok ? r : 0) * ldx;
    uint32_t *dst = out + i * ldo;
    if (VEC) {
        for (int32_t c = lane * 4; c < width; c += 256) {
            uint4 v = ok ? *(const uint4 *)(src + c) : uint4{0, 0, 0, 0};
            *(uint4 *)(dst + c) = v;
        }
    } else {
        for (int32_t c = lane; c < width; c += 64) dst[c] = ok ? src[c] : 0u;
    }
}

int blocks_for(int64_t n, int per) { return (int)std::min<int64_t>((n + per - 1) / per, 65535); }

}  // namespace

size_t sampler_lds_bytes(int32_t db_cap, int32_t ia_cap) {
    return align256((size_t)ia_cap * 12 + (size_t)db_cap * 2);
}

int frontier_sample(const SampArgs &a, int32_t S, size_t lds, hipStream_t s) {
    static std::once_flag attr;
    std::call_once(attr, [] {
        hipFuncSetAttribute((const void *)frontier_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kSamplerMaxLds);
        hipFuncSetAttribute((const void *)frontier_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kSamplerMaxLds);
    });
    // without a cap, or with one that few degrees reach, a vertex's entries are
    // its degree, which cannot be guessed, and a Dashboard may have no room for
    // the guess (cap 5000: 4.56 ms with pops ahead, 1.73 without; cap 128 on
    // 200,000 vertices of degree 40: 2.85 and 2.75; cap 64: 2.41 and 2.65)
    if (a.cap > 0 && a.cap <= 256) frontier_kernel<true><<<S, kSampThreads, lds, s>>>(a);
    else frontier_kernel<false><<<S, kSampThreads, lds, s>>>(a);
    GCN_LAUNCH_CHECK("frontier_kernel");
    return GCN_OK;
}

}  // namespace gcn

using namespace gcn;

namespace {
struct InduceWs {
    uint32_t *bits;     // [S][W]: membership bitmap of each list (W = words of nV bits)
    int32_t *wpre;      // [S][W]: sampled vertices in the words before each word
    int64_t *tsum;      // [S][tiles]: tile sums, then their exclusive scan
    int64_t *n_sub64;   // [S]
    int64_t *nnz_sub;   // [S]
    int32_t *rowlen;    // [S][n]: row lengths, then the mean weights 1 / length (float bits)
};
InduceWs carve_induce(Arena &ar, int32_t nV, int32_t n, int32_t S) {
    InduceWs w;
    const int32_t W = (nV + 31) / 32;
    const int32_t tiles = (int32_t)((W + kTile - 1) / kTile);
    w.bits = ar.take<uint32_t>((size_t)S * W);
    w.wpre = ar.take<int32_t>((size_t)S * W);
    w.tsum = ar.take<int64_t>((size_t)S * tiles);
    w.n_sub64 = ar.take<int64_t>(S);
    w.nnz_sub = ar.take<int64_t>(S);
    w.rowlen = ar.take<int32_t>((size_t)S * n);
    return w;
}
}  // namespace

extern "C" {

int gcn_sampler_plan(int32_t n_vertices, const int32_t *indptr_host, int32_t m, int32_t n, double eta,
                     int32_t cap, uint64_t seed, gcn_sampler_params *out) {
    if (!indptr_host || !out || n_vertices <= 0 || m <= 0 || m > n_vertices || n < m || !(eta > 1.0) ||
        cap < 0) {
        set_error("gcn_sampler_plan: need indptr_host, out, 0 < m <= n_vertices, n >= m, eta > 1, cap >= 0");
        return GCN_EINVAL;
    }
    double sum_w = 0.0;
    int64_t wmax = 0;
    for (int32_t v = 0; v < n_vertices; ++v) {
        int64_t d = (int64_t)indptr_host[v + 1] - indptr_host[v];
        if (cap > 0 && d > cap) d = cap;
        sum_w += (double)d;
        wmax = std::max(wmax, d);
    }
    // Dashboard of eta * m * (mean entries per vertex) entries (Sec. IV-B), and
    // at least a frontier of m vertices of the largest weight (no overflow is
    // then possible); Index Array m + 512 slots.  Clamped to one CU's LDS;
    // at <= 80 KB two samplers share a CU.
    const int64_t ia = std::min<int64_t>((int64_t)m + 512, 65535);
    if (ia <= m || (size_t)ia * 12 + 2 > kSamplerMaxLds) {
        set_error("gcn_sampler_plan: a frontier of m = %d does not fit the %zu bytes of LDS", m,
                  (size_t)kSamplerMaxLds);
        return GCN_EUNSUPPORTED;
    }
    int64_t db = (int64_t)std::ceil(eta * (double)m * (sum_w / n_vertices));
    db = std::max<int64_t>(db, (int64_t)m * wmax);
    db = std::max<int64_t>(db, 1);
    db = std::min<int64_t>(db, ((int64_t)kSamplerMaxLds - ia * 12) / 2);
    out->m = m;
    out->n = n;
    out->db_entries = (int32_t)db;
    out->ia_slots = (int32_t)ia;
    out->cap = cap;
    out->seed = seed;
    return GCN_OK;
}

int gcn_frontier_sample(const gcn_csr *G, const gcn_sampler_params *p, int64_t first_sampler, int32_t S,
                        int32_t *vertices, int32_t *counts, int32_t *status, void *stream) {
    if (!G || !p || !vertices || !counts || !status || S < 0 || first_sampler < 0) {
        set_error("gcn_frontier_sample: null argument or negative count");
        return GCN_EINVAL;
    }
    if (G->n_rows != G->n_cols || G->n_rows <= 0 || !G->indptr || (G->nnz > 0 && !G->indices) || G->indices16) {
        set_error("gcn_frontier_sample: G must be a square CSR with at least one vertex and int32 indices");
        return GCN_ESHAPE;
    }
    if (p->m <= 0 || p->m > G->n_rows || p->n < p->m || p->ia_slots <= p->m || p->ia_slots > 65535 ||
        p->db_entries <= 0 || p->cap < 0) {
        set_error("gcn_frontier_sample: need 0 < m <= n_vertices, n >= m, m < ia_slots <= 65535, db_entries > 0");
        return GCN_EINVAL;
    }
    const size_t lds = sampler_lds_bytes(p->db_entries, p->ia_slots);
    int dev = 0, max_lds = 0;
    GCN_HIP_CHECK(hipGetDevice(&dev));
    GCN_HIP_CHECK(hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    const size_t limit = std::min<size_t>((size_t)max_lds, kSamplerMaxLds);
    if (lds > limit) {
        set_error("gcn_frontier_sample: Dashboard of %d entries and %d slots needs %zu bytes of LDS (limit %zu)",
                  p->db_entries, p->ia_slots, lds, limit);
        return GCN_EUNSUPPORTED;
    }
    if (S == 0) return GCN_OK;
    SampArgs a;
    a.nV = G->n_rows;
    a.indptr = G->indptr;
    a.indices = G->indices;
    a.m = p->m;
    a.n = p->n;
    a.db_cap = p->db_entries;
    a.ia_cap = p->ia_slots;
    a.cap = p->cap;
    a.seed = p->seed;
    a.first_sampler = first_sampler;
    a.vertices = vertices;
    a.counts = counts;
    a.status = status;
    hipStream_t s = (hipStream_t)stream;
    ProfScope prof(K_SAMPLE, s, 0.0, 0.0);
    return frontier_sample(a, S, lds, s);
}

size_t gcn_induce_workspace_bytes(int32_t n_vertices, int32_t n, int32_t S) {
    if (n_vertices <= 0 || n < 0 || S <= 0) return 256;
    Arena ar(nullptr, 0);
    carve_induce(ar, n_vertices, n, S);
    return ar.used;
}

int gcn_induce_subgraphs(const gcn_csr *G, int32_t S, int32_t n, const int32_t *vertices, const int32_t *counts,
                         int32_t *n_sub, int32_t *vsub, int32_t *indptr_sub, int64_t *edge_offsets,
                         int32_t *sub_indices, float *sub_vals, float *sub_vals_t, int64_t edge_capacity,
                         int32_t *status, void *ws, size_t ws_bytes, void *stream) {
    if (!G || !vertices || !counts || !n_sub || !vsub || !indptr_sub || !edge_offsets || !status || S < 0 ||
        n < 0 || edge_capacity < 0 || (edge_capacity > 0 && (!sub_indices || !sub_vals))) {
        set_error("gcn_induce_subgraphs: null argument or negative size");
        return GCN_EINVAL;
    }
    if (G->n_rows != G->n_cols || G->n_rows <= 0 || !G->indptr || (G->nnz > 0 && !G->indices) || G->indices16) {
        set_error("gcn_induce_subgraphs: G must be a square CSR with at least one vertex and int32 indices");
        return GCN_ESHAPE;
    }
    if (S == 0) return GCN_OK;
    const int32_t nV = G->n_rows;
    Arena ar(ws, ws_bytes);
    InduceWs w = carve_induce(ar, nV, n, S);
    if (!w.bits || !w.rowlen || ((uintptr_t)ws & 255u)) {
        set_error("gcn_induce_subgraphs: workspace of %zu bytes is too small or misaligned (need %zu)", ws_bytes,
                  gcn_induce_workspace_bytes(nV, n, S));
        return GCN_EWORKSPACE;
    }
    if (S > 65535) {
        set_error("gcn_induce_subgraphs: at most 65535 subgraphs per call");
        return GCN_EINVAL;
    }
    hipStream_t s = (hipStream_t)stream;
    ProfScope prof(K_INDUCE, s, 0.0, 0.0);
    const int32_t W = (nV + 31) / 32;
    const int32_t tiles = (W + kTile - 1) / kTile;
    const int64_t words = (int64_t)S * W;
    fill_i32_kernel<<<blocks_for(words, kTB * 8), kTB, 0, s>>>((int32_t *)w.bits, words, 0);
    if (n > 0) {
        mark_kernel<<<dim3(blocks_for(n, kTB), S), kTB, 0, s>>>(nV, n, W, vertices, counts, w.bits);
    }
    popc_tile_sum_kernel<<<dim3(tiles, S), kTB, 0, s>>>(w.bits, W, w.tsum, tiles);
    seg_tile_scan_kernel<<<S, kTB, 0, s>>>(w.tsum, tiles, w.n_sub64);
    rank_kernel<<<dim3(tiles, S), kTB, 0, s>>>(n, W, w.bits, w.tsum, tiles, w.wpre, vsub);
    copy_n_sub_kernel<<<blocks_for(S, kTB), kTB, 0, s>>>(S, w.n_sub64, n_sub);
    // the row kernels hold a list's bitmap (and prefix) in LDS when they fit
    const size_t count_lds = (size_t)W * 4, fill_lds = (size_t)W * 8;
    const bool lds = fill_lds <= kInduceMaxLds;
    static std::once_flag lds_attr;
    std::call_once(lds_attr, [] {
        hipFuncSetAttribute((const void *)row_count_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kInduceMaxLds);
        hipFuncSetAttribute((const void *)fill_rows_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kInduceMaxLds);
    });
    const dim3 rgrid((n + kRowsPerBlock - 1) / kRowsPerBlock, S);
    if (n > 0) {
        if (lds)
            row_count_kernel<true><<<rgrid, kRowThreads, count_lds, s>>>(nV, n, W, G->indptr, G->indices, w.bits,
                                                                        w.n_sub64, vsub, w.rowlen);
        else
            row_count_kernel<false><<<rgrid, kRowThreads, 0, s>>>(nV, n, W, G->indptr, G->indices, w.bits,
                                                                 w.n_sub64, vsub, w.rowlen);
    }
    row_scan_kernel<<<S, kTB, 0, s>>>(n, w.rowlen, w.n_sub64, indptr_sub, w.nnz_sub);
    edge_offsets_kernel<<<1, kTB, 0, s>>>(S, w.nnz_sub, edge_offsets, edge_capacity, status);
    if (n > 0) {
        if (lds)
            fill_rows_kernel<true><<<rgrid, kRowThreads, fill_lds, s>>>(
                nV, n, W, G->indptr, G->indices, w.bits, w.wpre, w.n_sub64, vsub, indptr_sub,
                (const float *)w.rowlen, edge_offsets, status,
                sub_indices, sub_vals, sub_vals_t);
        else
            fill_rows_kernel<false><<<rgrid, kRowThreads, 0, s>>>(
                nV, n, W, G->indptr, G->indices, w.bits, w.wpre, w.n_sub64, vsub, indptr_sub,
                (const float *)w.rowlen, edge_offsets, status,
                sub_indices, sub_vals, sub_vals_t);
    }
    GCN_LAUNCH_CHECK("induce kernels");
    return GCN_OK;
}

int gcn_gather_rows(const void *X, int32_t n_rows_X, int32_t width, int64_t ldx, const int32_t *rows,
                    int32_t count, void *out, int64_t ldo, void *stream) {
    if (count < 0 || width < 0 || n_rows_X < 0 || (count > 0 && (!X || !rows || !out))) {
        set_error("gcn_gather_rows: null argument or negative size");
        return GCN_EINVAL;
    }
    if (ldx < width || ldo < width) {
        set_error("gcn_gather_rows: leading dimensions must be >= width");
        return GCN_ESHAPE;
    }
    if (count == 0 || width == 0) return GCN_OK;
    hipStream_t s = (hipStream_t)stream;
    ProfScope prof(K_GATHER, s, 0.0, 2.0 * 4.0 * (double)count * width);
    const bool vec = width % 4 == 0 && ldx % 4 == 0 && ldo % 4 == 0 && ((uintptr_t)X & 15u) == 0 &&
                     ((uintptr_t)out & 15u) == 0;
    const int blocks = (int)(((int64_t)count + kTB / 64 - 1) / (kTB / 64));
    if (vec)
        gather_kernel<true><<<blocks, kTB, 0, s>>>((const uint32_t *)X, n_rows_X, width, ldx, rows, count,
                                                   (uint32_t *)out, ldo);
    else
        gather_kernel<false><<<blocks, kTB, 0, s>>>((const uint32_t *)X, n_rows_X, width, ldx, rows, count,
                                                    (uint32_t *)out, ldo);
    GCN_LAUNCH_CHECK("gather_kernel");
    return GCN_OK;
}

}  // extern "C"

extern "C" int gcn_csr_pattern_symmetric_host(int32_t n, const int32_t *indptr, const int32_t *indices) {
    if (n < 0 || !indptr || (indptr[n] > 0 && !indices)) {
        set_error("gcn_csr_pattern_symmetric_host: null pointer or negative size");
        return GCN_EINVAL;
    }
    for (int32_t i = 0; i < n; ++i) {
        for (int32_t p = indptr[i]; p < indptr[i + 1]; ++p) {
            const int32_t j = indices[p];
            if (j < 0 || j >= n || (p > indptr[i] && indices[p - 1] >= j)) {
                set_error("gcn_csr_pattern_symmetric_host: row %d is not strictly ascending within [0, n)", i);
                return GCN_EINVAL;
            }
        }
    }
    for (int32_t i = 0; i < n; ++i) {
        for (int32_t p = indptr[i]; p < indptr[i + 1]; ++p) {
            const int32_t j = indices[p];
            if (!std::binary_search(indices + indptr[j], indices + indptr[j + 1], i)) return 0;
        }
    }
    return 1;
}
