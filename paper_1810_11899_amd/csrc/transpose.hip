// CSR of A^T for the backward propagation.
//
// Row j of A^T lists the rows i of A that hold column j, in ascending i, with
// equal entries in their CSR order.  The CSR entries are already in row-major
// order, so A^T is exactly a *stable* sort of the entries by column.  This is
// done as an LSD radix sort with digits of up to 9 bits (two passes up to
// 262,144 columns), whose payload is what the output holds: the entry's row
// and value (bit for bit), so that the last pass writes t_indices and t_vals.
// Per pass:
//   1. per-tile digit histograms (integer LDS atomics: counts do not depend on
//      the order of the increments);
//   2. per digit, an exclusive scan over the tiles and the digit's total;
//   3. a stable scatter: each wavefront ranks its part of the tile in order
//      with ballots (lane order) and running counts, the tile is sorted by
//      digit in LDS, and every digit's run is written as one piece.  Every key
//      lands at a position that only depends on the input.
// Then t_indptr[j] = lower_bound(sorted keys, j).  The integer output is
// unique, hence bit-exact.
//
// What bounds it: the passes move 12 bytes an entry in and out (2 M entries:
// 48 MB a pass), and a 2048-key tile scattered key by key wrote 4-byte pieces
// and gathered rows and values at the end (50,000 columns, 2 M entries: 151
// us; 4096-key tiles, sorted, with their payload: 70 us).
#include <algorithm>

#include "common.h"

namespace gcn {
namespace {

constexpr int kTB = 256;            // threads per tile block
constexpr int kItems = 16;          // keys per thread per tile
constexpr int kTile = kTB * kItems; // keys per tile
constexpr int kDigitBits = 9;       // digits of at most this many bits
constexpr int kRadix = 1 << kDigitBits;
constexpr int kWaves = kTB / 64;

// the keys of a pass: A's column indices (first pass) or the last pass's keys
__global__ __launch_bounds__(kTB) void hist_kernel(int32_t nnz, IdxRef first, const uint32_t *__restrict__ keys,
                                                   int shift, uint32_t mask, int32_t ntiles,
                                                   int32_t *__restrict__ hist) {
    __shared__ int32_t cnt[kRadix];
    for (int d = threadIdx.x; d < kRadix; d += kTB) cnt[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kTile;
    uint32_t k[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int64_t p = min(base + it * kTB + (int64_t)threadIdx.x, (int64_t)nnz - 1);
        k[it] = keys ? keys[p] : (uint32_t)first[p];
    }
#pragma unroll
    for (int it = 0; it < kItems; ++it)
        if (base + it * kTB + threadIdx.x < nnz) atomicAdd(&cnt[(k[it] >> shift) & mask], 1);
    __syncthreads();
    for (uint32_t d = threadIdx.x; d <= mask; d += kTB) hist[(int64_t)d * ntiles + blockIdx.x] = cnt[d];
}

// exclusive scan over the block of one value per thread; total: their sum
__device__ __forceinline__ int32_t block_scan(int32_t x, int32_t *sh, int32_t &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) sh[wave] = incl;
    __syncthreads();
    int32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w < wave) before += sh[w];
        total += sh[w];
    }
    __syncthreads();
    return before + incl - x;
}

// one block per digit: its counts per tile become their exclusive scan, in
// place; total[d] = their sum
__global__ __launch_bounds__(kTB) void scan_tiles_kernel(int32_t ntiles, int32_t *__restrict__ hist,
                                                         int32_t *__restrict__ total) {
    __shared__ int32_t sh[kWaves];
    int32_t *h = hist + (int64_t)blockIdx.x * ntiles;
    int32_t carry = 0;
    for (int32_t t0 = 0; t0 < ntiles; t0 += 4 * kTB) {
        const int32_t t = t0 + 4 * (int32_t)threadIdx.x;
        int32_t v[4], sum = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = t + e < ntiles ? h[t + e] : 0;
            sum += v[e];
        }
        int32_t all;
        int32_t run = carry + block_scan(sum, sh, all);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (t + e < ntiles) h[t + e] = run;
            run += v[e];
        }
        carry += all;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// A pass takes the payload as two arrays (rows, vals: A's, or an earlier
// pass's t_indices and t_vals) or as pairs, and leaves it as the other form,
// so that a pass never reads what it writes and the last one ends in
// t_indices and t_vals.
template <bool IN_PAIRS>
__global__ __launch_bounds__(kTB) void scatter_kernel(int32_t nnz, IdxRef first, const uint32_t *__restrict__ keys_in,
                                                      const int32_t *__restrict__ rows,
                                                      const float *__restrict__ vals,
                                                      const uint2 *__restrict__ pairs_in, int shift, int dbits,
                                                      int32_t ntiles, const int32_t *__restrict__ offs,
                                                      const int32_t *__restrict__ total,
                                                      uint32_t *__restrict__ keys_out, uint2 *__restrict__ pairs_out,
                                                      int32_t *__restrict__ t_indices, float *__restrict__ t_vals) {
    __shared__ uint32_t skey[kTile];
    __shared__ uint2 spay[kTile];
    __shared__ int32_t cnt[kWaves][kRadix];   // a wavefront's keys of each digit, then where its next one goes
    __shared__ int32_t gbase[kRadix];         // a digit's first output minus its first place in the tile
    __shared__ int32_t sh[kWaves];
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const uint32_t mask = (1u << dbits) - 1u;
    const int64_t base = (int64_t)blockIdx.x * kTile + wave * (64 * kItems);
    const int32_t count = (int32_t)min((int64_t)kTile, (int64_t)nnz - (int64_t)blockIdx.x * kTile);
    uint32_t key[kItems];
    uint2 pay[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int64_t p = min(base + it * 64 + lane, (int64_t)nnz - 1);
        key[it] = keys_in ? keys_in[p] : (uint32_t)first[p];
        pay[it] = IN_PAIRS ? pairs_in[p] : make_uint2((uint32_t)rows[p], __float_as_uint(vals[p]));
    }
    for (int d = t; d < kWaves * kRadix; d += kTB) (&cnt[0][0])[d] = 0;
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
    int32_t rank[kItems];   // among the wavefront's keys of the same digit
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const bool valid = base + it * 64 + lane < nnz;
        const uint32_t digit = (key[it] >> shift) & mask;
        uint64_t match = __ballot(valid);
        for (int bit = 0; bit < dbits; ++bit) {
            const uint64_t bb = __ballot((digit >> bit) & 1u);
            match &= ((digit >> bit) & 1u) ? bb : ~bb;
        }
        const int32_t seen = valid ? cnt[wave][digit] : 0;
        rank[it] = seen + (int32_t)__popcll(match & below);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // every lane has read its count
        if (valid && (match & below) == 0) cnt[wave][digit] = seen + (int32_t)__popcll(match);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    // thread t: digits 2t and 2t + 1 (in order over the block)
    {
        int32_t c[2], g[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t d = 2 * t + e;
            c[e] = 0;
            for (int w = 0; w < kWaves; ++w) {
                const int32_t x = cnt[w][d];
                cnt[w][d] = c[e];
                c[e] += x;
            }
            g[e] = d <= mask ? total[d] : 0;
        }
        int32_t all;
        const int32_t l0 = block_scan(c[0] + c[1], sh, all);
        const int32_t g0 = block_scan(g[0] + g[1], sh, all);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t d = 2 * t + e;
            const int32_t l = l0 + (e ? c[0] : 0);
            for (int w = 0; w < kWaves; ++w) cnt[w][d] += l;
            if (d <= mask) gbase[d] = g0 + (e ? g[0] : 0) + offs[(int64_t)d * ntiles + blockIdx.x] - l;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kItems; ++it)
        if (base + it * 64 + lane < nnz) {
            const int32_t pos = cnt[wave][(key[it] >> shift) & mask] + rank[it];
            skey[pos] = key[it];
            spay[pos] = pay[it];
        }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int32_t i = it * kTB + t;
        if (i < count) {
            const uint32_t k = skey[i];
            const uint2 x = spay[i];
            const int64_t q = (int64_t)gbase[(k >> shift) & mask] + i;
            keys_out[q] = k;
            if (!pairs_out) {
                t_indices[q] = (int32_t)x.x;
                t_vals[q] = __uint_as_float(x.y);
            } else {
                pairs_out[q] = x;
            }
        }
    }
}

// t_indptr[j] = number of sorted keys < j, for j in [0, n_cols]
__global__ __launch_bounds__(kTB) void bounds_kernel(int32_t n_cols, int32_t nnz,
                                                     const uint32_t *__restrict__ keys,
                                                     int32_t *__restrict__ t_indptr) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j > n_cols) return;
    int64_t lo = 0, hi = nnz;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)keys[mid] < j) lo = mid + 1; else hi = mid;
    }
    t_indptr[j] = (int32_t)lo;
}

// rowid[p] = the row of A that holds entry p (one wavefront per row)
__global__ __launch_bounds__(kTB) void rowid_kernel(int32_t n_rows, const int32_t *__restrict__ indptr,
                                                    int32_t *__restrict__ rowid) {
    const int64_t r = (int64_t)blockIdx.x * (kTB / 64) + (threadIdx.x >> 6);
    if (r >= n_rows) return;
    const int32_t b = indptr[r], e = indptr[r + 1];
    // (unsigned or 64-bit positions here and in the other row walks: a lane's
    // last one passes the row's end, which is at up to 2^31 - 1; unsigned ones
    // cost nothing, 64-bit ones 1 of 72 us at 2 M entries)
    const uint32_t end = (uint32_t)max(e, 0);
    for (uint32_t p = (uint32_t)b + (threadIdx.x & 63); p < end; p += 64) rowid[p] = (int32_t)r;
}

// Symmetric pattern: A^T has A's row pointers and indices; the value at
// (row j, column i) is A's value at (i, j).
// Pass 1: whether row i's values are all the same bits (true of every row
// of a mean aggregation matrix, Sec. II), in which case that value is
// A(i, j) for every j.  A wavefront takes four rows, 16 lanes each: a row of
// at most 64 entries is checked by its lane group with four loads per lane
// in flight; the longer rows of the wavefront are then checked one at a time
// by all 64 lanes with eight loads each in flight (a hub row of 14,000
// entries is one wavefront's walk).  Four rows per wavefront, not one: the
// pass is bound by the latency of its two dependent loads, and a quarter of
// the wavefronts cover it in fewer rounds.
__global__ __launch_bounds__(kTB) void sym_rows_kernel(int32_t n, const int32_t *__restrict__ indptr,
                                                       const float *__restrict__ vals,
                                                       uint32_t *__restrict__ rowval, int32_t *__restrict__ rowconst) {
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, gl = lane & 15;
    const int64_t i = ((int64_t)blockIdx.x * (kTB / 64) + (threadIdx.x >> 6)) * 4 + g;
    const bool live = i < n;
    int32_t b = 0, e = 0;
    if (live) {
        b = indptr[i];
        e = indptr[i + 1];
    }
    const bool shortrow = e - b <= 64;
    const uint32_t first = live && e > b ? __float_as_uint(vals[b]) : 0u;
    bool same = true;
    if (live && shortrow) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t p = (int64_t)b + gl + 16 * u;
            v[u] = p < e ? __float_as_uint(vals[p]) : first;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) same = same && (v[u] == first);
    }
    const uint64_t bad = __ballot(!same);
    bool row_same = ((bad >> (16 * g)) & 0xFFFFull) == 0;
    // the long rows, one at a time (the loop is uniform over the wavefront)
    uint64_t longs = __ballot(live && !shortrow && gl == 0);
    while (longs) {
        const int lg = (__ffsll((unsigned long long)longs) - 1) >> 4;
        longs &= longs - 1;
        const int32_t lb = __shfl(b, 16 * lg), le = __shfl(e, 16 * lg);
        const uint32_t lf = __shfl(first, 16 * lg);
        bool s2 = true;
        constexpr int U = 8;
        int64_t p = (int64_t)lb + lane;
        for (; p + 64 * (U - 1) < le; p += 64 * U) {
            uint32_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = __float_as_uint(vals[p + 64 * u]);
#pragma unroll
            for (int u = 0; u < U; ++u) s2 = s2 && (v[u] == lf);
        }
        for (; p < le; p += 64) s2 = s2 && (__float_as_uint(vals[p]) == lf);
        const bool all_same = __all(s2);
        if (g == lg) row_same = all_same;
    }
    if (live && gl == 0) {
        rowval[i] = first;
        rowconst[i] = row_same ? 1 : 0;
    }
}

// Pass 2, one thread per entry p (row j, column i): the constant value of row
// i, or else j (the row holding p, by a search of indptr) and a binary search
// for j in row i.  An index outside [0, n), or a missing (i, j) found by the
// search, gives NaN.
__global__ __launch_bounds__(kTB) void sym_vals_kernel(int32_t n, int32_t nnz, const int32_t *__restrict__ indptr,
                                                       IdxRef indices,
                                                       const float *__restrict__ vals,
                                                       const uint32_t *__restrict__ rowval,
                                                       const int32_t *__restrict__ rowconst,
                                                       float *__restrict__ t_vals) {
    const int64_t stride = (int64_t)gridDim.x * kTB;
    for (int64_t p = (int64_t)blockIdx.x * kTB + threadIdx.x; p < nnz; p += stride) {
        const int32_t i = indices[p];
        float t = __int_as_float(0x7FC00000);
        if ((uint32_t)i < (uint32_t)n) {
            if (rowconst[i]) {
                t = __uint_as_float(rowval[i]);
            } else {
                int32_t a = 0, b = n;   // the last row r with indptr[r] <= p
                while (a < b) {
                    const int32_t mid = a + ((b - a + 1) >> 1);
                    if (indptr[mid] <= p) a = mid; else b = mid - 1;
                }
                const int32_t j = a;
                int32_t lo = indptr[i], hi = indptr[i + 1];   // first index >= j in row i
                while (lo < hi) {
                    const int32_t mid = lo + ((hi - lo) >> 1);
                    if (indices[mid] < j) lo = mid + 1; else hi = mid;
                }
                if (lo < indptr[i + 1] && indices[lo] == j) t = vals[lo];
            }
        }
        t_vals[p] = t;
    }
}

__global__ void fill_zero_kernel(int32_t *__restrict__ x, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0;
}

int key_bits(int32_t n_cols) {
    int b = 0;
    while (b < 31 && ((int64_t)1 << b) < (int64_t)n_cols) ++b;
    return b;  // keys are < n_cols <= 2^b
}

}  // namespace

namespace {
// Arrays of a sort: keys twice (the second first holds the entries' rows) and
// (row, value) pairs once.
struct SortPlan {
    int passes, dbits;
    int32_t ntiles;
};
SortPlan sort_plan(int32_t n_cols, int32_t nnz) {
    SortPlan p;
    const int bits = std::max(1, key_bits(n_cols));
    p.ntiles = (int32_t)(((int64_t)nnz + kTile - 1) / kTile);
    // a single tile counts at most 256 digits, which keeps its workspace to 16
    // bytes an entry and 3 KB (more tiles: 2 KB each of 4096 entries on top, and
    // the digits' totals)
    const int most = p.ntiles == 1 ? 8 : kDigitBits;
    p.passes = (bits + most - 1) / most;
    p.dbits = (bits + p.passes - 1) / p.passes;
    return p;
}
}  // namespace

size_t transpose_workspace_bytes(int32_t n_rows, int32_t n_cols, int32_t nnz) {
    (void)n_rows;
    if (nnz <= 0) return 256;
    const SortPlan p = sort_plan(n_cols, nnz);
    return 2 * align256((size_t)nnz * 4) + align256((size_t)nnz * 8) +
           align256((size_t)p.ntiles * 4 << p.dbits) + align256((size_t)4 << p.dbits);
}

int csr_transpose(int32_t n_rows, int32_t n_cols, int32_t nnz, const int32_t *indptr, IdxRef indices,
                  const float *vals, int32_t *t_indptr, int32_t *t_indices, float *t_vals, void *ws,
                  size_t ws_bytes, hipStream_t s) {
    if (nnz == 0) {
        ProfScope ps(K_T_FINAL, s, 0.0, (double)(n_cols + 1) * 4.0);
        hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n_cols + 1 + 255) / 256)), dim3(256), 0, s,
                           t_indptr, (int64_t)n_cols + 1);
        GCN_LAUNCH_CHECK("fill_zero_kernel");
        return GCN_OK;
    }
    const SortPlan p = sort_plan(n_cols, nnz);
    Arena ar(ws, ws_bytes);
    uint32_t *ka = ar.take<uint32_t>(nnz), *kb = ar.take<uint32_t>(nnz);
    uint2 *pairs = ar.take<uint2>(nnz);
    int32_t *hist = ar.take<int32_t>((size_t)p.ntiles << p.dbits);
    int32_t *total = ar.take<int32_t>((size_t)1 << p.dbits);
    if (!ka || !kb || !pairs || !hist || !total) {
        set_error("csr_transpose: workspace too small (%zu < %zu bytes)", ws_bytes,
                  transpose_workspace_bytes(n_rows, n_cols, nnz));
        return GCN_EWORKSPACE;
    }
    int32_t *rowid = (int32_t *)kb;   // read by the first pass, before kb is written
    {
        ProfScope ps(K_T_COUNT, s, 0.0, (double)nnz * 4.0);
        hipLaunchKernelGGL(rowid_kernel, dim3((unsigned)((n_rows + kTB / 64 - 1) / (kTB / 64))), dim3(kTB), 0, s,
                           n_rows, indptr, rowid);
        GCN_LAUNCH_CHECK("rowid_kernel");
    }
    const uint32_t *kin = nullptr;
    uint32_t *kout = ka;
    const int32_t *rows = rowid;
    const uint32_t mask = (1u << p.dbits) - 1u;
    for (int pass = 0; pass < p.passes; ++pass) {
        const int shift = pass * p.dbits;
        {
            ProfScope ps(K_T_COUNT, s, 0.0, (double)nnz * 4.0);
            hipLaunchKernelGGL(hist_kernel, dim3(p.ntiles), dim3(kTB), 0, s, nnz, indices, kin, shift, mask, p.ntiles,
                               hist);
            GCN_LAUNCH_CHECK("hist_kernel");
        }
        {
            ProfScope ps(K_T_SCAN, s, 0.0, (double)p.ntiles * (mask + 1) * 8.0);
            hipLaunchKernelGGL(scan_tiles_kernel, dim3(mask + 1), dim3(kTB), 0, s, p.ntiles, hist, total);
            GCN_LAUNCH_CHECK("scan_tiles_kernel");
        }
        {
            ProfScope ps(K_T_FILL, s, 0.0, (double)nnz * 24.0);
            // pairs are left by every other pass, counted from the last
            const bool to_pairs = (p.passes - pass) % 2 == 0;
            auto kernel = !to_pairs && pass > 0 ? scatter_kernel<true> : scatter_kernel<false>;
            hipLaunchKernelGGL(kernel, dim3(p.ntiles), dim3(kTB), 0, s, nnz, indices, kin, rows, vals, pairs, shift,
                               p.dbits, p.ntiles, hist, total, kout, to_pairs ? pairs : nullptr, t_indices, t_vals);
            GCN_LAUNCH_CHECK("scatter_kernel");
        }
        kin = kout;
        kout = kout == ka ? kb : ka;
        rows = t_indices;
        vals = t_vals;
    }
    {
        ProfScope ps(K_T_FINAL, s, 0.0, (double)(n_cols + 1) * 4.0);
        hipLaunchKernelGGL(bounds_kernel, dim3((unsigned)((n_cols + 1 + kTB - 1) / kTB)), dim3(kTB), 0, s,
                           n_cols, nnz, kin, t_indptr);
        GCN_LAUNCH_CHECK("bounds_kernel");
    }
    return GCN_OK;
}

size_t transpose_symmetric_workspace_bytes(int32_t n, int32_t nnz) {
    (void)nnz;
    return 2 * align256((size_t)n * 4) + 256;
}

int csr_transpose_symmetric(int32_t n, int32_t nnz, const int32_t *indptr, IdxRef indices,
                            const float *vals, float *t_vals, void *ws, size_t ws_bytes, hipStream_t s) {
    if (n == 0 || nnz == 0) return GCN_OK;
    Arena ar(ws, ws_bytes);
    uint32_t *rowval = ar.take<uint32_t>(n);
    int32_t *rowconst = ar.take<int32_t>(n);
    if (!rowval || !rowconst) {
        set_error("csr_transpose_symmetric: workspace too small (%zu < %zu bytes)", ws_bytes,
                  transpose_symmetric_workspace_bytes(n, nnz));
        return GCN_EWORKSPACE;
    }
    ProfScope ps(K_T_SYM, s, 0.0, (double)nnz * 12.0 + (double)n * 16.0);
    hipLaunchKernelGGL(sym_rows_kernel, dim3((unsigned)((n + kTB / 16 - 1) / (kTB / 16))), dim3(kTB), 0, s, n,
                       indptr, vals, rowval, rowconst);
    unsigned g = (unsigned)std::min<int64_t>(((int64_t)nnz + kTB - 1) / kTB, 16384);
    hipLaunchKernelGGL(sym_vals_kernel, dim3(g), dim3(kTB), 0, s, n, nnz, indptr, indices, vals, rowval,
                       rowconst, t_vals);
    GCN_LAUNCH_CHECK("transpose_symmetric kernels");
    return GCN_OK;
}

// ------------------------------------------------------- content check
// The first violation in row order, as a 64-bit key for an integer atomicMin
// (the minimum is unique, so the result does not depend on timing):
//   endpoints:        key = which (0: indptr[0] != 0, 1: indptr[n_rows] != nnz)
//   row r decreasing: key = (r + 1) << 32
//   row r, entry q (q-th of the row) out of range / not ascending:
//                     key = (r + 1) << 32 | (1 + 2q + (not ascending))
namespace {
constexpr int64_t kValidKey = 0x7fffffffffffffffLL;

__global__ void validate_init_kernel(int64_t *key) { *key = kValidKey; }

__global__ __launch_bounds__(256) void validate_rows_kernel(int32_t n_rows, int32_t n_cols, int32_t nnz,
                                                            const int32_t *__restrict__ indptr,
                                                            IdxRef indices, int sorted,
                                                            int64_t *__restrict__ key) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r == 0 && lane == 0) {
        if (indptr[0] != 0) atomicMin((long long *)key, 0LL);
        if (indptr[n_rows] != nnz) atomicMin((long long *)key, 1LL);
    }
    if (r >= n_rows) return;
    const int32_t b = indptr[r], e = indptr[r + 1];
    const int64_t base = (r + 1) << 32;
    if (e < b) {
        if (lane == 0) atomicMin((long long *)key, (long long)base);
        return;
    }
    if (b < 0 || e > nnz) return;   // then an endpoint or a decrease is reported elsewhere
    // the row's first bad entry: lanes take entries b + lane, b + lane + 64, ...
    int64_t mine = kValidKey;
    for (int64_t p = (int64_t)b + lane; p < e; p += 64) {
        const int32_t j = indices[p];
        int bad = -1;
        if (j < 0 || j >= n_cols) bad = 0;
        else if (sorted && p > b && indices[p - 1] >= j) bad = 1;
        if (bad >= 0) {
            mine = base | (1 + 2 * (p - b) + bad);
            break;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int64_t other = __shfl_xor(mine, o);
        mine = other < mine ? other : mine;
    }
    if (lane == 0 && mine != kValidKey) atomicMin((long long *)key, (long long)mine);
}

// status[0] = code (0 valid, 1 endpoints, 2 indptr decreases, 3 index out of
// range, 4 not ascending), status[1] = row (0 or n_rows for endpoints)
__global__ void validate_final_kernel(int32_t n_rows, int64_t *key_status) {
    const int64_t key = *key_status;
    int32_t code = 0, row = 0;
    if (key != kValidKey) {
        const int64_t r = (key >> 32) - 1;
        const int64_t sub = key & 0xffffffffLL;
        if (r < 0) {
            code = 1;
            row = sub == 0 ? 0 : n_rows;
        } else {
            row = (int32_t)r;
            code = sub == 0 ? 2 : (((sub - 1) & 1) ? 4 : 3);
        }
    }
    int32_t *st = (int32_t *)key_status;
    st[0] = code;
    st[1] = row;
}
}  // namespace

int csr_validate_device(int32_t n_rows, int32_t n_cols, int32_t nnz, const int32_t *indptr,
                        IdxRef indices, int sorted, int32_t *status, hipStream_t s) {
    int64_t *key = (int64_t *)status;
    hipLaunchKernelGGL(validate_init_kernel, dim3(1), dim3(1), 0, s, key);
    GCN_LAUNCH_CHECK("validate_init_kernel");
    const int64_t blocks = ((int64_t)n_rows + 3) / 4;
    hipLaunchKernelGGL(validate_rows_kernel, dim3((unsigned)(blocks > 0 ? blocks : 1)), dim3(256), 0, s, n_rows,
                       n_cols, nnz, indptr, indices, sorted, key);
    GCN_LAUNCH_CHECK("validate_rows_kernel");
    hipLaunchKernelGGL(validate_final_kernel, dim3(1), dim3(1), 0, s, n_rows, key);
    GCN_LAUNCH_CHECK("validate_final_kernel");
    return GCN_OK;
}

}  // namespace gcn
