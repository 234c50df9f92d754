// K0 CSR validation and K1 feature extraction (paper Section 3: CSR input;
// Section 4, Table 3: the feature parameters; Section 6: staged extraction).
//
// Entry-parallel passes give every thread a short contiguous run of
// nonzeros, so work is balanced over nnz whatever the row-length distribution
// (the same nnz-balanced split the paper uses for its threads, Section 6).  A
// wave takes a contiguous share of the entries in chunks of 64 runs; it finds
// the rows a chunk spans with 64 probes of row_ptr at a time, walking on from
// the chunk before, and a lane the row of its first entry by binary search
// among those.
//
// What bounds these passes is not their bytes (5.3M entries are 21 MB) but
// atomics on one address, served one after the other (about 10 ns each), and
// chains of dependent loads: with an atomic per wave and a binary search over
// all rows per 8 entries, the checks took 135 us, the row statistics 44 and the
// diagonal totals 45 on a 220k x 220k matrix of 5.3M entries.  So few, large
// workgroups, one atomic each and only where it changes the word, and the row
// pass joined to the checks: 36 us for checks and statistics, 6 for the totals.
#include "internal.hpp"

#include <algorithm>
#include <climits>

namespace smat {
namespace {

constexpr int kEntryRun = 8;      // nonzeros per thread in entry passes
constexpr int kBlock = 256;
constexpr int kHash = 1024;       // LDS hash slots for the diagonal census
constexpr int kStatsBlock = 1024;
constexpr int kStatsGrid = 512;   // two such workgroups a compute unit
constexpr int kRowHistLds = 1024; // row-length bins kept in LDS

// Largest i in [lo, m) with rp[i] <= p, given that lo is one (or 0), by the
// whole wave: 64 probes a round at steps of `step` (a power of 64, at least
// (m - lo) / 64 or growing until a probe fails), then at smaller steps.  With
// a valid row_ptr this is the row that holds entry p (empty rows have rp[i] ==
// rp[i+1] and lose); with any other it stays in [0, m).
__device__ __forceinline__ int64_t wave_row(const int32_t *__restrict__ rp, int64_t m, int64_t lo,
                                            int64_t p, int64_t step) {
    const int lane = threadIdx.x & (kWave - 1);
    bool grow = true;
    for (;;) {
        const int64_t pos = lo + (lane + 1) * step;
        const unsigned long long hit = __ballot(pos < m && rp[pos < m ? pos : 0] <= p);
        const int cnt = hit == ~0ull ? kWave : __ffsll((long long)~hit) - 1;
        lo += cnt * step;
        if (cnt == kWave && grow) {
            step *= kWave;
            continue;
        }
        grow = false;
        if (step == 1) return lo;
        step /= kWave;
    }
}

// Calls f(p0, len, c, row) for each thread's runs of entries [p0, p0 + len), c
// holding their columns and the entry's after them (0 past the end), row
// being the row of entry p0.  f returns whether the wave should go on.
template <typename F>
__device__ __forceinline__ void walk_runs(int64_t m, int64_t nnz, const int32_t *__restrict__ rp,
                                          const int32_t *__restrict__ col, F f) {
    constexpr int64_t kChunk = (int64_t)kWave * kEntryRun;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    const int64_t w = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave;
    const int64_t chunks = (nnz + kChunk - 1) / kChunk, per = (chunks + waves - 1) / waves;
    const int64_t c0 = w * per, c1 = c0 + per < chunks ? c0 + per : chunks;
    int64_t first = 0, step = 1;
    while (step * kWave < m) step *= kWave;
    for (int64_t c = c0; c < c1; ++c) {
        const int64_t q0 = c * kChunk, q1 = q0 + kChunk < nnz ? q0 + kChunk : nnz;
        const int64_t p0 = q0 + lane * kEntryRun;
        const int len = (int)(p0 >= q1 ? 0 : q1 - p0 < kEntryRun ? q1 - p0 : kEntryRun);
        int32_t v[kEntryRun + 1];
        if (len == kEntryRun) {
            __builtin_memcpy(v, col + p0, sizeof(int32_t) * kEntryRun);
        } else {
#pragma unroll
            for (int j = 0; j < kEntryRun; ++j) v[j] = j < len ? col[p0 + j] : 0;
        }
        v[kEntryRun] = p0 + kEntryRun < nnz ? col[p0 + kEntryRun] : 0;
        first = wave_row(rp, m, first, q0, c == c0 ? step : 1);
        // the next rows' starts, one a lane: most chunks span fewer than 64
        // rows, and the lanes' rows are then found by shuffles
        const int64_t pos = first + 1 + lane;
        const int32_t start = pos < m ? rp[pos] : INT_MAX;
        int64_t row;
        if (__shfl(start, kWave - 1) > q1 - 1) {
            int k = 0;
#pragma unroll
            for (int h = kWave / 2; h > 0; h >>= 1)
                if (__shfl(start, k + h - 1) <= p0) k += h;
            row = first + k;
        } else {
            int64_t last = wave_row(rp, m, first, q1 - 1, 1);
            row = first;
            while (row < last) {
                const int64_t mid = (row + last + 1) >> 1;
                if (rp[mid] <= p0)
                    row = mid;
                else
                    last = mid - 1;
            }
        }
        if (!f(p0, len, v, row)) return;
    }
}

template <typename T, typename Op>
__device__ T block_reduce(T v, Op op, T *lds, T identity) {
    // wave reduction by xor shuffles, then across the waves of the block
    for (int off = kWave / 2; off > 0; off >>= 1) v = op(v, __shfl_xor(v, off, kWave));
    int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (lane == 0) lds[w] = v;
    __syncthreads();
    int nw = blockDim.x / kWave;
    if (w == 0) {
        v = lane < nw ? lds[lane] : identity;
        for (int off = kWave / 2; off > 0; off >>= 1) v = op(v, __shfl_xor(v, off, kWave));
    }
    __syncthreads();
    return v;  // valid in thread 0
}

struct OpAdd { template <typename T> __device__ T operator()(T a, T b) const { return a + b; } };

__device__ __forceinline__ int load_word(const int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The CSR checks with the row statistics and the bandwidth max |j - i|, which
// mean something once the checks pass.  flags: row_ptr; flags2: columns.  The
// entries are walked beside the row_ptr check, so the walk stays in bounds
// whatever row_ptr holds: rows are only looked up in rp[0..m] (m >= 1
// whenever nnz > 0) and columns only read below nnz; a row_ptr that ends a
// row past the last one is flagged as out of order.
//
// Bound by latency: the search for the first row, then columns, row starts and
// the next row's end one after the other, and at the end one cache line that
// every workgroup updates.  4.4M entries in 20 us; 34 with a barrier pair per
// statistic and an atomic for each.
//
// One workgroup a compute unit up to kCheckMany entries, two above: each ends
// on that line.  Measured (256 | 512 workgroups): 4.4M entries 19.5 | 25.3 us,
// 11.7M 30.9 | 33.6, 27M 87 | 68.
constexpr int kCheckBlock = 1024, kCheckGrid = 512;
constexpr int64_t kCheckMany = int64_t(1) << 24;

__global__ __launch_bounds__(kCheckBlock) void k_check(int64_t m, int64_t n, int64_t nnz,
                                                       const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col,
                                                       uint32_t *flags, uint32_t *flags2,
                                                       RowStats *rs, int *bandwidth) {
    constexpr int kWaves = kCheckBlock / kWave;
    __shared__ unsigned long long w2[kWaves];
    __shared__ int wx[kWaves], wn[kWaves], wb[kWaves];
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t threads = (int64_t)gridDim.x * blockDim.x;
    uint32_t bad = 0, bad2 = 0;
    unsigned long long s2 = 0;
    int mx = 0, mn = INT_MAX, bw = 0;
    for (int64_t i = t; i <= m; i += threads) {
        const int32_t v = rp[i];
        if (i == 0 && v != 0) bad |= kBadRowPtr0;
        if (i == m && (int64_t)v != nnz) bad |= kBadRowPtrEnd;
        if (v < 0 || (int64_t)v > nnz) bad |= kBadRowPtrOrder;
        if (i < m) {
            const int32_t k = rp[i + 1] - v;
            if (rp[i + 1] < v) bad |= kBadRowPtrOrder;
            s2 += (unsigned long long)k * (unsigned long long)k;
            mx = k > mx ? k : mx;
            mn = k < mn ? k : mn;
        }
    }
    walk_runs(m, nnz, rp, col, [&](int64_t p0, int len, const int32_t *c, int64_t row) {
        if (len == 0) return true;
        int64_t rend = rp[row + 1];
#pragma unroll
        for (int j = 0; j < kEntryRun; ++j) {
            const int64_t p = p0 + j;
            if (j >= len) continue;
            while (p >= rend && row + 1 < m) rend = rp[++row + 1];
            if (p >= rend) {   // entries beyond rp[m]: a broken row_ptr
                bad2 |= kBadRowPtrOrder;
                continue;
            }
            if (c[j] < 0 || (int64_t)c[j] >= n) bad2 |= kBadColRange;
            if (p + 1 < rend && p + 1 < nnz && c[j + 1] <= c[j]) bad2 |= kBadColOrder;
            const int64_t d = (int64_t)c[j] - row;
            const int ad = (int)(d < 0 ? -d : d);
            bw = ad > bw ? ad : bw;
        }
        return true;
    });
    if (bad) atomicOr(flags, bad);
    if (bad2) atomicOr(flags2, bad2);
    // all four across the workgroup with one exchange
    auto wave = [&](int from) {
        for (int off = from; off > 0; off >>= 1) {
            s2 += __shfl_xor(s2, off, kWave);
            mx = max(mx, __shfl_xor(mx, off, kWave));
            mn = min(mn, __shfl_xor(mn, off, kWave));
            bw = max(bw, __shfl_xor(bw, off, kWave));
        }
    };
    wave(kWave / 2);
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (lane == 0) {
        w2[w] = s2;
        wx[w] = mx;
        wn[w] = mn;
        wb[w] = bw;
    }
    __syncthreads();
    if (w > 0) return;
    s2 = lane < kWaves ? w2[lane] : 0ull;
    mx = lane < kWaves ? wx[lane] : 0;
    mn = lane < kWaves ? wn[lane] : INT_MAX;
    bw = lane < kWaves ? wb[lane] : 0;
    wave(kWaves / 2);
    if (lane == 0) {
        // the rows' lengths add up to nnz wherever the checks pass
        if (blockIdx.x == 0) rs->sum_rd = (unsigned long long)nnz;
        // what the others found so far, read together: an atomic that changes
        // nothing is left out, and the words of all workgroups lie in one line
        const int gx = load_word(&rs->max_rd), gn = load_word(&rs->min_rd), gb = load_word(bandwidth);
        atomicAdd(&rs->sum_rd2, s2);
        if (mx > gx) atomicMax(&rs->max_rd, mx);
        if (mn < gn) atomicMin(&rs->min_rd, mn);
        if (bw > gb) atomicMax(bandwidth, bw);
    }
}

__global__ void k_row_hist(int64_t m, const int32_t *__restrict__ rp, int max_rd,
                           unsigned int *hist) {
    __shared__ unsigned int h[kRowHistLds];
    int nl = max_rd + 1 < kRowHistLds ? max_rd + 1 : kRowHistLds;
    for (int b = threadIdx.x; b < nl; b += blockDim.x) h[b] = 0;
    __syncthreads();
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x) {
        int k = rp[i + 1] - rp[i];
        if (k < kRowHistLds)
            atomicAdd(&h[k], 1u);
        else
            atomicAdd(&hist[k], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nl; b += blockDim.x)
        if (h[b]) atomicAdd(&hist[b], h[b]);
}

// Least-squares fit of ln(count_k / m) on ln k over k >= 1 with count_k > 0
// (Section 4, parameter R).  One workgroup, fixed summation order, centred
// second pass.  sums = {count, mean_x, mean_y, sxy, sxx}.
__global__ void k_powerlaw_fit(const unsigned int *__restrict__ hist, int max_rd, int64_t m,
                               double *sums) {
    __shared__ double lds[1024 / kWave];
    double c = 0, sx = 0, sy = 0;
    double dm = (double)m;
    for (int k = 1 + threadIdx.x; k <= max_rd; k += blockDim.x) {
        unsigned int h = hist[k];
        if (h) {
            c += 1.0;
            sx += log((double)k);
            sy += log((double)h / dm);
        }
    }
    c = block_reduce(c, OpAdd(), lds, 0.0);
    sx = block_reduce(sx, OpAdd(), lds, 0.0);
    sy = block_reduce(sy, OpAdd(), lds, 0.0);
    __shared__ double mean[3];
    if (threadIdx.x == 0) {
        mean[0] = c;
        mean[1] = c > 0 ? sx / c : 0.0;
        mean[2] = c > 0 ? sy / c : 0.0;
    }
    __syncthreads();
    double xb = mean[1], yb = mean[2];
    double sxy = 0, sxx = 0;
    for (int k = 1 + threadIdx.x; k <= max_rd; k += blockDim.x) {
        unsigned int h = hist[k];
        if (h) {
            double dx = log((double)k) - xb;
            double dy = log((double)h / dm) - yb;
            sxy += dx * dy;
            sxx += dx * dx;
        }
    }
    sxy = block_reduce(sxy, OpAdd(), lds, 0.0);
    sxx = block_reduce(sxx, OpAdd(), lds, 0.0);
    if (threadIdx.x == 0) {
        sums[0] = mean[0];
        sums[1] = xb;
        sums[2] = yb;
        sums[3] = sxy;
        sums[4] = sxx;
    }
}

// Does row r (sorted columns [rp[r], rp[r+1])) hold a column in [lo, lo+3]?
__device__ __forceinline__ bool row_has_block(const int32_t *__restrict__ rp,
                                              const int32_t *__restrict__ col, int64_t r,
                                              int32_t lo) {
    int64_t a = rp[r], b = rp[r + 1];
    while (a < b) {  // first entry >= lo
        int64_t mid = (a + b) >> 1;
        if (col[mid] < lo)
            a = mid + 1;
        else
            b = mid;
    }
    return a < rp[r + 1] && col[a] <= lo + 3;
}

// BLOCKS: count the nonempty aligned 4x4 blocks (a few binary searches per
// block start); with a histogram, take the diagonal census.  Either or both.
//
// A census launched together with the CSR checks (gate, gate_rs non-NULL)
// runs only when both checks passed (gate[0] | gate[1] == 0) and the
// zero-fill bound still allows DIA (max_RD M <= 20 NNZ); the checks and the
// row pass precede it on the stream.  Every thread reads the same words, so
// a workgroup leaves as a whole.
//
// Census: counts gather in an LDS table and reach the histogram once per
// workgroup.  A matrix of many diagonals fills the table at once; its entries
// then either go straight to the histogram (spill NULL), or the census stops,
// *spill is set and the histogram void: the bitmap census below takes over.
constexpr int kProbes = 4;

template <bool BLOCKS>
__global__ __launch_bounds__(kStatsBlock) void k_entry_stats(
    int64_t m, int64_t n, int64_t nnz, const int32_t *__restrict__ rp,
    const int32_t *__restrict__ col, EntryStats *out, unsigned int *diag_hist,
    const uint32_t *gate, const RowStats *gate_rs, uint32_t *spill) {
    if (gate && (gate[0] | gate[1])) return;
    if (gate_rs && (int64_t)gate_rs->max_rd * m > 20 * nnz) return;
    __shared__ int spilled;
    __shared__ int hkey[kHash + kProbes];
    __shared__ unsigned int hcnt[kHash + kProbes];
    __shared__ unsigned long long lds_u[kStatsBlock / kWave];
    const bool census = diag_hist != nullptr;
    if (census) {
        for (int b = threadIdx.x; b < kHash + kProbes; b += blockDim.x) {
            hkey[b] = INT_MIN;
            hcnt[b] = 0;
        }
        if (threadIdx.x == 0) spilled = 0;
        __syncthreads();
    }
    unsigned long long nb = 0;
    walk_runs(m, nnz, rp, col, [&](int64_t p0, int len, const int32_t *c, int64_t row) {
        const bool count = census && !__builtin_amdgcn_readfirstlane(__hip_atomic_load(
                                         &spilled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
        if (!BLOCKS && !count) return false;
        if (len == 0) return true;
        int64_t rbeg = rp[row], rend = rp[row + 1];
        int32_t prev = BLOCKS && p0 > rbeg ? col[p0 - 1] : 0;
#pragma unroll
        for (int j = 0; j < kEntryRun; ++j) {
            if (j >= len) continue;
            const int64_t p = p0 + j;
            while (p >= rend) {
                ++row;
                rbeg = rend;
                rend = rp[row + 1];
            }
            if (BLOCKS) {  // first entry of its aligned 4x4 block, in row-major order?
                const int32_t lo = c[j] & ~3;
                bool fresh = !(p > rbeg && (prev & ~3) == lo);
                for (int64_t r2 = row & ~(int64_t)3; fresh && r2 < row; ++r2)
                    if (row_has_block(rp, col, r2, lo)) fresh = false;
                nb += fresh;
                prev = c[j];
            }
            if (count) {
                const int64_t d = (int64_t)c[j] - row;
                const int key = (int)d;
                const unsigned h = ((unsigned int)key * 2654435761u) >> 22;  // 10 bits
                bool done = false;
#pragma unroll
                for (int q = 0; q < kProbes; ++q) {
                    int have = hkey[h + q];
                    if (!done && have == INT_MIN) have = atomicCAS(&hkey[h + q], INT_MIN, key);
                    if (!done && (have == INT_MIN || have == key)) {
                        atomicAdd(&hcnt[h + q], 1u);
                        done = true;
                    }
                }
                if (!done) {
                    if (spill)
                        __hip_atomic_store(&spilled, 1, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                    else
                        atomicAdd(&diag_hist[d + m - 1], 1u);
                }
            }
        }
        return true;
    });
    if (BLOCKS) {
        nb = block_reduce(nb, OpAdd(), lds_u, 0ull);
        if (threadIdx.x == 0) atomicAdd(&out->blocks4, nb);
    }
    if (census) {
        __syncthreads();
        if (spill && spilled) {
            if (threadIdx.x == 0 && !load_word(reinterpret_cast<const int *>(spill)))
                atomicOr(spill, 1u);
            return;
        }
        for (int b = threadIdx.x; b < kHash + kProbes; b += blockDim.x)
            if (hcnt[b]) atomicAdd(&diag_hist[(int64_t)hkey[b] + m - 1], hcnt[b]);
    }
}

// ---- bitmap census, for matrices whose diagonals spill the table
// One random count after the other into a histogram of m + n - 1 words goes at
// 25 G/s (atomics on scattered words): 208 us for 5.3M entries.  Here
//   bits    each of up to kBitsGrid workgroups marks the diagonals of its share
//           of the entries in an LDS bitmap and writes the bitmap out;
//   merge   the bitmaps are joined, and a diagonal's count is bounded by the
//           rows of the shares it occurs in: where 5 bound <= 3 length it is
//           not true, and its entries need no counting;
//   count   the entries of the other diagonals are counted (the corners'
//           short diagonals, and those that are nearly full).
// All exact; 19 + 18 + 22 us for those entries (and 16 until the table spills).
// Bitmaps beyond one workgroup's LDS are made in kBitsParts parts, each walking
// the entries again, from kPartsMinNnz entries on: 11.7M random entries of
// 730k rows 56 + 43 + 43 us where the histogram took 440 (about 170 at the
// line, as long as the bitmaps take there).
constexpr int kBitsBlock = 1024, kBitsGrid = 256, kBitsParts = 2;
constexpr int64_t kPartsMinNnz = int64_t(1) << 22;

__global__ __launch_bounds__(kBitsBlock) void k_diag_bits(int64_t m, int64_t nnz, int words,
                                                          const int32_t *__restrict__ rp,
                                                          const int32_t *__restrict__ col,
                                                          const uint32_t *__restrict__ spill,
                                                          uint32_t *__restrict__ maps,
                                                          int *__restrict__ rows) {
    if (!*spill) return;
    extern __shared__ uint32_t bits[];
    __shared__ int r0, r1;
    // this workgroup's part of the diagonals
    const int pw = (words + (int)gridDim.y - 1) / (int)gridDim.y, w0 = (int)blockIdx.y * pw;
    const int wn = min(pw, words - w0);
    if (threadIdx.x == 0) {
        r0 = INT_MAX;
        r1 = -1;
    }
    for (int w = threadIdx.x; w < wn; w += kBitsBlock) bits[w] = 0;
    __syncthreads();
    int64_t lo = INT64_MAX, hi = -1;
    walk_runs(m, nnz, rp, col, [&](int64_t p0, int len, const int32_t *c, int64_t row) {
        if (len == 0) return true;
        lo = row < lo ? row : lo;
        int64_t rend = rp[row + 1];
#pragma unroll
        for (int j = 0; j < kEntryRun; ++j) {
            if (j >= len) continue;
            while (p0 + j >= rend) rend = rp[++row + 1];
            const int64_t b = (int64_t)c[j] - row + m - 1;
            const unsigned at = (unsigned)((int)(b >> 5) - w0);
            if (at < (unsigned)wn) atomicOr(&bits[at], 1u << (b & 31));
        }
        hi = row > hi ? row : hi;
        return true;
    });
    if (hi >= 0) {
        atomicMin(&r0, (int)lo);
        atomicMax(&r1, (int)hi);
    }
    __syncthreads();
    uint32_t *out = maps + (int64_t)blockIdx.x * words + w0;
    for (int w = threadIdx.x; w < wn; w += kBitsBlock) out[w] = bits[w];
    if (threadIdx.x == 0 && w0 == 0) rows[blockIdx.x] = r1 >= 0 ? r1 - r0 + 1 : 0;
}

// A workgroup per 32 words: the joined words, the words of diagonals to count,
// and zero counts.
__global__ __launch_bounds__(256) void k_diag_merge(int64_t m, int64_t n, int words, int nmaps,
                                                    const uint32_t *__restrict__ spill,
                                                    const uint32_t *__restrict__ maps,
                                                    const int *__restrict__ rows,
                                                    uint32_t *__restrict__ seen,
                                                    uint32_t *__restrict__ cand,
                                                    unsigned *__restrict__ hist) {
    if (!*spill) return;
    __shared__ uint32_t part[kBitsGrid][33];   // 32 words of every bitmap
    __shared__ int srows[kBitsGrid];
    const int w0 = blockIdx.x * 32, t = threadIdx.x;
    constexpr int kPer = kBitsGrid * 32 / 256, kAhead = 8;
    for (int q = 0; q < kPer && q * 8 < nmaps; q += kAhead) {
        uint32_t v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int k = (q + u) * 8 + t / 32, w = w0 + t % 32;
            v[u] = k < nmaps && w < words ? maps[(int64_t)k * words + w] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) part[(q + u) * 8 + t / 32][t % 32] = v[u];
    }
    for (int k = t; k < nmaps; k += 256) srows[k] = rows[k];
    __syncthreads();
    const int64_t nb = m + n - 1;
    // thread (word, bit group): 32 words, 8 groups of 4 bits
    const int w = t & 31, g = t / 32;
    int bound[4] = {0, 0, 0, 0};
#pragma unroll 8
    for (int k = 0; k < nmaps; ++k) {
        const uint32_t v = part[k][w] >> (4 * g);
        const int r = srows[k];
#pragma unroll
        for (int e = 0; e < 4; ++e) bound[e] += r & -(int)(v >> e & 1u);
    }
    uint32_t have = 0, want = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t b = (int64_t)(w0 + w) * 32 + 4 * g + e;
        if (b >= nb) continue;
        const int64_t d = b - (m - 1);
        const int64_t len = (m < n - d ? m : n - d) - (d < 0 ? -d : 0);
        if (bound[e]) have |= 1u << (4 * g + e);
        if (5 * (int64_t)bound[e] > 3 * len) want |= 1u << (4 * g + e);
        hist[b] = 0;
    }
    __syncthreads();
    part[g][w] = have;
    part[g + 8][w] = want;
    __syncthreads();
    if (t < 32 && w0 + t < words) {
        uint32_t a = 0, c = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            a |= part[k][t];
            c |= part[k + 8][t];
        }
        seen[w0 + t] = a;
        cand[w0 + t] = c;
    }
}

// Counts of the diagonals marked in cand.
__global__ __launch_bounds__(kStatsBlock) void k_diag_count(int64_t m, int64_t nnz,
                                                            const int32_t *__restrict__ rp,
                                                            const int32_t *__restrict__ col,
                                                            const uint32_t *__restrict__ spill,
                                                            const uint32_t *__restrict__ cand,
                                                            unsigned *__restrict__ hist) {
    if (!*spill) return;
    walk_runs(m, nnz, rp, col, [&](int64_t p0, int len, const int32_t *c, int64_t row) {
        if (len == 0) return true;
        int64_t rend = rp[row + 1];
#pragma unroll
        for (int j = 0; j < kEntryRun; ++j) {
            if (j >= len) continue;
            while (p0 + j >= rend) rend = rp[++row + 1];
            const int64_t b = (int64_t)c[j] - row + m - 1;
            if (cand[b >> 5] >> (b & 31) & 1u) atomicAdd(&hist[b], 1u);
        }
        return true;
    });
}

// Occupied diagonals and "true" diagonals (5 count > 3 length).  After the
// bitmap census (*spill) the occupied ones are those in seen, and those whose
// counts were not needed get a count of one: occupied, not true.
constexpr int kDiagGrid = 128;

__global__ __launch_bounds__(kStatsBlock) void k_diag_stats(int64_t m, int64_t n,
                                                            unsigned int *__restrict__ hist,
                                                            const uint32_t *__restrict__ spill,
                                                            const uint32_t *__restrict__ seen,
                                                            DiagStats *out) {
    __shared__ unsigned long long lds[kStatsBlock / kWave];
    unsigned long long nd = 0, nt = 0;
    const int64_t nb = m + n - 1;
    const bool bitmap = spill && *spill;
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < nb;
         b += (int64_t)gridDim.x * blockDim.x) {
        unsigned int c = hist[b];
        if (c) {
            int64_t d = b - (m - 1);
            int64_t len = (m < n - d ? m : n - d) - (d < 0 ? -d : 0);
            nd += 1;
            nt += 5ull * c > 3ull * (unsigned long long)len;
        } else if (bitmap && (seen[b >> 5] >> (b & 31) & 1u)) {
            nd += 1;
            hist[b] = 1;
        }
    }
    nd = block_reduce(nd, OpAdd(), lds, 0ull);
    nt = block_reduce(nt, OpAdd(), lds, 0ull);
    if (threadIdx.x == 0 && nd) {
        atomicAdd(&out->ndiags, nd);
        if (nt) atomicAdd(&out->ntrue, nt);
    }
}

constexpr int kCompactPer = 16;   // bins per thread in the compaction

__global__ void k_diag_count_blocks(int64_t nbins, const unsigned int *__restrict__ hist,
                                    unsigned int *block_counts) {
    __shared__ unsigned int lds[kBlock / kWave];
    int64_t base = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) * kCompactPer;
    unsigned int c = 0;
    for (int q = 0; q < kCompactPer; ++q)
        if (base + q < nbins && hist[base + q]) ++c;
    c = block_reduce(c, OpAdd(), lds, 0u);
    if (threadIdx.x == 0) block_counts[blockIdx.x] = c;
}

// Exclusive scan of `count` values in place by one workgroup of 1024 threads.
__global__ void k_scan_single(unsigned int *v, int64_t count) {
    __shared__ unsigned int part[1024];
    __shared__ unsigned int carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < count; base += 1024) {
        int64_t i = base + threadIdx.x;
        unsigned int x = i < count ? v[i] : 0;
        part[threadIdx.x] = x;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            unsigned int add = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
            __syncthreads();
            part[threadIdx.x] += add;
            __syncthreads();
        }
        unsigned int incl = part[threadIdx.x];
        if (i < count) v[i] = carry + incl - x;
        __syncthreads();
        if (threadIdx.x == 1023) carry += incl;
        __syncthreads();
    }
}

// Write the offsets of the occupied histogram bins, ascending.
__global__ void k_diag_write(int64_t m, int64_t nbins, const unsigned int *__restrict__ hist,
                             const unsigned int *__restrict__ block_base, int32_t *offsets) {
    __shared__ unsigned int part[kBlock];
    int64_t base = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) * kCompactPer;
    unsigned int c = 0;
    for (int q = 0; q < kCompactPer; ++q)
        if (base + q < nbins && hist[base + q]) ++c;
    part[threadIdx.x] = c;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        unsigned int add = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    unsigned int slot = block_base[blockIdx.x] + part[threadIdx.x] - c;
    for (int q = 0; q < kCompactPer; ++q) {
        int64_t b = base + q;
        if (b < nbins && hist[b]) {
            offsets[slot] = (int32_t)(b - (m - 1));
            ++slot;
        }
    }
}

inline unsigned int grid_for(int64_t work, int block, int64_t cap = 1 << 20) {
    int64_t g = (work + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned int)g;
}

}  // namespace

spmv_status launch_check(int64_t m, int64_t n, int64_t nnz, const int32_t *rp, const int32_t *col,
                         uint32_t *flags, uint32_t *flags2, RowStats *rs, int *bandwidth,
                         hipStream_t s) {
    // enough threads for a row or a run of entries each, in whole workgroups
    const int64_t work = std::max(m + 1, (nnz + kEntryRun - 1) / kEntryRun);
    const int64_t most = std::max(m, nnz) < kCheckMany ? kCheckGrid / 2 : kCheckGrid;
    k_check<<<grid_for(work, kCheckBlock, most), kCheckBlock, 0, s>>>(
        m, n, nnz, rp, col, flags, flags2, rs, bandwidth);
    SMAT_LAUNCHED("check");
    return SPMV_OK;
}

spmv_status launch_row_hist(int64_t m, const int32_t *rp, int max_rd, unsigned int *hist,
                            hipStream_t s) {
    if (m == 0) return SPMV_OK;
    k_row_hist<<<grid_for(m, kBlock, 2048), kBlock, 0, s>>>(m, rp, max_rd, hist);
    SMAT_LAUNCHED("row_hist");
    return SPMV_OK;
}

spmv_status launch_powerlaw_fit(const unsigned int *hist, int max_rd, int64_t m, double *sums,
                                hipStream_t s) {
    k_powerlaw_fit<<<1, 1024, 0, s>>>(hist, max_rd, m, sums);
    SMAT_LAUNCHED("powerlaw_fit");
    return SPMV_OK;
}

spmv_status launch_entry_stats(int64_t m, int64_t n, int64_t nnz, const int32_t *rp,
                               const int32_t *col, EntryStats *out, unsigned int *diag_hist,
                               bool blocks, hipStream_t s, const uint32_t *gate,
                               const RowStats *gate_rs, uint32_t *spill) {
    if (nnz == 0) return SPMV_OK;
    int64_t threads = (nnz + kEntryRun - 1) / kEntryRun;
    // the census alone: a table a compute unit fills and spills soonest (11.7M
    // random entries 13.0 us, 16.5 with two; the block count 188 with one, 139)
    const unsigned g = grid_for(threads, kStatsBlock, blocks ? kStatsGrid : kStatsGrid / 2);
    if (blocks)
        k_entry_stats<true><<<g, kStatsBlock, 0, s>>>(m, n, nnz, rp, col, out, diag_hist, gate,
                                                      gate_rs, spill);
    else
        k_entry_stats<false><<<g, kStatsBlock, 0, s>>>(m, n, nnz, rp, col, out, diag_hist, gate,
                                                       gate_rs, spill);
    SMAT_LAUNCHED("entry_stats");
    return SPMV_OK;
}

// Bitmaps of kBitsGrid shares, their rows, the joined and the candidate words.
static int bits_grid(int64_t nnz) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(kBitsGrid, nnz / 8192));
}

size_t diag_bitmap_bytes(int64_t m, int64_t n, int64_t nnz) {
    const int64_t words = (m + n - 1 + 31) / 32;
    if (words * 4 > kBitsParts * (int64_t)kDiagBitmapLds || nnz < kDiagBitmapMinNnz ||
        (words * 4 > kDiagBitmapLds && nnz < kPartsMinNnz))
        return 0;
    return sizeof(uint32_t) * (size_t)(words * (bits_grid(nnz) + 2) + kBitsGrid);
}

spmv_status launch_diag_bitmap(int64_t m, int64_t n, int64_t nnz, const int32_t *rp,
                               const int32_t *col, const uint32_t *spill, void *work,
                               unsigned int *diag_hist, hipStream_t s) {
    const int words = (int)((m + n - 1 + 31) / 32), g = bits_grid(nnz);
    uint32_t *seen = static_cast<uint32_t *>(work), *cand = seen + words, *maps = cand + words;
    int *rows = reinterpret_cast<int *>(maps + (int64_t)g * words);
    SMAT_HIP(hipFuncSetAttribute((const void *)k_diag_bits,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, kDiagBitmapLds));
    const int parts = (int)(((int64_t)words * 4 + kDiagBitmapLds - 1) / kDiagBitmapLds);
    k_diag_bits<<<dim3(g, parts), kBitsBlock, (size_t)((words + parts - 1) / parts) * 4, s>>>(
        m, nnz, words, rp, col, spill, maps, rows);
    SMAT_LAUNCHED("diag_bits");
    k_diag_merge<<<(words + 31) / 32, 256, 0, s>>>(m, n, words, g, spill, maps, rows, seen, cand,
                                                   diag_hist);
    SMAT_LAUNCHED("diag_merge");
    const int64_t threads = (nnz + kEntryRun - 1) / kEntryRun;
    k_diag_count<<<grid_for(threads, kStatsBlock, kStatsGrid), kStatsBlock, 0, s>>>(
        m, nnz, rp, col, spill, cand, diag_hist);
    SMAT_LAUNCHED("diag_count");
    return SPMV_OK;
}

spmv_status launch_diag_stats(int64_t m, int64_t n, unsigned int *diag_hist, DiagStats *out,
                              hipStream_t s, const uint32_t *spill, const void *work) {
    k_diag_stats<<<grid_for(m + n - 1, kStatsBlock, kDiagGrid), kStatsBlock, 0, s>>>(
        m, n, diag_hist, spill, static_cast<const uint32_t *>(work), out);
    SMAT_LAUNCHED("diag_stats");
    return SPMV_OK;
}

spmv_status launch_diag_compact(int64_t m, int64_t n, unsigned int *diag_hist, int32_t *offsets,
                                unsigned int *block_scratch, hipStream_t s) {
    int64_t nbins = m + n - 1;
    int64_t per_block = (int64_t)kBlock * kCompactPer;
    int64_t nblk = (nbins + per_block - 1) / per_block;
    k_diag_count_blocks<<<(unsigned)nblk, kBlock, 0, s>>>(nbins, diag_hist, block_scratch);
    SMAT_LAUNCHED("diag_count_blocks");
    k_scan_single<<<1, 1024, 0, s>>>(block_scratch, nblk);
    SMAT_LAUNCHED("scan_single");
    k_diag_write<<<(unsigned)nblk, kBlock, 0, s>>>(m, nbins, diag_hist, block_scratch, offsets);
    SMAT_LAUNCHED("diag_write");
    return SPMV_OK;
}

// Shared with the conversion file: exclusive scan of per-row counts into a
// row_ptr of m+1 entries.
namespace {
__global__ void k_block_sums(int64_t m, const int32_t *__restrict__ counts, unsigned int *bsum) {
    __shared__ unsigned int lds[kBlock / kWave];
    int64_t base = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) * kCompactPer;
    unsigned int c = 0;
    for (int q = 0; q < kCompactPer; ++q)
        if (base + q < m) c += (unsigned int)counts[base + q];
    c = block_reduce(c, OpAdd(), lds, 0u);
    if (threadIdx.x == 0) bsum[blockIdx.x] = c;
}

__global__ void k_scan_write(int64_t m, const int32_t *__restrict__ counts,
                             const unsigned int *__restrict__ bbase, int32_t *rp) {
    __shared__ unsigned int part[kBlock];
    int64_t base = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) * kCompactPer;
    unsigned int c = 0;
    for (int q = 0; q < kCompactPer; ++q)
        if (base + q < m) c += (unsigned int)counts[base + q];
    part[threadIdx.x] = c;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        unsigned int add = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    unsigned int run = bbase[blockIdx.x] + part[threadIdx.x] - c;
    for (int q = 0; q < kCompactPer; ++q) {
        int64_t i = base + q;
        if (i < m) {
            rp[i] = (int32_t)run;
            run += (unsigned int)counts[i];
        }
        if (i == m - 1) rp[m] = (int32_t)run;
    }
}
}  // namespace

spmv_status launch_exclusive_scan_rows(int64_t m, const int32_t *counts, int32_t *rp,
                                       unsigned int *scratch, hipStream_t s) {
    if (m == 0) {
        SMAT_HIP(hipMemsetAsync(rp, 0, sizeof(int32_t), s));
        return SPMV_OK;
    }
    int64_t per_block = (int64_t)kBlock * kCompactPer;
    int64_t nblk = (m + per_block - 1) / per_block;
    k_block_sums<<<(unsigned)nblk, kBlock, 0, s>>>(m, counts, scratch);
    SMAT_LAUNCHED("block_sums");
    k_scan_single<<<1, 1024, 0, s>>>(scratch, nblk);
    SMAT_LAUNCHED("scan_single");
    k_scan_write<<<(unsigned)nblk, kBlock, 0, s>>>(m, counts, scratch, rp);
    SMAT_LAUNCHED("scan_write");
    return SPMV_OK;
}

}  // namespace smat
