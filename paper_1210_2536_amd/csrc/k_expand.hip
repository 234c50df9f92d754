// CSR column panels in two steps: x expanded panel by panel, then row sums.
//
// What bounds the short rows of a matrix with random columns is not HBM but
// the rate at which an XCD's L2 answers one request per gathered element
// (160-200 G gathers/s on the GPU, less once x leaves the 4 MB L2, about
// 100 G/s for an x of 32 MB).  Here no gather goes to L2:
//
//   expand  x is cut into panels of kExpandBytes.  A workgroup copies its
//           panel into LDS and writes xe[k] = x[column of k] for its share of
//           the panel's entries k, in the order (panel, row block): a 16-bit
//           panel offset in, a value of x out, both streams contiguous.
//   rows    a workgroup takes a row block (consecutive rows with at most
//           kRowsThreads * PER entries), copies the block's pieces of xe
//           into LDS (one contiguous run per panel, 8 bytes to say where;
//           4 bytes per piece until then cost 4-6% of the matrices below),
//           and walks the block's entries in row order, each naming its LDS
//           slot with 16 bits.
//
// Both gathers are LDS reads, so an entry costs 2 + s bytes in the first
// step and 2 s + 2 in the second, all of it streamed.  x is only copied in between, so a row is summed in float64 from
// the same products as in any other CSR kernel.
//
// Measured (MI355X): uniform 33 a row, n = 730k, float32 33 + 48 us (5.2 and
// 5.3 TB/s), float64 52 + 79 us, where slot-major ELL takes 118 and 190 us and
// the XCD panels 143 and 222 us; the 7.98M rows of up to 1024 entries of a Zipf
// matrix with n = 8M, float32, 117 + 240 us for 968 + 102 us by XCD panels.
// Rows as plain blocks of 16384 (8192 float64) entries: shrinking the blocks
// so that their number fills the last round of resident workgroups was no
// faster (n = 300k float32 39 -> 44 us: a block's fixed cost outweighs the
// half-empty round).
//
// Long rows by tiles (tiles_device.hpp) run in the same two launches: their
// workgroups hold a panel of x as well, and their sums run beside the row
// blocks.  Two launches instead of four: n = 310k float32 41 -> 37 us, n =
// 700k float64 404 -> 391 us, n = 1M float64 with 5M entries 45 -> 39 us.
//
// Row sums: a thread takes PER consecutive entries whatever their rows, with
// a bit per entry marking where a row starts; the piece of a row that
// crosses threads is carried by a segmented scan over the wave and, through
// LDS, over the workgroup, in a fixed order.  A block is cut between rows, so
// no sum leaves it.  The float64 chain of a row is at most PER + 6 + 16 + its
// share of threads.
#include "tiles_device.hpp"

#include <algorithm>
#include <climits>

namespace smat {
namespace {

constexpr int kExpandThreads = kTileThreads;
constexpr int kExpandBytes = kTileBytes;   // x per panel: two workgroups fill a CU's LDS
constexpr int kRowsThreads = 1024;
constexpr int kRunsAhead = 4;         // runs of xe that a lane requests together
constexpr int kRowsPieces = 5100;     // 16-byte pieces of xe per row block, at most
// Behind a block's pieces lies one of zeros: its first value is the slot of an
// entry that adds zero, its second that of the entry standing for a row which
// another kernel writes.
static_assert((kRowsPieces + 1) * 16 + 256 <= 81920, "two row workgroups fill a CU's LDS");
static_assert((kRowsPieces + 1) * 4 < 65536, "slots must fit 16 bits");

// G: values per 16-byte piece.
template <typename T> constexpr int kPiece = 16 / (int)sizeof(T);

// Entry `pos` of row block b belongs to thread pos / PER; the entries of a
// wave are interleaved in vectors of V (16 bytes), so that a wave's loads of
// "my next V entries" are one contiguous KiB.
template <int PER, int V>
__host__ __device__ __forceinline__ int64_t expand_at(int64_t b, int pos) {
    const int t = pos / PER, j = pos % PER;
    return ((b * (kRowsThreads / kWave) + t / kWave) * (PER / V) + j / V) * (kWave * V) +
           t % kWave * V + j % V;
}
constexpr int kSlotVec = 8;   // 16-bit slots per 16 bytes

// xe pieces [begin, end) per workgroup, panel after panel; G 16-bit offsets
// in, G values of x out per lane and piece, kExpandAhead pieces in flight.
constexpr int kExpandAhead = 4;

template <typename T> struct ExpandArgs {
    const ExpandChunk *__restrict__ chunks;
    const int32_t *__restrict__ starts;
    const uint16_t *__restrict__ off;
    const T *__restrict__ x;
    int64_t n;
    T *__restrict__ xe;
};

template <typename T, bool NT>
__device__ __forceinline__ void expand_block(const ExpandArgs<T> &a, unsigned bid,
                                             unsigned char *smem) {
    constexpr int G = kPiece<T>;
    typedef T vec __attribute__((ext_vector_type(G)));
    typedef uint16_t ovec __attribute__((ext_vector_type(G)));
    const ExpandChunk ch = a.chunks[bid];
    const ovec *ov = reinterpret_cast<const ovec *>(a.off);
    vec *out = reinterpret_cast<vec *>(a.xe);
    vec *xv = reinterpret_cast<vec *>(smem);
    const T *xs = reinterpret_cast<const T *>(smem);
    int64_t begin = ch.begin;
    for (int p = ch.panel; begin < ch.end; ++p) {
        const int64_t stop = a.starts[p + 1], end = stop < ch.end ? stop : ch.end;
        if (begin >= end) continue;   // a panel without entries
        const int64_t c0 = (int64_t)p * (kExpandBytes / (int)sizeof(T));
        if (p != ch.panel) __syncthreads();   // the panel before is done with
        copy_panel<T>(a.x, a.n, c0, xv);
        __syncthreads();
        constexpr int U = kExpandAhead;
        int64_t v = begin + (int)threadIdx.x;
        for (; v + (U - 1) * kExpandThreads < end; v += U * kExpandThreads) {
            ovec o[U];
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] = ld<NT>(ov + v + u * kExpandThreads);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                vec w;
#pragma unroll
                for (int e = 0; e < G; ++e) w[e] = xs[o[u][e]];
                out[v + u * kExpandThreads] = w;
            }
        }
        for (; v < end; v += kExpandThreads) {
            const ovec o = ld<NT>(ov + v);
            vec w;
#pragma unroll
            for (int e = 0; e < G; ++e) w[e] = xs[o[e]];
            out[v] = w;
        }
        begin = end;
    }
}

// First launch: workgroups [0, tiles) take the long rows' tiles, if the plan
// has any, the others the first step; both hold a panel of x, and the second
// kind fills the compute units that the last round of tiles leaves.
template <typename T, bool NT>
__global__ __launch_bounds__(kExpandThreads, 8) void k_panel_expand(ExpandArgs<T> a,
                                                                    unsigned tiles,
                                                                    TileArgs<T> ta) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ TileLds lds;
    if (blockIdx.x < tiles)
        tile_block<T, NT>(ta, blockIdx.x, smem, lds);
    else
        expand_block<T, NT>(a, blockIdx.x - tiles, smem);
}

// Row block b of the second step.  meta[b * threads + t]: bit j of the low
// half set when entry j of thread t starts a row, the high half the rows
// started before the thread's first entry.  The workgroups from `sums` on add
// the long rows' panel partials, kRowsThreads / 256 groups of kReduceRows rows
// each.
template <typename T, int PER, bool NT>
__global__ __launch_bounds__(kRowsThreads, 8) void k_panel_rows(
    const ExpandBlock *__restrict__ blocks, const uint32_t *__restrict__ meta,
    const uint16_t *__restrict__ slot, const T *__restrict__ val,
    const int2 *__restrict__ runs, int P, int lr, int pieces_stride, const T *__restrict__ xe,
    T *__restrict__ y, unsigned sums, int64_t n7, int64_t nparts,
    const int32_t *__restrict__ lrows, const double *__restrict__ part) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (blockIdx.x >= sums) {
        constexpr int kThreads = kReduceRows * kReduceGroups, kParts = kRowsThreads / kThreads;
        typedef double gs_t[kReduceGroups][kReduceRows];
        const unsigned sub = threadIdx.x / kThreads;
        tiles_reduce_block<T>((blockIdx.x - sums) * kParts + sub, threadIdx.x % kThreads, n7, nparts,
                              lrows, part, y, reinterpret_cast<gs_t *>(smem)[sub]);
        return;
    }
    __shared__ double wtail[kRowsThreads / kWave];
    __shared__ unsigned wflag[kRowsThreads / kWave];
    constexpr int G = kPiece<T>;
    typedef T vec __attribute__((ext_vector_type(G)));
    constexpr int SV = kSlotVec;
    typedef uint32_t svec __attribute__((ext_vector_type(SV / 2)));   // two slots a word
    const int t = threadIdx.x, lane = t & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const int64_t b = blockIdx.x;
    const ExpandBlock blk = blocks[b];
    const int zero = pieces_stride * G;   // slot holding +0.0
    vec *xv = reinterpret_cast<vec *>(smem);
    const T *xs = reinterpret_cast<const T *>(smem);
    // the thread's entries and the block's pieces of xe, all requested before
    // any is used
    const uint32_t mw = meta[b * kRowsThreads + t];
    svec sl[PER / SV];
    vec vv[PER / G];
#pragma unroll
    for (int q = 0; q < PER / SV; ++q)
#pragma unroll
        for (int e = 0; e < SV / 2; ++e) sl[q][e] = (unsigned)zero * 0x10001u;
#pragma unroll
    for (int q = 0; q < PER / G; ++q)
#pragma unroll
        for (int e = 0; e < G; ++e) vv[q][e] = T(0);
    if (t * PER < blk.entries) {
#pragma unroll
        for (int q = 0; q < PER / SV; ++q)
            sl[q] = ld<NT>(reinterpret_cast<const svec *>(
                slot + expand_at<PER, SV>(b, t * PER + q * SV)));
#pragma unroll
        for (int q = 0; q < PER / G; ++q)
            vv[q] = ld<NT>(reinterpret_cast<const vec *>(
                val + expand_at<PER, G>(b, t * PER + q * G)));
    }
    // the block's run of each panel by 1 << lr lanes, kRunsAhead runs of a lane at
    // once
    const vec *xp = reinterpret_cast<const vec *>(xe);
    const int2 *run = runs + b * P;
    constexpr int A = kRunsAhead;
    const int lanes = 1 << lr, groups = kRowsThreads >> lr;
    for (int p0 = t >> lr; p0 < P; p0 += A * groups) {
        int32_t from[A], to[A], left[A], most = 0;
#pragma unroll
        for (int q = 0; q < A; ++q) {
            const int p = p0 + q * groups;
            const int2 d = p < P ? run[p] : int2{0, 0};
            const int i = t & (lanes - 1);
            from[q] = d.x + i;
            to[q] = (d.y & 0xFFFF) + i;
            left[q] = (int)((unsigned)d.y >> 16) - i;
            most = max(most, left[q]);
        }
        for (int o = 0; o < most; o += lanes) {
            vec w[A];
#pragma unroll
            for (int q = 0; q < A; ++q)
                if (o < left[q]) w[q] = xp[from[q] + o];
#pragma unroll
            for (int q = 0; q < A; ++q)
                if (o < left[q]) xv[to[q] + o] = w[q];
        }
    }
    if (t == 0) {
        vec z;
#pragma unroll
        for (int e = 0; e < G; ++e) z[e] = T(0);
        xv[pieces_stride] = z;
    }
    __syncthreads();

    const unsigned flags = mw & 0xFFFFu;
    const int before = (int)(mw >> 16);   // rows started before this thread
    T *yb = y + blk.row0;
    double acc = 0.0, head = 0.0;
    int r = before - 1;                   // the row open now
    bool skip = false;                    // it is a row another kernel writes
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const unsigned s = sl[j / SV][j % SV / 2] >> (j % 2 * 16) & 0xFFFFu;
        if (flags >> j & 1u) {
            if (r < before)
                head = acc;
            else if (!skip)
                yb[r] = (T)acc;
            acc = 0.0;
            ++r;
            skip = s == (unsigned)zero + 1u;
        }
        acc = fma((double)vv[j / G][j % G], (double)xs[s], acc);
    }
    // rows across threads: acc is the sum of the row still open (of all
    // entries if the thread starts no row)
    const bool any = flags != 0;
    const unsigned long long bal = __ballot(any);
    double tail;
    double carry = wave_carry(acc, bal, lane, &tail);
    const int sk = __shfl_up((int)skip, 1, kWave);
    if (lane == kWave - 1) {
        wtail[wave] = tail;
        wflag[wave] = (bal ? 1u : 0u) | (skip ? 2u : 0u);
    }
    __syncthreads();
    // the piece carried into the wave by the waves before it
    bool prev_skip = sk != 0;
    if (wave > 0 && !(bal & ((1ull << lane) - 1ull))) {
        double w = 0.0;
        for (int q = wave - 1; q >= 0; --q) {
            w += wtail[q];
            if (wflag[q] & 1u) break;
        }
        carry += w;
    }
    if (lane == 0) prev_skip = wave > 0 && (wflag[wave - 1] & 2u);
    // a row another kernel writes is one entry, so it is open here only when
    // it was the entry before this thread's first
    if (any && before > 0 && !prev_skip) yb[before - 1] = (T)(carry + head);
    if (t == kRowsThreads - 1 && r < blk.rows) {   // no padding: the block's last row ends here
        if (!any) {
            yb[r] = (T)(carry + acc);
        } else if (!skip) {
            yb[r] = (T)acc;
        }
    }
}

// ------------------------------------------------------------ plan time

// Entries a row takes in its block: its own, or one that stands for an empty
// row (value 0, the zero slot) or for a row left to another kernel.
__device__ __forceinline__ int expand_slots(int32_t len, int32_t lmax) {
    return len == 0 || len > lmax ? 1 : len;
}

__global__ __launch_bounds__(256) void k_expand_lengths(int64_t m, const int32_t *__restrict__ rp,
                                                        int32_t lmax, int32_t *__restrict__ len) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < m) len[i] = expand_slots(rp[i + 1] - rp[i], lmax);
}

// first row of [0, m) whose entries start at or after v
__device__ __forceinline__ int64_t expand_lower_row(const int32_t *__restrict__ spos, int64_t m,
                                                    int64_t v) {
    int64_t lo = 0, hi = m;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (spos[mid] < v)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Row block b: the rows whose entries start in [b step, (b + 1) step).  Its
// pieces per panel into cnt[p * nb + b], their sum into blocks[b], the largest
// sum into stats[0], the panels that hold any, over all blocks, into stats[1].
template <int W, int G>
__global__ __launch_bounds__(1024) void k_expand_count(
    int64_t m, int64_t nb, int64_t step, int P, int32_t lmax, int lg,
    const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const int32_t *__restrict__ spos, ExpandBlock *__restrict__ blocks,
    int32_t *__restrict__ cnt, int *__restrict__ stats) {
    extern __shared__ int hist[];
    __shared__ int64_t rows[2];
    __shared__ int total, filled;
    const int64_t b = blockIdx.x;
    for (int p = threadIdx.x; p < P; p += 1024) hist[p] = 0;
    if (threadIdx.x < 2) rows[threadIdx.x] = expand_lower_row(spos, m, (b + threadIdx.x) * step);
    if (threadIdx.x == 0) total = filled = 0;
    __syncthreads();
    const int64_t r0 = rows[0], r1 = rows[1];
    const int lanes = 1 << lg, lane = threadIdx.x & (lanes - 1);
    for (int64_t r = r0 + (threadIdx.x >> lg); r < r1; r += 1024 >> lg) {
        const int32_t e0 = rp[r], e1 = rp[r + 1];
        if (e1 - e0 > lmax) continue;
        for (int32_t e = e0 + lane; e < e1; e += lanes) atomicAdd(&hist[col[e] / W], 1);
    }
    __syncthreads();
    int sum = 0, any = 0;
    for (int p = threadIdx.x; p < P; p += 1024) {
        const int c = (hist[p] + G - 1) / G;
        cnt[(int64_t)p * nb + b] = c;
        sum += c;
        any += c > 0;
    }
    if (sum) {
        atomicAdd(&total, sum);
        atomicAdd(&filled, any);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        blocks[b] = ExpandBlock{(int32_t)r0, (int32_t)(r1 - r0), spos[r1] - spos[r0], total};
        atomicMax(&stats[0], total);
        atomicAdd(&stats[1], filled);
    }
}

__global__ void k_expand_starts(int P, int64_t nb, const int32_t *__restrict__ runs,
                                int32_t *__restrict__ starts) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p <= P) starts[p] = runs[(int64_t)p * nb];
}

// The entries of row block b into both steps' arrays.  Where an entry lies
// within its piece of (panel, block) does not matter for the result (the
// row-order walk names its slot), so the places come from LDS counters.
template <typename U, int W, int G, int PER>
__global__ __launch_bounds__(1024) void k_expand_fill(
    int64_t m, int64_t nb, int P, int32_t lmax, int lg, const int32_t *__restrict__ rp,
    const int32_t *__restrict__ col, const U *__restrict__ val,
    const int32_t *__restrict__ spos, const ExpandBlock *__restrict__ blocks,
    const int32_t *__restrict__ runs, int pieces_stride, uint16_t *__restrict__ off,
    uint32_t *__restrict__ meta, uint16_t *__restrict__ slot, U *__restrict__ oval,
    int2 *__restrict__ run) {
    extern __shared__ int lds[];
    // per panel: entries placed, first piece in LDS, first piece of all
    int *cur = lds, *base = lds + P, *first = lds + 2 * P;
    __shared__ unsigned bits[1024 * PER / 32];  // row starts
    __shared__ int scan[1024];
    const int t = threadIdx.x;
    const int64_t b = blockIdx.x;
    const ExpandBlock blk = blocks[b];
    const int64_t r0 = blk.row0, r1 = r0 + blk.rows;
    const int32_t s0 = spos[r0];
    const uint16_t zero = (uint16_t)(pieces_stride * G);
    for (int i = t; i < 1024 * PER / 32; i += 1024) bits[i] = 0;
    // exclusive scan of the panels' piece counts, 1024 panels at a time
    int carry = 0;
    for (int p0 = 0; p0 < P; p0 += 1024) {
        const int p = p0 + t;
        const int c = p < P ? runs[(int64_t)p * nb + b + 1] - runs[(int64_t)p * nb + b] : 0;
        scan[t] = c;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            const int a = t >= o ? scan[t - o] : 0;
            __syncthreads();
            scan[t] += a;
            __syncthreads();
        }
        if (p < P) {
            base[p] = carry + scan[t] - c;
            first[p] = runs[(int64_t)p * nb + b];
            cur[p] = 0;
        }
        carry += scan[1023];
        __syncthreads();
    }
    const int lanes = 1 << lg, lane = t & (lanes - 1);
    for (int64_t r = r0 + (t >> lg); r < r1; r += 1024 >> lg) {
        const int32_t e0 = rp[r], e1 = rp[r + 1];
        const int pos = spos[r] - s0;
        if (lane == 0) {
            atomicOr(&bits[pos / 32], 1u << (pos % 32));
            if (e1 == e0 || e1 - e0 > lmax) {
                slot[expand_at<PER, kSlotVec>(b, pos)] = e1 == e0 ? zero : (uint16_t)(zero + 1);
                oval[expand_at<PER, G>(b, pos)] = 0;
            }
        }
        if (e1 - e0 > lmax) continue;
        for (int32_t e = e0 + lane; e < e1; e += lanes) {
            const int c = col[e], p = c / W;
            const int k = atomicAdd(&cur[p], 1);
            const int i = pos + (e - e0);
            slot[expand_at<PER, kSlotVec>(b, i)] = (uint16_t)(base[p] * G + k);
            oval[expand_at<PER, G>(b, i)] = val[e];
            off[(int64_t)first[p] * G + k] = (uint16_t)(c - p * W);
        }
    }
    // padding up to the end of the last thread's entries starts a row past
    // the block's
    const int end = (blk.entries + PER - 1) / PER * PER;
    for (int i = blk.entries + t; i < end; i += 1024) {
        slot[expand_at<PER, kSlotVec>(b, i)] = zero;
        oval[expand_at<PER, G>(b, i)] = 0;
    }
    if (t == 0 && blk.entries < 1024 * PER) atomicOr(&bits[blk.entries / 32], 1u << (blk.entries % 32));
    __syncthreads();
    for (int p = t; p < P; p += 1024) {
        const int64_t s = first[p];
        const int c = runs[(int64_t)p * nb + b + 1] - (int)s;
        for (int k = cur[p]; k < c * G; ++k) off[s * G + k] = 0;
        run[b * P + p] = int2{(int32_t)s, (int)((unsigned)base[p] | (unsigned)c << 16)};
    }
    const unsigned w = bits[t * PER / 32] >> (t * PER % 32) & ((1u << PER) - 1u);
    scan[t] = __popc(w);
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int a = t >= o ? scan[t - o] : 0;
        __syncthreads();
        scan[t] += a;
        __syncthreads();
    }
    meta[b * 1024 + t] = w | (unsigned)(scan[t] - __popc(w)) << 16;
}

// CSR entries of the rows in blocks, rebuilt from the two steps' arrays: an
// entry's slot lies in its panel's run, which says where the entry's offset is.
template <typename U, int W, int G, int PER>
__global__ __launch_bounds__(1024) void k_expand_to_csr(
    int P, int32_t lmax, const int32_t *__restrict__ rp, const ExpandBlock *__restrict__ blocks,
    const uint16_t *__restrict__ off, const uint16_t *__restrict__ slot,
    const U *__restrict__ oval, const int2 *__restrict__ runs, int32_t *__restrict__ col,
    U *__restrict__ val) {
    const int64_t b = blockIdx.x;
    const ExpandBlock blk = blocks[b];
    if (threadIdx.x) return;
    const int2 *run = runs + b * P;
    int q = 0;
    for (int64_t r = blk.row0; r < (int64_t)blk.row0 + blk.rows; ++r) {
        const int32_t e0 = rp[r], len = rp[r + 1] - e0;
        if (len == 0 || len > lmax) {
            ++q;
            continue;
        }
        for (int32_t e = 0; e < len; ++e, ++q) {
            const int s = slot[expand_at<PER, kSlotVec>(b, q)], k = s / G;
            int lo = 0, hi = P - 1;   // last panel whose run starts at or before the piece
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if ((run[mid].y & 0xFFFF) <= k)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            const int64_t at = run[lo].x + (k - (run[lo].y & 0xFFFF));
            col[e0 + e] = lo * W + off[at * G + s % G];
            val[e0 + e] = oval[expand_at<PER, G>(b, q)];
        }
    }
}

}  // namespace

int64_t expand_width(int elt) { return kExpandBytes / elt; }
int expand_per(int elt) { return 64 / elt; }
int64_t expand_block_entries(int elt) { return (int64_t)kRowsThreads * expand_per(elt); }
int expand_max_pieces() { return kRowsPieces; }

// Lanes (a power of two, its logarithm) that copy a run of one panel's pieces,
// from the pieces, the runs that hold any and the blocks.  Steps of one
// workgroup, each of which waits for memory: its P runs by groups of lanes, and
// as many more as the runs of such a step are longer than the lanes.  Spread
// columns (all runs alike) keep the mean run's lanes, at most a wave; where a
// block's entries lie in a few panels their runs take up to the whole
// workgroup.  By 64 lanes a run | this: 12 columns a row within 50000 of 1M
// float32 58 | 49 us, float64 77 | 74; 280 within 20000 of 150k 187 | 124 and
// 379 | 265.
int expand_run_lanes(int P, int64_t nb, int64_t pieces, int64_t runs) {
    int lr = 0;
    while (lr < 6 && ((int64_t)P * nb << lr) <= pieces) ++lr;
    if (runs * 4 > (int64_t)P * nb * 3) return lr;
    const double run = (double)pieces / (double)std::max<int64_t>(1, runs);
    const double filled = (double)runs / (double)nb;
    double best = 1e300;
    for (int l = 0; (1 << l) <= kRowsThreads; ++l) {
        const double at_once = (double)kRunsAhead * (kRowsThreads >> l);
        const double steps = std::ceil(P / at_once) + (std::ceil(run / (1 << l)) - 1.0) *
                                                          std::ceil(filled / at_once);
        if (steps < best) {
            best = steps;
            lr = l;
        }
    }
    return lr;
}

spmv_status expand_prepare() {
#define ATTR(F, BYTES)                                                                      \
    SMAT_HIP(hipFuncSetAttribute((const void *)(F), hipFuncAttributeMaxDynamicSharedMemorySize, \
                                 (int)(BYTES)))
    ATTR((k_panel_expand<float, false>), kTileLds);
    ATTR((k_panel_expand<float, true>), kTileLds);
    ATTR((k_panel_expand<double, false>), kTileLds);
    ATTR((k_panel_expand<double, true>), kTileLds);
    ATTR((k_panel_rows<float, 16, false>), (kRowsPieces + 1) * 16);
    ATTR((k_panel_rows<float, 16, true>), (kRowsPieces + 1) * 16);
    ATTR((k_panel_rows<double, 8, false>), (kRowsPieces + 1) * 16);
    ATTR((k_panel_rows<double, 8, true>), (kRowsPieces + 1) * 16);
#undef ATTR
    return SPMV_OK;
}

spmv_status launch_expand_lengths(int64_t m, const int32_t *rp, int32_t lmax, int32_t *len,
                                  hipStream_t s) {
    if (m == 0) return SPMV_OK;
    k_expand_lengths<<<(unsigned)((m + 255) / 256), 256, 0, s>>>(m, rp, lmax, len);
    SMAT_LAUNCHED("expand_lengths");
    return SPMV_OK;
}

spmv_status launch_expand_count(int elt, int64_t m, int64_t nb, int64_t step, int P, int32_t lmax,
                                int lg, const int32_t *rp, const int32_t *col,
                                const int32_t *spos, ExpandBlock *blocks, int32_t *cnt, int *stats,
                                hipStream_t s) {
    const size_t sh = sizeof(int) * (size_t)P;
    if (elt == 8)
        k_expand_count<kExpandBytes / 8, 2><<<(unsigned)nb, 1024, sh, s>>>(
            m, nb, step, P, lmax, lg, rp, col, spos, blocks, cnt, stats);
    else
        k_expand_count<kExpandBytes / 4, 4><<<(unsigned)nb, 1024, sh, s>>>(
            m, nb, step, P, lmax, lg, rp, col, spos, blocks, cnt, stats);
    SMAT_LAUNCHED("expand_count");
    return SPMV_OK;
}

spmv_status launch_expand_starts(int P, int64_t nb, const int32_t *runs, int32_t *starts,
                                 hipStream_t s) {
    k_expand_starts<<<(unsigned)(P / 256 + 1), 256, 0, s>>>(P, nb, runs, starts);
    SMAT_LAUNCHED("expand_starts");
    return SPMV_OK;
}

spmv_status launch_expand_fill(int elt, int64_t m, int64_t nb, int P, int32_t lmax, int lg,
                               const int32_t *rp, const int32_t *col, const void *val,
                               const int32_t *spos, const ExpandBlock *blocks,
                               const int32_t *runs, int pieces_stride, uint16_t *off,
                               uint32_t *meta, uint16_t *slot, void *oval, int2 *run,
                               hipStream_t s) {
    const size_t sh = 3 * sizeof(int) * (size_t)P;
    if (elt == 8)
        k_expand_fill<uint64_t, kExpandBytes / 8, 2, 8><<<(unsigned)nb, 1024, sh, s>>>(
            m, nb, P, lmax, lg, rp, col, (const uint64_t *)val, spos, blocks, runs, pieces_stride,
            off, meta, slot, (uint64_t *)oval, run);
    else
        k_expand_fill<uint32_t, kExpandBytes / 4, 4, 16><<<(unsigned)nb, 1024, sh, s>>>(
            m, nb, P, lmax, lg, rp, col, (const uint32_t *)val, spos, blocks, runs, pieces_stride,
            off, meta, slot, (uint32_t *)oval, run);
    SMAT_LAUNCHED("expand_fill");
    return SPMV_OK;
}

spmv_status launch_expand_to_csr(int elt, int64_t nb, int P, int32_t lmax, const int32_t *rp,
                                 const ExpandBlock *blocks, const uint16_t *off,
                                 const uint16_t *slot, const void *oval, const int2 *runs,
                                 int32_t *col, void *val, hipStream_t s) {
    if (nb == 0) return SPMV_OK;
    if (elt == 8)
        k_expand_to_csr<uint64_t, kExpandBytes / 8, 2, 8><<<(unsigned)nb, 64, 0, s>>>(
            P, lmax, rp, blocks, off, slot, (const uint64_t *)oval, runs, col, (uint64_t *)val);
    else
        k_expand_to_csr<uint32_t, kExpandBytes / 4, 4, 16><<<(unsigned)nb, 64, 0, s>>>(
            P, lmax, rp, blocks, off, slot, (const uint32_t *)oval, runs, col, (uint32_t *)val);
    SMAT_LAUNCHED("expand_to_csr");
    return SPMV_OK;
}

template <typename T, int PER>
static spmv_status expand_dispatch(const ExpandRun &r, const TileRun *t, const T *x, int64_t n,
                                   T *y, hipStream_t s) {
    const ExpandArgs<T> a{r.chunks, r.starts, r.off, x, n, (T *)r.xe};
    TileArgs<T> ta{};
    unsigned tiles = 0, sum_blocks = 0;
    if (t) {
        ta = TileArgs<T>{t->n7, t->P, t->blocks, t->start, t->meta, t->off, (const T *)t->val, x,
                         n, t->part};
        tiles = (unsigned)(t->P * t->nblocks);
        constexpr int kPer = kReduceRows * (kRowsThreads / (kReduceRows * kReduceGroups));
        sum_blocks = (unsigned)((t->n7 + kPer - 1) / kPer);
    }
    const unsigned first = tiles + (unsigned)r.nchunks;
    if (first > 0) {
        if (r.nt1 || (t && t->nt))
            k_panel_expand<T, true><<<first, kExpandThreads, kTileLds, s>>>(a, tiles, ta);
        else
            k_panel_expand<T, false><<<first, kExpandThreads, kTileLds, s>>>(a, tiles, ta);
        SMAT_LAUNCHED("panel_expand");
    }
    const unsigned second = (unsigned)r.nb + sum_blocks;
    if (second > 0) {
        const size_t sums_lds = sum_blocks ? sizeof(double) * kRowsThreads : 0;
        const size_t sh = std::max(((size_t)r.stride + 1) * 16, sums_lds);
#define ROWS(NT)                                                                             \
    k_panel_rows<T, PER, NT><<<second, kRowsThreads, sh, s>>>(                               \
        r.blocks, r.meta, r.slot, (const T *)r.val, r.runs, r.P, r.lr, r.stride,                     (const T *)r.xe, y,                                                                  \
        (unsigned)r.nb, t ? t->n7 : 0, t ? t->P : 0, t ? t->rows : nullptr, t ? t->part : nullptr)
        if (r.nt)
            ROWS(true);
        else
            ROWS(false);
#undef ROWS
        SMAT_LAUNCHED("panel_rows");
    }
    return SPMV_OK;
}

spmv_status run_expand(int elt, const ExpandRun &r, const TileRun *t, const void *x, int64_t n,
                       void *y, hipStream_t s) {
    if (r.stride < 0 || r.stride > kRowsPieces || r.nb > INT32_MAX || r.nchunks > INT32_MAX) {
        set_error("expanded panels: %d pieces per row block", r.stride);
        return SPMV_EINVAL;
    }
    if (t) SMAT_TILES_OK(*t, elt);
    if ((t ? t->P * t->nblocks : 0) + r.nchunks > INT32_MAX) {
        set_error("expanded panels: too many workgroups");
        return SPMV_EINVAL;
    }
    return elt == 8 ? expand_dispatch<double, 8>(r, t, (const double *)x, n, (double *)y, s)
                    : expand_dispatch<float, 16>(r, t, (const float *)x, n, (float *)y, s);
}

}  // namespace smat
