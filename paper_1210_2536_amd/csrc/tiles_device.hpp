// Long rows by x-panel tiles: the work of one workgroup, shared by the launch
// of its own (binned CSR) and the first launch of the two-step panels.
#pragma once

#include "spmv_device.hpp"

namespace smat {

// The long rows are cut into row blocks of about equal entry counts and x
// into panels of kTileBytes.  Workgroup (b, p) copies x panel p into LDS once
// and streams the entries of block b's rows in that panel, row after row (a
// row without entries there leaves one that adds zero), into one float64
// partial per (row, panel); k_long_tiles_reduce (or, in binned CSR, the first
// workgroups of k_csr_adaptive_tiles) adds a row's partials in a fixed order
// and rounds once.
//
// A thread takes TileShape::PER consecutive entries whatever their rows: their
// 16-bit offsets into the panel (2 + sizeof(T) bytes an entry) and values in
// 16-byte loads, contiguous over the wave, and a bit per entry where a row
// starts.  Pieces of a row in several threads are carried by a segmented scan
// over the wave and through LDS over the workgroup and its passes.  Lane
// groups per row, as this kernel had before, spend a pass of dependent loads
// (bounds, entries) on every few entries once the segments are short: 17
// entries each on the n = 8M Zipf matrix.  Measured on the rows above 1024
// entries: n = 8M float32 342 -> 171 us, n = 700k float64 (140 a segment) 352
// -> 292 us (1.66e8 entries, 6 TB/s), n = 310k float32 21 -> 19 us with the
// rows above 256 as well.  A next pass's entries requested before this one's
// carries, or all of x's LDS reads before the first addition, spill registers
// (64 for two workgroups a compute unit): 568 -> 580 and 547 -> 562 us on the
// whole n = 8M product.
//
// A float64 chain is at most PER + 6 + 16 + 2 passes, then the panels.
constexpr int kTileThreads = 1024;
// x per workgroup: two workgroups fill a CU's LDS, the carries' words included
constexpr int kTileBytes = 81920 - 512;
// behind the panel a piece of zeros, whose first value is the offset of an
// entry that adds zero
constexpr int kTileLds = kTileBytes + 16;
template <typename T> constexpr uint16_t kTileEmpty = kTileBytes / (int)sizeof(T);
static_assert(kTileBytes / 4 < 65536, "panel offsets must fit 16 bits");

// x[c0 .. c0 + panel) into LDS by the workgroup, zeros past n.  All of a
// thread's loads are requested before the first is stored: with the test for
// the end of x between them they came back one after the other, five times the
// memory latency a tile.
template <typename T>
__device__ __forceinline__ void copy_panel(
    const T *__restrict__ x, int64_t n, int64_t c0,
    T __attribute__((ext_vector_type(16 / sizeof(T)))) *xv) {
    constexpr int G = 16 / (int)sizeof(T), PIECES = kTileBytes / 16;
    constexpr int PER = (PIECES + kTileThreads - 1) / kTileThreads;
    typedef T vec __attribute__((ext_vector_type(G)));
    if (c0 + PIECES * G <= n) {
        vec w[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = q * kTileThreads + threadIdx.x;   // past the panel: its last piece
            __builtin_memcpy(&w[q], x + c0 + (k < PIECES ? k : PIECES - 1) * G, sizeof(vec));
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = q * kTileThreads + threadIdx.x;
            if (k < PIECES) xv[k] = w[q];
        }
        return;
    }
    for (int k = threadIdx.x; k < PIECES; k += kTileThreads) {
        vec w;
#pragma unroll
        for (int e = 0; e < G; ++e) {
            const int64_t j = c0 + (int64_t)k * G + e;
            w[e] = j < n ? x[j] : T(0);
        }
        xv[k] = w;
    }
}

// Dispatch order: panels fastest (workgroup w serves panel w mod P of row
// block w / P).  The workgroups in flight then cover a few row blocks across
// all panels and the GPU streams a small part of the matrix at a time.
template <typename T> struct TileArgs {
    int64_t n7, P;
    const TileBlock *__restrict__ blocks;
    const int32_t *__restrict__ start;
    const uint32_t *__restrict__ meta;
    const uint16_t *__restrict__ off;
    const T *__restrict__ val;
    const T *__restrict__ x;
    int64_t n;
    double *__restrict__ part;
};

// Carries between the waves of a pass, for this pass and the one before.
struct TileLds {
    double wtail[2][kTileThreads / kWave];
    unsigned wflag[2][kTileThreads / kWave];
    int wrows[2];
};
static_assert(sizeof(TileLds) + kTileLds <= 81920, "two workgroups fill a CU's LDS");

// Tile `bid` by the kTileThreads threads of a workgroup; smem: kTileLds bytes.
template <typename T, bool NT>
__device__ __forceinline__ void tile_block(const TileArgs<T> &a, unsigned bid,
                                           unsigned char *smem, TileLds &lds) {
    constexpr int kWaves = kTileThreads / kWave;
    constexpr int G = 16 / (int)sizeof(T);      // values per 16-byte piece
    constexpr int PER = TileShape<T>::PER, SV = 8;
    typedef T vec __attribute__((ext_vector_type(G)));
    typedef uint32_t svec __attribute__((ext_vector_type(SV / 2)));   // two offsets a word
    constexpr int PIECES = kTileBytes / 16;
    // the same for the whole workgroup: kept in scalar registers
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const unsigned P = (unsigned)a.P, b = bid / P, p = bid - b * P;
    const int u0 = uniform(a.start[bid]), u1 = uniform(a.start[bid + 1]);
    if (u0 == u1) return;   // no entries: the partials are zero since the plan was made
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    // the thread's entries of a pass, all requested before any is used
    unsigned flags;
    int before;
    svec o[PER / SV];
    vec vv[PER / G];
    auto request = [&](int64_t u) {
        flags = 0;
        before = 0;
#pragma unroll
        for (int q = 0; q < PER / SV; ++q)
#pragma unroll
            for (int e = 0; e < SV / 2; ++e) o[q][e] = kTileEmpty<T> * 0x10001u;
#pragma unroll
        for (int q = 0; q < PER / G; ++q)
#pragma unroll
            for (int e = 0; e < G; ++e) vv[q][e] = T(0);
        if (u < u1) {
            const uint32_t mw = ld<NT>(a.meta + u * kWave + (unsigned)lane);
            flags = mw & 0xFFFFu;
            before = (int)(mw >> 16);
#pragma unroll
            for (int q = 0; q < PER / SV; ++q)
                o[q] = ld<NT>(reinterpret_cast<const svec *>(
                    a.off + (u * (PER / SV) + q) * (kWave * SV) + (unsigned)(lane * SV)));
#pragma unroll
            for (int q = 0; q < PER / G; ++q)
                vv[q] = ld<NT>(reinterpret_cast<const vec *>(
                    a.val + (u * (PER / G) + q) * (kWave * G) + (unsigned)(lane * G)));
        }
    };
    const int64_t c0 = (int64_t)p * (kTileBytes / (int)sizeof(T));
    vec *xv = reinterpret_cast<vec *>(smem);
    copy_panel<T>(a.x, a.n, c0, xv);
    if (threadIdx.x == 0) {
        vec z;
#pragma unroll
        for (int e = 0; e < G; ++e) z[e] = T(0);
        xv[PIECES] = z;
    }
    __syncthreads();
    const T *xs = reinterpret_cast<const T *>(smem);
    const int rows = uniform(a.blocks[b].rows), row0 = uniform(a.blocks[b].row0);
    double *pp = a.part + (int64_t)p * a.n7 + row0;
    double open = 0.0;   // the row open at the start of the pass, so far
    int rbase = 0;       // rows started in the passes before
    int buf = 0;
    for (int ub = u0; ub < u1; ub += kWaves, buf ^= 1) {
        const int64_t u = (int64_t)ub + wave;
        request(u);
        double acc = 0.0, head = 0.0;
        const int first = rbase + before;   // row the thread's first flag starts
        int r = first - 1;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (flags >> j & 1u) {
                if (r < first)
                    head = acc;
                else
                    pp[r] = acc;
                acc = 0.0;
                ++r;
            }
            acc = fma((double)vv[j / G][j % G], (double)xs[o[j / SV][j % SV / 2] >> (j % 2 * 16) & 0xFFFFu], acc);
        }
        const bool any = flags != 0;
        const int started = before + __popc(flags);
        const unsigned long long bal = __ballot(any);
        double tail;
        double carry = wave_carry(acc, bal, lane, &tail);
        if (lane == kWave - 1) {
            lds.wtail[buf][wave] = tail;
            lds.wflag[buf][wave] = bal != 0;
            if (u == (ub + kWaves < u1 ? ub + kWaves : u1) - 1) lds.wrows[buf] = started;
        }
        __syncthreads();
        if (!(bal & ((1ull << lane) - 1ull))) {   // the row comes from waves before
            double w = 0.0;
            int q = wave - 1;
            for (; q >= 0; --q) {
                w += lds.wtail[buf][q];
                if (lds.wflag[buf][q]) break;
            }
            carry += q < 0 ? w + open : w;
        }
        if (any && first > 0) pp[first - 1] = carry + head;
        double w = 0.0;
        int q = kWaves - 1;
        for (; q >= 0; --q) {
            w += lds.wtail[buf][q];
            if (lds.wflag[buf][q]) break;
        }
        open = q < 0 ? w + open : w;
        rbase += lds.wrows[buf];
    }
    // without padding the last row ends with the entries
    if (threadIdx.x == 0 && rbase <= rows) pp[rbase - 1] = open;
}

// A long row's result: its panel partials added in a fixed order, rounded
// once.  A workgroup takes 32 rows; thread (g, i) adds the partials of panels
// g, g + 8, g + 16, ... of row i in that order (32 neighbouring rows per
// load, four of a thread's loads issued before their additions), and the
// eight group sums are added in group order.  Workgroup `bid` of such a
// reduction by the 256 threads t; every thread of the workgroup calls it.
constexpr int kReduceRows = 32, kReduceGroups = 8;

template <typename T>
__device__ __forceinline__ void tiles_reduce_block(unsigned bid, unsigned t, int64_t n7,
                                                   int64_t P,
                                                   const int32_t *__restrict__ rows,
                                                   const double *__restrict__ part,
                                                   T *__restrict__ y,
                                                   double (*gs)[kReduceRows]) {
    const int i = t % kReduceRows, g = t / kReduceRows;
    const int64_t r = (int64_t)bid * kReduceRows + i;
    double acc = 0.0;
    if (r < n7) {
        constexpr int G = kReduceGroups;
        int64_t p = g;
        for (; p + 3 * G < P; p += 4 * G) {
            const double v0 = part[p * n7 + r], v1 = part[(p + G) * n7 + r];
            const double v2 = part[(p + 2 * G) * n7 + r], v3 = part[(p + 3 * G) * n7 + r];
            acc += v0;
            acc += v1;
            acc += v2;
            acc += v3;
        }
        for (; p < P; p += G) acc += part[p * n7 + r];
    }
    gs[g][i] = acc;
    __syncthreads();
    if (g == 0 && r < n7) {
        double s = gs[0][i];
#pragma unroll
        for (int k = 1; k < kReduceGroups; ++k) s += gs[k][i];
        y[rows[r]] = (T)s;
    }
}

}  // namespace smat
