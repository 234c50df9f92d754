// K2 format conversions (paper Section 2.1: the four basic formats; Table 4
// and Section 4: ELL and DIA pay for zero fill) and K5 row binning for the
// length-adaptive CSR kernel.
//
// Layouts (Figure 1 did not survive; standard definitions):
//   COO  row index per stored entry, CSR order; columns and values are the
//        CSR arrays themselves.
//   ELL  K = max_RD slots per row, slot k of row i at k*m_pad + i (slot-major,
//        coalesced across rows); empty slots hold col -1 and value +0.0.
//   DIA  occupied diagonals d = j - i ascending; entry (i, i+off) at
//        slot*m_pad + i; absent slots hold +0.0; a presence bitmap (bit s of
//        uint32 word s >> 5) keeps explicit zeros distinguishable.
// Values are copied as raw bit patterns (uint32 / uint64), never through
// floating-point registers, so conversions are bit exact.
#include "internal.hpp"

#include <algorithm>

namespace smat {
namespace {

constexpr int kBlock = 256;
constexpr int kEntryRun = 8;

__device__ __forceinline__ int64_t row_of_entry(const int32_t *__restrict__ rp, int64_t m,
                                                int64_t p) {
    int64_t lo = 0, hi = m - 1;
    while (lo < hi) {
        int64_t mid = (lo + hi + 1) >> 1;
        if (rp[mid] <= p)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

inline unsigned grid_for(int64_t work, int block) {
    int64_t g = (work + block - 1) / block;
    return (unsigned)(g < 1 ? 1 : g);
}

__global__ void k_csr_to_coo(int64_t m, int64_t nnz, const int32_t *__restrict__ rp,
                             int32_t *__restrict__ row_idx) {
    int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    int64_t p0 = t * kEntryRun;
    if (p0 >= nnz) return;
    int64_t p1 = p0 + kEntryRun < nnz ? p0 + kEntryRun : nnz;
    int64_t row = row_of_entry(rp, m, p0);
    int64_t rend = rp[row + 1];
    for (int64_t p = p0; p < p1; ++p) {
        while (p >= rend) rend = rp[++row + 1];
        row_idx[p] = (int32_t)row;
    }
}

// A workgroup takes kEllRows rows: windows of 32 entries of each row are read
// 32 lanes a row (one or two cache lines a load), turned in LDS and written
// slot by slot, 64 rows a wave.  One thread a row, each walking its own part
// of the CSR arrays, took 103 us for 220k rows of 24 float64 entries (every load
// touching a cache line per lane), so 21.
constexpr int kEllRows = 64, kEllWindow = 32;

template <typename U>
__global__ __launch_bounds__(kBlock) void k_csr_to_ell(int64_t m, int64_t m_pad, int K,
                                                       const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col,
                                                       const U *__restrict__ val,
                                                       int32_t *__restrict__ ecol,
                                                       U *__restrict__ eval) {
    __shared__ int32_t sc[kEllRows][kEllWindow + 1];
    __shared__ U sv[kEllRows][kEllWindow + 1];
    __shared__ int32_t sb[kEllRows + 1];
    const int64_t r0 = (int64_t)blockIdx.x * kEllRows;
    const int t = threadIdx.x;
    if (t <= kEllRows) sb[t] = rp[r0 + t < m ? r0 + t : m];
    __syncthreads();
    constexpr int kGroups = kBlock / kEllWindow, kPer = kEllRows / kGroups;
    const int l = t % kEllWindow, g = t / kEllWindow;
    for (int k0 = 0; k0 < K; k0 += kEllWindow) {
        int32_t c[kPer];
        U v[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int r = g + q * kGroups;
            const int64_t e = (int64_t)sb[r] + k0 + l;
            const bool on = e < sb[r + 1];
            c[q] = on ? col[e] : -1;
            v[q] = on ? val[e] : U(0);
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            sc[g + q * kGroups][l] = c[q];
            sv[g + q * kGroups][l] = v[q];
        }
        __syncthreads();
        const int r = t % kEllRows;
#pragma unroll
        for (int k = t / kEllRows; k < kEllWindow; k += kBlock / kEllRows) {
            if (k0 + k < K) {
                const int64_t s = (int64_t)(k0 + k) * m_pad + r0 + r;
                ecol[s] = sc[r][k];
                eval[s] = sv[r][k];
            }
        }
        __syncthreads();
    }
}

// A wave takes 64 consecutive rows, a lane a row, and walks the diagonals in
// ascending order beside each row's ascending columns: every slot is written
// once, zeros included, 64 rows a store, and the presence bits of 64 rows are
// the wave's ballot.  Entry-parallel scatter with an atomic OR per entry into
// a zero-filled copy took 149 us for 500k rows of 9 float64 diagonals (and 13 to
// fill), so 31; 4.3 -> 0.76 ms for the 7-point 256^3 matrix.
template <typename U>
__global__ __launch_bounds__(kBlock) void k_csr_to_dia(int64_t m, int64_t m_pad, int D,
                                                       const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col,
                                                       const U *__restrict__ val,
                                                       const int32_t *__restrict__ offs,
                                                       U *__restrict__ data,
                                                       uint32_t *__restrict__ present) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (row - lane >= m_pad) return;   // whole waves
    int32_t q = row < m ? rp[row] : 0;
    const int32_t e = row < m ? rp[row + 1] : 0;
    int32_t c = q < e ? col[q] : INT32_MAX;   // INT32_MAX is no column: n < 2^31
    U v = q < e ? val[q] : U(0);
    for (int d = 0; d < D; ++d) {
        const bool hit = (int64_t)c == row + offs[d] && q < e;
        const unsigned long long bits = __ballot(hit);
        const int64_t s = (int64_t)d * m_pad + row;
        data[s] = hit ? v : U(0);
        if (lane == 0) {
            present[s >> 5] = (uint32_t)bits;
            present[(s >> 5) + 1] = (uint32_t)(bits >> 32);
        }
        if (hit) {
            ++q;
            c = q < e ? col[q] : INT32_MAX;
            v = q < e ? val[q] : U(0);
        }
    }
}

__global__ void k_coo_to_csr(int64_t m, int64_t nnz, const int32_t *__restrict__ row_idx,
                             int32_t *__restrict__ rp) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i > m) return;
    int64_t a = 0, b = nnz;  // first entry with row_idx >= i
    while (a < b) {
        int64_t mid = (a + b) >> 1;
        if (row_idx[mid] < i)
            a = mid + 1;
        else
            b = mid;
    }
    rp[i] = (int32_t)a;
}

__global__ void k_ell_count(int64_t m, int64_t m_pad, int K, const int32_t *__restrict__ ecol,
                            int32_t *__restrict__ counts) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= m) return;
    int c = 0;
    for (int k = 0; k < K; ++k) c += ecol[(int64_t)k * m_pad + i] >= 0;
    counts[i] = c;
}

template <typename U>
__global__ void k_ell_gather(int64_t m, int64_t m_pad, int K, const int32_t *__restrict__ ecol,
                             const U *__restrict__ eval, const int32_t *__restrict__ rp,
                             int32_t *__restrict__ col, U *__restrict__ val) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= m) return;
    int64_t o = rp[i];
    for (int k = 0; k < K; ++k) {
        int64_t s = (int64_t)k * m_pad + i;
        int32_t c = ecol[s];
        if (c >= 0) {
            col[o] = c;
            val[o] = eval[s];
            ++o;
        }
    }
}

__device__ __forceinline__ bool bit_at(const uint32_t *__restrict__ w, int64_t s) {
    return (w[s >> 5] >> (s & 31)) & 1u;
}

__global__ void k_dia_count(int64_t m, int64_t m_pad, int D, const uint32_t *__restrict__ present,
                            int32_t *__restrict__ counts) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= m) return;
    int c = 0;
    for (int d = 0; d < D; ++d) c += bit_at(present, (int64_t)d * m_pad + i);
    counts[i] = c;
}

template <typename U>
__global__ void k_dia_gather(int64_t m, int64_t m_pad, int D, const int32_t *__restrict__ offs,
                             const U *__restrict__ data, const uint32_t *__restrict__ present,
                             const int32_t *__restrict__ rp, int32_t *__restrict__ col,
                             U *__restrict__ val) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= m) return;
    int64_t o = rp[i];
    for (int d = 0; d < D; ++d) {
        int64_t s = (int64_t)d * m_pad + i;
        if (bit_at(present, s)) {
            col[o] = (int32_t)(i + offs[d]);
            val[o] = data[s];
            ++o;
        }
    }
}

// ---- column panels (cache blocking of x)
// first index in [b, e) whose column is >= v (columns sorted within a row)
__device__ __forceinline__ int32_t col_lower_bound(const int32_t *__restrict__ col, int32_t b,
                                                   int32_t e, int64_t v) {
    while (b < e) {
        int32_t mid = b + ((e - b) >> 1);
        if ((int64_t)col[mid] < v)
            b = mid + 1;
        else
            e = mid;
    }
    return b;
}

__global__ void k_inverse_perm(int64_t m, const int32_t *__restrict__ rows,
                               int32_t *__restrict__ inv) {
    int64_t pos = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (pos < m) inv[rows[pos]] = (int32_t)pos;
}

// cnt[p*(m+1) + pos] = entries of row rows[pos] in panel p; position m is a
// zero pad so one exclusive scan over the whole array yields every panel's
// segment starts and, at position m, the panel's end.
__global__ void k_panel_count(int64_t m, const int32_t *__restrict__ rp,
                              const int32_t *__restrict__ col, const int32_t *__restrict__ rows,
                              int P, int64_t w, int32_t *__restrict__ cnt) {
    int64_t pos = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (pos > m) return;
    if (pos == m) {
        for (int p = 0; p < P; ++p) cnt[(int64_t)p * (m + 1) + m] = 0;
        return;
    }
    int64_t row = rows[pos];
    int32_t b = rp[row], e = rp[row + 1];
    int32_t prev = b;
    for (int p = 0; p < P; ++p) {
        int32_t next = p == P - 1 ? e : col_lower_bound(col, prev, e, (int64_t)(p + 1) * w);
        cnt[(int64_t)p * (m + 1) + pos] = next - prev;
        prev = next;
    }
}

template <typename U>
__global__ void k_panel_scatter(int64_t m, int64_t nnz, const int32_t *__restrict__ rp,
                                const int32_t *__restrict__ col, const U *__restrict__ val,
                                const int32_t *__restrict__ inv, int64_t w,
                                const int32_t *__restrict__ prow, int32_t *__restrict__ pcol,
                                U *__restrict__ pval) {
    int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    int64_t p0 = t * kEntryRun;
    if (p0 >= nnz) return;
    int64_t p1 = p0 + kEntryRun < nnz ? p0 + kEntryRun : nnz;
    int64_t row = row_of_entry(rp, m, p0);
    int64_t rend = rp[row + 1];
    for (int64_t p = p0; p < p1; ++p) {
        while (p >= rend) rend = rp[++row + 1];
        int32_t c = col[p];
        int64_t panel = c / w;
        int32_t seg = col_lower_bound(col, rp[row], (int32_t)rend, panel * w);
        int64_t dst = prow[panel * (m + 1) + inv[row]] + (p - seg);
        pcol[dst] = c;
        pval[dst] = val[p];
    }
}

__global__ void k_panel_rowcount(int64_t m, const int32_t *__restrict__ rows, int P,
                                 const int32_t *__restrict__ prow, int32_t *__restrict__ counts) {
    int64_t pos = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (pos >= m) return;
    int32_t tot = 0;
    for (int p = 0; p < P; ++p) {
        const int32_t *pr = prow + (int64_t)p * (m + 1);
        tot += pr[pos + 1] - pr[pos];
    }
    counts[rows[pos]] = tot;
}

template <typename U>
__global__ void k_panel_gather(int64_t m, const int32_t *__restrict__ rows, int P,
                               const int32_t *__restrict__ prow, const int32_t *__restrict__ pcol,
                               const U *__restrict__ pval, const int32_t *__restrict__ rp,
                               int32_t *__restrict__ col, U *__restrict__ val) {
    int64_t pos = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (pos >= m) return;
    int64_t o = rp[rows[pos]];
    for (int p = 0; p < P; ++p) {
        const int32_t *pr = prow + (int64_t)p * (m + 1);
        for (int32_t j = pr[pos]; j < pr[pos + 1]; ++j) {
            col[o] = pcol[j];
            val[o] = pval[j];
            ++o;
        }
    }
}

// ---- row binning: bin b holds rows with upper[b-1] < len <= upper[b]
__device__ __forceinline__ int bin_of(int len, const BinSpec &spec) {
    int b = 0;
    while (b < kAdaptiveBins - 1 && len > spec.upper[b]) ++b;
    return b;
}

// A workgroup bins kBinThreads rows `steps` times (more for large matrices, so
// that the one-workgroup scan of the counts stays short).
constexpr int kBinThreads = 1024;

__global__ __launch_bounds__(kBinThreads) void k_bin_count(int64_t m, int steps,
                                                           const int32_t *__restrict__ rp,
                                                           BinSpec spec,
                                                           unsigned int *__restrict__ block_counts) {
    __shared__ unsigned int cnt[kAdaptiveBins];
    if (threadIdx.x < kAdaptiveBins) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * kBinThreads * steps + threadIdx.x;
    const int lane = threadIdx.x % kWave;
    for (int k = 0; k < steps; ++k) {
        const int64_t i = r0 + (int64_t)k * kBinThreads;
        const int b = i < m ? bin_of(rp[i + 1] - rp[i], spec) : -1;
        for (int q = 0; q < kAdaptiveBins; ++q) {
            const unsigned int c = __popcll(__ballot(b == q));
            if (lane == 0 && c) atomicAdd(&cnt[q], c);
        }
    }
    __syncthreads();
    // bin-major layout so each bin's blocks are contiguous for the scan
    if (threadIdx.x < kAdaptiveBins)
        block_counts[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = cnt[threadIdx.x];
}

// Exclusive scan over the bin-major block counts, one workgroup of 1024
// threads with 8 counts each at a time; also the per-bin start offsets
// (bin_offsets[b], b <= kAdaptiveBins).  (One count a thread, scanned through
// LDS with two barriers a step, a count per 256 rows: 540 us for 8M rows, now
// 6.)
__global__ __launch_bounds__(1024) void k_bin_scan(unsigned int *v, int64_t nblk,
                                                   unsigned int *bin_offsets) {
    constexpr int kPer = 8;
    __shared__ unsigned int wsum[1024 / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const int64_t count = nblk * kAdaptiveBins;
    unsigned int carry = 0;
    for (int64_t base = 0; base < count; base += 1024 * kPer) {
        const int64_t i0 = base + (int64_t)t * kPer;
        unsigned int x[kPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) x[k] = i0 + k < count ? v[i0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < kPer; ++k) sum += x[k];
        unsigned int incl = sum;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const unsigned int u = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += u;
        }
        if (lane == kWave - 1) wsum[w] = incl;
        __syncthreads();
        unsigned int before = carry, total = 0;
        for (int k = 0; k < 1024 / kWave; ++k) {
            before += k < w ? wsum[k] : 0u;
            total += wsum[k];
        }
        unsigned int run = before + incl - sum;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (i0 + k < count) v[i0 + k] = run;
            run += x[k];
        }
        carry += total;
        __syncthreads();
    }
    if (t < kAdaptiveBins) bin_offsets[t] = v[(int64_t)t * nblk];
    if (t == 0) bin_offsets[kAdaptiveBins] = carry;
}

// Stable scatter: rows keep ascending order inside each bin.
__global__ __launch_bounds__(kBinThreads) void k_bin_scatter(
    int64_t m, int steps, const int32_t *__restrict__ rp, BinSpec spec,
    const unsigned int *__restrict__ block_base, int32_t *__restrict__ rows_out) {
    constexpr int kWaves = kBinThreads / kWave;
    __shared__ unsigned int wave_cnt[kWaves][kAdaptiveBins];
    __shared__ unsigned int base[kAdaptiveBins];
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const unsigned long long below = lane ? (~0ull >> (kWave - lane)) : 0ull;
    if (threadIdx.x < kAdaptiveBins)
        base[threadIdx.x] = block_base[(int64_t)threadIdx.x * gridDim.x + blockIdx.x];
    const int64_t r0 = (int64_t)blockIdx.x * kBinThreads * steps + threadIdx.x;
    for (int k = 0; k < steps; ++k) {
        const int64_t i = r0 + (int64_t)k * kBinThreads;
        const int b = i < m ? bin_of(rp[i + 1] - rp[i], spec) : -1;
        unsigned int rank = 0;
        for (int q = 0; q < kAdaptiveBins; ++q) {
            const unsigned long long mask = __ballot(b == q);
            if (b == q) rank = __popcll(mask & below);
            if (lane == 0) wave_cnt[w][q] = __popcll(mask);
        }
        __syncthreads();
        if (b >= 0) {
            unsigned int pos = base[b] + rank;
            for (int w2 = 0; w2 < w; ++w2) pos += wave_cnt[w2][b];
            rows_out[pos] = (int32_t)i;
        }
        __syncthreads();
        if (threadIdx.x < kAdaptiveBins) {
            unsigned int c = 0;
            for (int w2 = 0; w2 < kWaves; ++w2) c += wave_cnt[w2][threadIdx.x];
            base[threadIdx.x] += c;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- BCSR 4x4
// Four lanes per block row R, lane k walking row 4R + k: the distinct column
// blocks col >> 2 of those rows, ascending, by a 4-way merge.  A lane keeps its
// row's next four columns (all that a block can take) and writes its quarter of
// the block, zeros included, in one store.  One thread merging four rows,
// entry by entry, into zero-filled blocks took 65 + 201 us for 25k block rows
// of 16 float32 blocks (counts + blocks), so 19 + 66.
//
// Values are moved as bit patterns (U = uint32 / uint64).  pres holds 16
// presence bits per block.
template <typename U, bool FILL>
__device__ __forceinline__ int bcsr_walk(int64_t R, int k, int64_t m,
                                         const int32_t *__restrict__ rp,
                                         const int32_t *__restrict__ col,
                                         const U *__restrict__ val, int64_t kb,
                                         int32_t *__restrict__ bcol, U *__restrict__ bval,
                                         uint16_t *__restrict__ pres) {
    typedef U vec4 __attribute__((ext_vector_type(4)));
    const int64_t r = 4 * R + k;
    int32_t p = r < m ? rp[r] : 0;
    const int32_t e = r < m ? rp[r + 1] : 0;
    int n = 0;
    for (;;) {
        int32_t c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) c[j] = p + j < e ? col[p + j] : INT32_MAX;
        int32_t blk = c[0] == INT32_MAX ? INT32_MAX : c[0] >> 2;   // no column is INT32_MAX
        blk = min(blk, __shfl_xor(blk, 1));
        blk = min(blk, __shfl_xor(blk, 2));
        if (blk == INT32_MAX) break;
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) cnt += c[j] != INT32_MAX && (c[j] >> 2) == blk;
        if constexpr (FILL) {
            vec4 v = {0, 0, 0, 0};
            unsigned bits = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j < cnt) {
                    const U x = val[p + j];
                    const int q = c[j] & 3;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = q == i ? x : v[i];
                    bits |= 1u << (k * 4 + q);
                }
            }
            bits |= __shfl_xor(bits, 1);
            bits |= __shfl_xor(bits, 2);
            *reinterpret_cast<vec4 *>(bval + (kb + n) * 16 + k * 4) = v;
            if (k == 0) {
                bcol[kb + n] = blk;
                pres[kb + n] = (uint16_t)bits;
            }
        }
        ++n;
        p += cnt;
    }
    return n;
}

__global__ __launch_bounds__(kBlock) void k_bcsr_count(int64_t mb, int64_t m,
                                                       const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col,
                                                       int32_t *__restrict__ counts) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, R = t >> 2;
    if (R >= mb) return;   // whole groups of four
    const int n = bcsr_walk<uint32_t, false>(R, (int)(t & 3), m, rp, col, nullptr, 0, nullptr,
                                             nullptr, nullptr);
    if ((t & 3) == 0) counts[R] = n;
}

template <typename U>
__global__ __launch_bounds__(kBlock) void k_bcsr_fill(
    int64_t mb, int64_t m, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const U *__restrict__ val, const int32_t *__restrict__ brp, int32_t *__restrict__ bcol,
    U *__restrict__ bval, uint16_t *__restrict__ pres) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, R = t >> 2;
    if (R >= mb) return;
    bcsr_walk<U, true>(R, (int)(t & 3), m, rp, col, val, brp[R], bcol, bval, pres);
}

// Inverse: per row, the count of stored entries, then the entries in block
// order (ascending columns).
__global__ void k_bcsr_rowcount(int64_t mb, int64_t m, const int32_t *__restrict__ brp,
                                const uint16_t *__restrict__ pres, int32_t *__restrict__ counts) {
    int64_t R = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (R >= mb) return;
    int32_t c[4] = {0, 0, 0, 0};
    for (int64_t kb = brp[R]; kb < brp[R + 1]; ++kb) {
        const unsigned bits = pres[kb];
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] += __popc((bits >> (4 * k)) & 15u);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (4 * R + k < m) counts[4 * R + k] = c[k];
}

template <typename U>
__global__ void k_bcsr_gather(int64_t mb, int64_t m, const int32_t *__restrict__ brp,
                              const int32_t *__restrict__ bcol, const U *__restrict__ bval,
                              const uint16_t *__restrict__ pres, const int32_t *__restrict__ rp,
                              int32_t *__restrict__ col, U *__restrict__ val) {
    int64_t R = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (R >= mb) return;
    for (int k = 0; k < 4; ++k) {
        const int64_t r = 4 * R + k;
        if (r >= m) break;
        int64_t q = rp[r];
        for (int64_t kb = brp[R]; kb < brp[R + 1]; ++kb) {
            const unsigned bits = pres[kb];
            for (int cc = 0; cc < 4; ++cc)
                if ((bits >> (4 * k + cc)) & 1u) {
                    col[q] = bcol[kb] * 4 + cc;
                    val[q] = bval[kb * 16 + k * 4 + cc];
                    ++q;
                }
        }
    }
}

}  // namespace


spmv_status launch_csr_to_coo(int64_t m, int64_t nnz, const int32_t *rp, int32_t *row_idx,
                              hipStream_t s) {
    if (nnz == 0) return SPMV_OK;
    k_csr_to_coo<<<grid_for((nnz + kEntryRun - 1) / kEntryRun, kBlock), kBlock, 0, s>>>(
        m, nnz, rp, row_idx);
    SMAT_LAUNCHED("csr_to_coo");
    return SPMV_OK;
}

spmv_status launch_csr_to_ell(int64_t m, int64_t m_pad, int K, const int32_t *rp,
                              const int32_t *col, const void *val, int elt, int32_t *ecol,
                              void *eval, hipStream_t s) {
    if (K == 0 || m_pad == 0) return SPMV_OK;
    const unsigned g = grid_for(m_pad, kEllRows);
    if (elt == 8)
        k_csr_to_ell<uint64_t><<<g, kBlock, 0, s>>>(m, m_pad, K, rp, col, (const uint64_t *)val,
                                                    ecol, (uint64_t *)eval);
    else
        k_csr_to_ell<uint32_t><<<g, kBlock, 0, s>>>(m, m_pad, K, rp, col, (const uint32_t *)val,
                                                    ecol, (uint32_t *)eval);
    SMAT_LAUNCHED("csr_to_ell");
    return SPMV_OK;
}

spmv_status launch_csr_to_dia(int64_t m, int64_t m_pad, int D, const int32_t *rp,
                              const int32_t *col, const void *val, int elt, const int32_t *offs,
                              void *data, uint32_t *present, hipStream_t s) {
    if (D == 0 || m_pad == 0) return SPMV_OK;
    const unsigned g = grid_for(m_pad, kBlock);
    if (elt == 8)
        k_csr_to_dia<uint64_t><<<g, kBlock, 0, s>>>(m, m_pad, D, rp, col, (const uint64_t *)val,
                                                    offs, (uint64_t *)data, present);
    else
        k_csr_to_dia<uint32_t><<<g, kBlock, 0, s>>>(m, m_pad, D, rp, col, (const uint32_t *)val,
                                                    offs, (uint32_t *)data, present);
    SMAT_LAUNCHED("csr_to_dia");
    return SPMV_OK;
}

spmv_status launch_coo_to_csr(int64_t m, int64_t nnz, const int32_t *row_idx, int32_t *rp,
                              hipStream_t s) {
    k_coo_to_csr<<<grid_for(m + 1, kBlock), kBlock, 0, s>>>(m, nnz, row_idx, rp);
    SMAT_LAUNCHED("coo_to_csr");
    return SPMV_OK;
}

spmv_status launch_ell_to_csr(int64_t m, int64_t m_pad, int K, const int32_t *ecol,
                              const void *eval, int elt, int32_t *rp, int32_t *col, void *val,
                              int32_t *counts, unsigned int *scratch, hipStream_t s) {
    if (m > 0) {
        k_ell_count<<<grid_for(m, kBlock), kBlock, 0, s>>>(m, m_pad, K, ecol, counts);
        SMAT_LAUNCHED("ell_count");
    }
    spmv_status st = launch_exclusive_scan_rows(m, counts, rp, scratch, s);
    if (st != SPMV_OK) return st;
    if (m == 0) return SPMV_OK;
    if (elt == 8)
        k_ell_gather<uint64_t><<<grid_for(m, kBlock), kBlock, 0, s>>>(
            m, m_pad, K, ecol, (const uint64_t *)eval, rp, col, (uint64_t *)val);
    else
        k_ell_gather<uint32_t><<<grid_for(m, kBlock), kBlock, 0, s>>>(
            m, m_pad, K, ecol, (const uint32_t *)eval, rp, col, (uint32_t *)val);
    SMAT_LAUNCHED("ell_gather");
    return SPMV_OK;
}

spmv_status launch_dia_to_csr(int64_t m, int64_t n, int64_t m_pad, int D, const int32_t *offs,
                              const void *data, const uint32_t *present, int elt, int32_t *rp,
                              int32_t *col, void *val, int32_t *counts, unsigned int *scratch,
                              hipStream_t s) {
    (void)n;
    if (m > 0) {
        k_dia_count<<<grid_for(m, kBlock), kBlock, 0, s>>>(m, m_pad, D, present, counts);
        SMAT_LAUNCHED("dia_count");
    }
    spmv_status st = launch_exclusive_scan_rows(m, counts, rp, scratch, s);
    if (st != SPMV_OK) return st;
    if (m == 0) return SPMV_OK;
    if (elt == 8)
        k_dia_gather<uint64_t><<<grid_for(m, kBlock), kBlock, 0, s>>>(
            m, m_pad, D, offs, (const uint64_t *)data, present, rp, col, (uint64_t *)val);
    else
        k_dia_gather<uint32_t><<<grid_for(m, kBlock), kBlock, 0, s>>>(
            m, m_pad, D, offs, (const uint32_t *)data, present, rp, col, (uint32_t *)val);
    SMAT_LAUNCHED("dia_gather");
    return SPMV_OK;
}

spmv_status launch_csr_to_panels(int64_t m, int64_t nnz, const int32_t *rp, const int32_t *col,
                                 const void *val, int elt, const int32_t *rows, int P, int64_t w,
                                 int32_t *inv, int32_t *cnt, int32_t *prow, unsigned *scan,
                                 int32_t *pcol, void *pval, hipStream_t s) {
    if (m == 0) return SPMV_OK;
    k_inverse_perm<<<grid_for(m, kBlock), kBlock, 0, s>>>(m, rows, inv);
    SMAT_LAUNCHED("inverse_perm");
    k_panel_count<<<grid_for(m + 1, kBlock), kBlock, 0, s>>>(m, rp, col, rows, P, w, cnt);
    SMAT_LAUNCHED("panel_count");
    spmv_status st = launch_exclusive_scan_rows((int64_t)P * (m + 1), cnt, prow, scan, s);
    if (st != SPMV_OK) return st;
    if (nnz == 0) return SPMV_OK;
    unsigned g = grid_for((nnz + kEntryRun - 1) / kEntryRun, kBlock);
    if (elt == 8)
        k_panel_scatter<uint64_t><<<g, kBlock, 0, s>>>(m, nnz, rp, col, (const uint64_t *)val, inv,
                                                       w, prow, pcol, (uint64_t *)pval);
    else
        k_panel_scatter<uint32_t><<<g, kBlock, 0, s>>>(m, nnz, rp, col, (const uint32_t *)val, inv,
                                                       w, prow, pcol, (uint32_t *)pval);
    SMAT_LAUNCHED("panel_scatter");
    return SPMV_OK;
}

spmv_status launch_panels_to_csr(int64_t m, const int32_t *rows, int P, const int32_t *prow,
                                 const int32_t *pcol, const void *pval, int elt, int32_t *rp,
                                 int32_t *col, void *val, int32_t *counts, unsigned *scan,
                                 hipStream_t s) {
    if (m > 0) {
        k_panel_rowcount<<<grid_for(m, kBlock), kBlock, 0, s>>>(m, rows, P, prow, counts);
        SMAT_LAUNCHED("panel_rowcount");
    }
    spmv_status st = launch_exclusive_scan_rows(m, counts, rp, scan, s);
    if (st != SPMV_OK || m == 0) return st;
    if (elt == 8)
        k_panel_gather<uint64_t><<<grid_for(m, kBlock), kBlock, 0, s>>>(
            m, rows, P, prow, pcol, (const uint64_t *)pval, rp, col, (uint64_t *)val);
    else
        k_panel_gather<uint32_t><<<grid_for(m, kBlock), kBlock, 0, s>>>(
            m, rows, P, prow, pcol, (const uint32_t *)pval, rp, col, (uint32_t *)val);
    SMAT_LAUNCHED("panel_gather");
    return SPMV_OK;
}

spmv_status launch_bin_rows(int64_t m, const int32_t *rp, const BinSpec &spec,
                            unsigned int *block_counts, int32_t *rows_out,
                            unsigned int *bin_offsets_dev, hipStream_t s) {
    if (m == 0) {
        SMAT_HIP(hipMemsetAsync(bin_offsets_dev, 0, sizeof(unsigned) * (kAdaptiveBins + 1), s));
        return SPMV_OK;
    }
    const int steps = (int)std::min<int64_t>(16, 1 + m / (512 * kBinThreads));
    const unsigned nblk = grid_for(m, kBinThreads * steps);
    k_bin_count<<<nblk, kBinThreads, 0, s>>>(m, steps, rp, spec, block_counts);
    SMAT_LAUNCHED("bin_count");
    k_bin_scan<<<1, 1024, 0, s>>>(block_counts, nblk, bin_offsets_dev);
    SMAT_LAUNCHED("bin_scan");
    k_bin_scatter<<<nblk, kBinThreads, 0, s>>>(m, steps, rp, spec, block_counts, rows_out);
    SMAT_LAUNCHED("bin_scatter");
    return SPMV_OK;
}

spmv_status launch_bcsr_count(int64_t m, const int32_t *rp, const int32_t *col, int32_t *counts,
                              int32_t *brp, unsigned int *scratch, hipStream_t s) {
    const int64_t mb = (m + 3) / 4;
    if (mb > 0) {
        k_bcsr_count<<<grid_for(4 * mb, kBlock), kBlock, 0, s>>>(mb, m, rp, col, counts);
        SMAT_LAUNCHED("bcsr_count");
    }
    return launch_exclusive_scan_rows(mb, counts, brp, scratch, s);
}

spmv_status launch_csr_to_bcsr(int64_t m, const int32_t *rp, const int32_t *col, const void *val,
                               int elt, const int32_t *brp, int32_t *bcol, void *bval,
                               uint16_t *pres, hipStream_t s) {
    const int64_t mb = (m + 3) / 4;
    if (mb == 0) return SPMV_OK;
    if (elt == 8)
        k_bcsr_fill<uint64_t><<<grid_for(4 * mb, kBlock), kBlock, 0, s>>>(
            mb, m, rp, col, (const uint64_t *)val, brp, bcol, (uint64_t *)bval, pres);
    else
        k_bcsr_fill<uint32_t><<<grid_for(4 * mb, kBlock), kBlock, 0, s>>>(
            mb, m, rp, col, (const uint32_t *)val, brp, bcol, (uint32_t *)bval, pres);
    SMAT_LAUNCHED("bcsr_fill");
    return SPMV_OK;
}

spmv_status launch_bcsr_to_csr(int64_t m, const int32_t *brp, const int32_t *bcol,
                               const void *bval, const uint16_t *pres, int elt, int32_t *rp,
                               int32_t *col, void *val, int32_t *counts, unsigned int *scratch,
                               hipStream_t s) {
    const int64_t mb = (m + 3) / 4;
    if (mb > 0) {
        k_bcsr_rowcount<<<grid_for(mb, kBlock), kBlock, 0, s>>>(mb, m, brp, pres, counts);
        SMAT_LAUNCHED("bcsr_rowcount");
    }
    spmv_status st = launch_exclusive_scan_rows(m, counts, rp, scratch, s);
    if (st != SPMV_OK || mb == 0) return st;
    if (elt == 8)
        k_bcsr_gather<uint64_t><<<grid_for(mb, kBlock), kBlock, 0, s>>>(
            mb, m, brp, bcol, (const uint64_t *)bval, pres, rp, col, (uint64_t *)val);
    else
        k_bcsr_gather<uint32_t><<<grid_for(mb, kBlock), kBlock, 0, s>>>(
            mb, m, brp, bcol, (const uint32_t *)bval, pres, rp, col, (uint32_t *)val);
    SMAT_LAUNCHED("bcsr_gather");
    return SPMV_OK;
}

}  // namespace smat
