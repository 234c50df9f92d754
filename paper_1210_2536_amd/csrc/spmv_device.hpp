// Per-row / per-tile SpMV device functions shared by the stand-alone kernels
// and the persistent multilevel kernel, so both compute every output with the
// same operations in the same order (bitwise-identical results).
//
// NT selects the cache policy of the matrix streams (values, column indices,
// diagonals): non-temporal loads keep them from displacing the reused x
// vector in L2, which helps banded matrices and can hurt gathers from
// large, randomly indexed x.  It is a tuning parameter (spmv_params
// stream_nt); the arithmetic is identical either way.
#pragma once

#include "internal.hpp"

namespace smat {

template <bool NT, typename T>
__device__ __forceinline__ T ld(const T *p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

// Plain CSR row: one thread, storage order.
template <typename T>
__device__ __forceinline__ double csr_row_seq(int64_t i, const int32_t *__restrict__ rp,
                                              const int32_t *__restrict__ col,
                                              const T *__restrict__ val,
                                              const T *__restrict__ x) {
    double acc = 0.0;
    int32_t b = rp[i], e = rp[i + 1];
    for (int32_t p = b; p < e; ++p) acc = fma((double)val[p], (double)x[col[p]], acc);
    return acc;
}

// CSR row by a group of L lanes (lane = 0..L-1); lanes stride the row and
// reduce by xor shuffles.  Every lane of the group returns the row sum.
template <typename T, int L, bool NT>
__device__ __forceinline__ double lanes_sum(int32_t b, int32_t e, int lane,
                                            const int32_t *__restrict__ col,
                                            const T *__restrict__ val,
                                            const T *__restrict__ x) {
    double acc = 0.0;
#pragma unroll 4
    for (int32_t p = b + lane; p < e; p += L)
        acc = fma((double)ld<NT>(val + p), (double)x[ld<NT>(col + p)], acc);
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, L);
    return acc;
}

template <typename T, int L, bool NT>
__device__ __forceinline__ double csr_row_lanes(int64_t row, int lane,
                                                const int32_t *__restrict__ rp,
                                                const int32_t *__restrict__ col,
                                                const T *__restrict__ val,
                                                const T *__restrict__ x) {
    return lanes_sum<T, L, NT>(rp[row], rp[row + 1], lane, col, val, x);
}

// Entries [b, e) summed by a whole workgroup of B threads (B a multiple of
// 64); thread 0 returns the sum.  `part` is LDS scratch of B / 64 doubles.
template <typename T, int B, bool NT>
__device__ __forceinline__ double block_sum(int32_t b, int32_t e, const int32_t *__restrict__ col,
                                            const T *__restrict__ val, const T *__restrict__ x,
                                            double *part) {
    double acc = 0.0;
#pragma unroll 4
    for (int32_t p = b + threadIdx.x; p < e; p += B)
        acc = fma((double)ld<NT>(val + p), (double)x[ld<NT>(col + p)], acc);
    for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = acc;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < B / kWave; ++w) s += part[w];
    __syncthreads();
    return s;
}

template <typename T, int B, bool NT>
__device__ __forceinline__ double csr_row_block(int64_t row, const int32_t *__restrict__ rp,
                                                const int32_t *__restrict__ col,
                                                const T *__restrict__ val,
                                                const T *__restrict__ x, double *part) {
    return block_sum<T, B, NT>(rp[row], rp[row + 1], col, val, x, part);
}

// Length-binned CSR (one launch serves every bin, longest first).  Workgroup
// `bid` of the launch geometry `a` finds its bin b (7: a whole workgroup per
// row; 6..0: 64..1 lanes per row) and its rows in the binned order `rows`.
constexpr int kAdaptBlock = 256;

template <typename T, int L, bool NT, bool PK = false>
__device__ __forceinline__ void adaptive_lanes(unsigned local, unsigned rbeg, unsigned rend,
                                               const int32_t *__restrict__ rows,
                                               const int32_t *__restrict__ rp,
                                               const int32_t *__restrict__ col,
                                               const T *__restrict__ val, const T *__restrict__ x,
                                               T *__restrict__ y) {
    int64_t r = (int64_t)rbeg + (int64_t)local * (kAdaptBlock / L) + threadIdx.x / L;
    int lane = threadIdx.x & (L - 1);
    if (r < rend) {
        int64_t row = rows[r];
        double acc = csr_row_lanes<T, L, NT>(PK ? r : row, lane, rp, col, val, x);
        if (lane == 0) y[row] = (T)acc;
    }
}

// Every thread of the (kAdaptBlock-thread) workgroup must call it; `part` is
// LDS scratch of kAdaptBlock / 64 doubles.
template <typename T, bool NT, bool PK = false>
__device__ __forceinline__ void adaptive_block(const AdaptiveLaunch &a, unsigned bid,
                                               const int32_t *__restrict__ rows,
                                               const int32_t *__restrict__ rp,
                                               const int32_t *__restrict__ col,
                                               const T *__restrict__ val, const T *__restrict__ x,
                                               T *__restrict__ y, double *part) {
    int q = 0;
    while (q < 7 && bid >= a.first[q + 1]) ++q;
    const int b = 7 - q;
    const unsigned local = bid - a.first[q];
    const unsigned rb = a.row_begin[b], re = a.row_begin[b + 1];
    switch (b) {
    case 7: {
        int64_t row = rows[rb + local];
        double s = csr_row_block<T, kAdaptBlock, NT>(PK ? (int64_t)(rb + local) : row, rp, col,
                                                     val, x, part);
        if (threadIdx.x == 0) y[row] = (T)s;
        break;
    }
    case 6: adaptive_lanes<T, 64, NT, PK>(local, rb, re, rows, rp, col, val, x, y); break;
    case 5: adaptive_lanes<T, 32, NT, PK>(local, rb, re, rows, rp, col, val, x, y); break;
    case 4: adaptive_lanes<T, 16, NT, PK>(local, rb, re, rows, rp, col, val, x, y); break;
    case 3: adaptive_lanes<T, 8, NT, PK>(local, rb, re, rows, rp, col, val, x, y); break;
    case 2: adaptive_lanes<T, 4, NT, PK>(local, rb, re, rows, rp, col, val, x, y); break;
    case 1: adaptive_lanes<T, 2, NT, PK>(local, rb, re, rows, rp, col, val, x, y); break;
    default: adaptive_lanes<T, 1, NT, PK>(local, rb, re, rows, rp, col, val, x, y); break;
    }
}

// ELL row: slots in order, U slots loaded ahead of use.
template <typename T, int U, bool NT>
__device__ __forceinline__ double ell_row(int64_t i, int64_t m_pad, int K,
                                          const int32_t *__restrict__ ecol,
                                          const T *__restrict__ eval, const T *__restrict__ x) {
    double acc = 0.0;
    int k = 0;
    for (; k + U <= K; k += U) {
        int32_t c[U];
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int64_t s = (int64_t)(k + u) * m_pad + i;
            c[u] = ld<NT>(ecol + s);
            v[u] = ld<NT>(eval + s);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c[u] >= 0) acc = fma((double)v[u], (double)x[c[u]], acc);
    }
    for (; k < K; ++k) {
        int64_t s = (int64_t)k * m_pad + i;
        int32_t c = ld<NT>(ecol + s);
        if (c >= 0) acc = fma((double)ld<NT>(eval + s), (double)x[c], acc);
    }
    return acc;
}

// V consecutive elements of a matrix stream as one load (V * sizeof(T) bytes;
// the address is a multiple of that size).
template <typename T, int V, bool NT>
__device__ __forceinline__ void ld_rows(const T *p, T (&v)[V]) {
    if constexpr (V == 1) {
        v[0] = ld<NT>(p);
    } else {
        typedef T vec __attribute__((ext_vector_type(V)));
        vec w = ld<NT>(reinterpret_cast<const vec *>(p));
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = w[e];
    }
}

// Rows i0 .. i0+V-1 of y as one store away from the end; y is only
// element-aligned.  past: around the caches (kHbmBytes).
template <typename T, int V>
__device__ __forceinline__ void st_rows(T *y, int64_t i0, int64_t m, const double (&acc)[V],
                                        bool past) {
    if (V > 1 && i0 + V <= m) {
        typedef T vec __attribute__((ext_vector_type(V), aligned(sizeof(T))));
        vec w;
#pragma unroll
        for (int e = 0; e < V; ++e) w[e] = (T)acc[e];
        if (past) {
            asm volatile("");   // on both sides: the compiler would merge the two
            __builtin_nontemporal_store(w, reinterpret_cast<vec *>(y + i0));
            asm volatile("");   // stores into a plain one
        } else {
            *reinterpret_cast<vec *>(y + i0) = w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (i0 + e < m) y[i0 + e] = (T)acc[e];
    }
}

// ELL rows i0 .. i0+V-1 of one lane (i0 a multiple of V, i0 < m): the slot
// columns and values of the V rows come in one load each.  Each row's sum
// runs over its slots in order, exactly as ell_row.
template <typename T, int U, int V, bool NT>
__device__ __forceinline__ void ell_rows_wide(int64_t i0, int64_t m, int64_t m_pad, int K,
                                              const int32_t *__restrict__ ecol,
                                              const T *__restrict__ eval,
                                              const T *__restrict__ x, double (&acc)[V]) {
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.0;
    int k = 0;
    for (; k + U <= K; k += U) {
        int32_t c[U][V];
        T v[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int64_t s = (int64_t)(k + u) * m_pad + i0;
            ld_rows<int32_t, V, NT>(ecol + s, c[u]);
            ld_rows<T, V, NT>(eval + s, v[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (i0 + e < m && c[u][e] >= 0)
                    acc[e] = fma((double)v[u][e], (double)x[c[u][e]], acc[e]);
    }
    for (; k < K; ++k) {
        int64_t s = (int64_t)k * m_pad + i0;
        int32_t c[V];
        T v[V];
        ld_rows<int32_t, V, NT>(ecol + s, c);
        ld_rows<T, V, NT>(eval + s, v);
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (i0 + e < m && c[e] >= 0) acc[e] = fma((double)v[e], (double)x[c[e]], acc[e]);
    }
}

// DIA tile with x windows staged in LDS; every thread of the workgroup must
// call it (it synchronises).  The tile holds R = blockDim * RPT * V rows; a
// lane takes V consecutive rows per step (one V-wide load of each diagonal),
// steps q = 0..RPT-1 being blockDim * V rows apart.  Each row sums its
// diagonals in ascending offset order whatever RPT and V.
template <typename T, int RPT, bool NT, int V = 1>
__device__ __forceinline__ void dia_tile_lds(int64_t r0, int64_t m, int64_t n, int64_t m_pad,
                                             const int32_t *__restrict__ offs, int nwin,
                                             const DiaWindow *__restrict__ win,
                                             const T *__restrict__ data,
                                             const T *__restrict__ x, T *__restrict__ y, T *xs,
                                             bool past = false) {
    const int R = blockDim.x * RPT * V;
    double acc[RPT][V];
#pragma unroll
    for (int q = 0; q < RPT; ++q)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[q][e] = 0.0;
    for (int w = 0; w < nwin; ++w) {
        const int d0 = win[w].d0, d1 = win[w].d1;
        const int lo = offs[d0], hi = offs[d1];
        const int len = R + (hi - lo);
        __syncthreads();  // previous window fully consumed
        for (int t = threadIdx.x; t < len; t += blockDim.x) {
            int64_t j = r0 + lo + t;
            xs[t] = (j >= 0 && j < n) ? x[j] : T(0);
        }
        __syncthreads();
        for (int d = d0; d <= d1; ++d) {
            const int sh = offs[d] - lo;
            const T *dd = data + (int64_t)d * m_pad + r0;
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const int il = (threadIdx.x + q * blockDim.x) * V;
                if (r0 + il < m) {
                    T v[V];
                    ld_rows<T, V, NT>(dd + il, v);
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        acc[q][e] = fma((double)v[e], (double)xs[il + e + sh], acc[q][e]);
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int64_t i0 = r0 + (int64_t)(threadIdx.x + q * blockDim.x) * V;
        st_rows<T, V>(y, i0, m, acc[q], past);
    }
}

// DIA tile reading x through the caches (same row layout as dia_tile_lds).
template <typename T, int RPT, bool NT, int V = 1>
__device__ __forceinline__ void dia_tile_direct(int64_t r0, int64_t m, int64_t n, int64_t m_pad,
                                                int D, const int32_t *__restrict__ offs,
                                                const T *__restrict__ data,
                                                const T *__restrict__ x, T *__restrict__ y,
                                                bool past = false) {
    double acc[RPT][V];
#pragma unroll
    for (int q = 0; q < RPT; ++q)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[q][e] = 0.0;
    for (int d = 0; d < D; ++d) {
        const int64_t off = offs[d];
        const T *dd = data + (int64_t)d * m_pad;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int64_t i0 = r0 + (int64_t)(threadIdx.x + q * blockDim.x) * V;
            if (i0 < m) {
                T v[V];
                ld_rows<T, V, NT>(dd + i0, v);
                const int64_t j0 = i0 + off;
                if (V > 1 && j0 >= 0 && j0 + V <= n) {
                    // x[j0 .. j0+V) in one load; j0 is only element-aligned
                    typedef T vec __attribute__((ext_vector_type(V)));
                    vec xv;
                    __builtin_memcpy(&xv, x + j0, sizeof(vec));
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        acc[q][e] = fma((double)v[e], (double)xv[e], acc[q][e]);
                } else {
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        const int64_t j = j0 + e;
                        if (j >= 0 && j < n)
                            acc[q][e] = fma((double)v[e], (double)x[j], acc[q][e]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int64_t i0 = r0 + (int64_t)(threadIdx.x + q * blockDim.x) * V;
        st_rows<T, V>(y, i0, m, acc[q], past);
    }
}

// dia_tile_groups: dia_tile_direct with the loads of 4 diagonals in flight, for
// streams from HBM.  Every x element and value of a group is requested before
// its first product (x first: its lines are shared by neighbouring diagonals,
// the values pass once).  EDGE: some rows or columns of the tile do
// not exist; addresses are clamped into the arrays and those products left
// out, so the tiles at the matrix's ends keep as many loads in flight as the
// others.
template <typename T, int U, int RPT, bool NT, int V, bool EDGE>
__device__ __forceinline__ void dia_group(int64_t r0, int64_t n, int64_t m_pad,
                                          const int32_t *__restrict__ offs,
                                          const T *__restrict__ dd, const T *__restrict__ x,
                                          double (&acc)[RPT][V]) {
    typedef T vec __attribute__((ext_vector_type(V)));
    T v[U][RPT][V];
    vec xv[U][RPT];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int64_t j0 = r0 + offs[u] + (int64_t)((threadIdx.x + q * blockDim.x) * V);
            if constexpr (EDGE) {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    xv[u][q][e] = x[min(max(j0 + e, (int64_t)0), n - 1)];
            } else {
                __builtin_memcpy(&xv[u][q], x + j0, sizeof(vec));   // only element-aligned
            }
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            int64_t i0 = r0 + (int64_t)((threadIdx.x + q * blockDim.x) * V);
            if constexpr (EDGE) i0 = min(i0, m_pad - V);
            ld_rows<T, V, NT>(dd + (int64_t)u * m_pad + i0, v[u][q]);
        }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int64_t j0 = r0 + offs[u] + (int64_t)((threadIdx.x + q * blockDim.x) * V);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const double t = fma((double)v[u][q][e], (double)xv[u][q][e], acc[q][e]);
                if (!EDGE || (j0 + e >= 0 && j0 + e < n)) acc[q][e] = t;
            }
        }
}

template <typename T, int RPT, bool NT, int V, bool EDGE>
__device__ __forceinline__ void dia_diagonals(int64_t r0, int64_t n, int64_t m_pad,
                                              int D, const int32_t *__restrict__ offs,
                                              const T *__restrict__ data,
                                              const T *__restrict__ x, double (&acc)[RPT][V]) {
    // at most 8 values and 8 x vectors of a lane in flight: more spill
    constexpr int U = EDGE ? 2 : 4;
    int d = 0;
    for (; d + U <= D; d += U)
        dia_group<T, U, RPT, NT, V, EDGE>(r0, n, m_pad, offs + d, data + (int64_t)d * m_pad, x,
                                          acc);
    if (U > 3 && d + 3 == D)
        dia_group<T, 3, RPT, NT, V, EDGE>(r0, n, m_pad, offs + d, data + (int64_t)d * m_pad, x,
                                          acc);
    else if (U > 2 && d + 2 == D)
        dia_group<T, 2, RPT, NT, V, EDGE>(r0, n, m_pad, offs + d, data + (int64_t)d * m_pad, x,
                                          acc);
    else if (U > 1 && d + 1 == D)
        dia_group<T, 1, RPT, NT, V, EDGE>(r0, n, m_pad, offs + d, data + (int64_t)d * m_pad, x,
                                          acc);
}

template <typename T, int RPT, bool NT, int V>
__device__ __forceinline__ void dia_tile_groups(int64_t r0, int64_t m, int64_t n, int64_t m_pad,
                                                int D, const int32_t *__restrict__ offs,
                                                const T *__restrict__ data,
                                                const T *__restrict__ x, T *__restrict__ y, bool past) {
    double acc[RPT][V];
#pragma unroll
    for (int q = 0; q < RPT; ++q)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[q][e] = 0.0;
    const int64_t R = (int64_t)blockDim.x * RPT * V;
    // offsets ascend, so the first and the last bound the tile's columns
    if (r0 + R <= m && r0 + offs[0] >= 0 && r0 + R + offs[D - 1] <= n)
        dia_diagonals<T, RPT, NT, V, false>(r0, n, m_pad, D, offs, data, x, acc);
    else
        dia_diagonals<T, RPT, NT, V, true>(r0, n, m_pad, D, offs, data, x, acc);
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int64_t i0 = r0 + (int64_t)(threadIdx.x + q * blockDim.x) * V;
        st_rows<T, V>(y, i0, m, acc[q], past);
    }
}

// Row sums over threads that take consecutive entries whatever their rows:
// `acc` is the thread's sum of the row still open at its end (of all its
// entries if no row starts in it), `bal` the ballot of the threads in which a
// row starts.  Returns what the wave's earlier threads carry into the row open
// at this thread's start; *tail (last lane) is the sum of the row open at the
// wave's end.
__device__ __forceinline__ double wave_carry(double acc, unsigned long long bal, int lane,
                                             double *tail) {
    const unsigned long long upto = bal & (~0ull >> (kWave - 1 - lane));
    const int start = upto ? 63 - __clzll(upto) : 0;
    double v = acc;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const double u = __shfl_up(v, off, kWave);
        if (lane - off >= start) v += u;
    }
    *tail = v;
    const double carry = __shfl_up(v, 1, kWave);
    return lane == 0 ? 0.0 : carry;
}

// ---------------------------------------------------------------- BCSR 4x4
// Block row R (rows 4R .. 4R+3) by L lanes; every lane of the wave must
// call (the lane sums are added by shuffles), R >= mb contributing nothing.
//
// BCSR block row by L lanes, 16 bytes of a block each (a row of the block in
// float32, half a row in float64), so a wave's loads are contiguous: S lanes
// hold a block, G = L / S groups take blocks g, g + G, ...  A lane reads the x
// values under its piece in one load and keeps one running sum for its row; the
// lanes of a row (the pair inside a float64 block, then the G groups) are added
// by xor shuffles in a fixed order.
__host__ __device__ constexpr int bcsr_block_lanes(int elt) { return elt; }   // 16 values

// Blocks k, k + G, ..., U of them: all columns and values are requested before
// the first x, all x before the first product.
template <typename T, int U, int G, bool NT>
__device__ __forceinline__ void bcsr_blocks(int32_t k, int j, int64_t n,
                                            const int32_t *__restrict__ bcol,
                                            const T *__restrict__ bval,
                                            const T *__restrict__ x, double &acc) {
    constexpr int W = 16 / (int)sizeof(T);   // values of a lane
    typedef T vec __attribute__((ext_vector_type(W)));
    vec w[U], xv[U];
    int64_t c0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        c0[u] = (int64_t)ld<NT>(bcol + k + u * G) * 4 + W * j % 4;
        w[u] = ld<NT>(reinterpret_cast<const vec *>(bval + (int64_t)(k + u * G) * 16) + j);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (c0[u] + W <= n) {
            __builtin_memcpy(&xv[u], x + c0[u], sizeof(vec));   // only element-aligned
        } else {
#pragma unroll
            for (int e = 0; e < W; ++e) xv[u][e] = c0[u] + e < n ? x[c0[u] + e] : T(0);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < W; ++e) acc = fma((double)w[u][e], (double)xv[u][e], acc);
}

// A: blocks a lane asks for together (4, or 1 where registers are short).
template <typename T, int L, bool NT, int A>
__device__ __forceinline__ void bcsr_row(int64_t R, int lane, int64_t mb, int64_t m, int64_t n,
                                         const int32_t *__restrict__ brp,
                                         const int32_t *__restrict__ bcol,
                                         const T *__restrict__ bval, const T *__restrict__ x,
                                         T *__restrict__ y) {
    constexpr int S = bcsr_block_lanes(sizeof(T));
    constexpr int G = L / S;                // blocks of a row side by side
    constexpr int Q = S / 4;                // lanes per row of a block
    static_assert(L >= S && L <= 64 && (L & (L - 1)) == 0, "lanes per block row");
    const int g = lane / S, j = lane % S;
    double acc = 0.0;
    if (R < mb) {
        const int32_t ke = brp[R + 1];
        int32_t k = brp[R] + g;
        for (; ke - k > (A - 1) * G; k += A * G)
            bcsr_blocks<T, A, G, NT>(k, j, n, bcol, bval, x, acc);
        if (A > 2 && ke - k > G) {
            bcsr_blocks<T, 2, G, NT>(k, j, n, bcol, bval, x, acc);
            k += 2 * G;
        }
        if (A > 1 && k < ke) bcsr_blocks<T, 1, G, NT>(k, j, n, bcol, bval, x, acc);
    }
    if (Q == 2) acc += __shfl_xor(acc, 1, L);   // the two halves of a block's row
#pragma unroll
    for (int off = S; off < L; off <<= 1) acc += __shfl_xor(acc, off, L);
    if (R < mb && g == 0 && j % Q == 0 && 4 * R + j / Q < m) y[4 * R + j / Q] = (T)acc;
}

}  // namespace smat
