// Kernel M: phase functions of the flattened two-dimensional tiles
// (MatrixArgs), in the manner of kernel_body.h.
#pragma once

#include "kernel_body.h"

namespace hptt {

// Tile of TC columns (contiguous in A) by TR rows (contiguous in B) for one
// workgroup of kBlock threads moving 16-byte vectors.  With shear, a column's
// B run starts on the LINE-byte boundary at or below the tile's first row,
// and S = LINE / elem - 1 rows before it are staged too (whole 128-byte lines:
// with 64-byte boundaries, which stage half as many rows more, MI355X ran 0
// to 7 % slower).
template <typename T, int TC_, int TR_, int LINE_>
struct MatrixShape {
    static constexpr int V = int(16 / sizeof(T));
    static constexpr int TC = TC_, TR = TR_, LINE = LINE_ / int(sizeof(T));
    static constexpr int S = LINE > 0 ? LINE - 1 : 0;
    static constexpr int laneC = TC / V;            // lanes that load one row
    static constexpr int rowStep = kBlock / laneC;  // rows the workgroup loads at once
    static constexpr int loads = (TR + S + rowStep - 1) / rowStep;
    static constexpr int rows = loads * rowStep;    // staged rows
    static constexpr int laneR = TR / V;            // lanes that store one column
    static constexpr int colStep = kBlock / laneR;
    static constexpr int stores = TC / colStep;
    static constexpr int pitch = TC + 1;
    static constexpr int tableBytes = (rows + 3 * TC) * 4;
    static constexpr int ldsBytes = (tableBytes + 15) / 16 * 16 + rows * pitch * int(sizeof(T));
    static_assert(TC % V == 0 && kBlock % laneC == 0 && kBlock % laneR == 0 && TC % colStep == 0,
                  "the workgroup covers whole rows and columns");
};

struct MatrixTile {
    int64_t a, b;   // byte offsets of the matrix (b: and of its row 0)
    int32_t col0;   // first column loaded
    int32_t qLo, qHi;  // columns of the tile that are stored: col0 + [qLo, qHi)
    int32_t row0;
};

template <class SH>
__host__ __device__ inline MatrixTile matrix_tile(const MatrixArgs& g, uint32_t t) {
    if (g.xcdGroupLog) t = xcd_group_map(t, g.numTiles, uint32_t(g.xcdGroupLog));
    MatrixTile m;
    uint32_t q = fast_div(t, g.chunksC);
    const uint32_t jc = t - q * g.chunksC.d;
    t = q;
    q = fast_div(t, g.chunksR);
    uint32_t jr = t - q * g.chunksR.d;
    t = q;
    if (g.skew) {
        jr += jc - fast_div(jc, g.chunksR) * g.chunksR.d;
        if (jr >= g.chunksR.d) jr -= g.chunksR.d;
    }
    // the last column chunk is loaded from TC columns before the end
    const int32_t c0 = int32_t(jc) * SH::TC, cols = int32_t(g.colsA);
    m.col0 = cols < SH::TC ? 0 : imin(c0, cols - SH::TC);
    m.qLo = c0 - m.col0;
    m.qHi = imin(SH::TC, cols - m.col0);
    m.row0 = int32_t(jr) * SH::TR;
    m.a = m.b = 0;
    for (int k = 0; k < g.nG; ++k) {
        q = fast_div(t, g.gExt[k]);
        const int64_t j = int64_t(t - q * g.gExt[k].d);
        m.a += j * g.gStrideA[k];
        m.b += j * g.gStrideB[k];
        t = q;
    }
    return m;
}

// The shapes, by number: columns, rows, line bytes of sheared B runs (0: runs
// start where the columns do).
#define HPTT_MATRIX_SHAPES_F32(X) \
    X(0, 32, 128, 128) X(1, 64, 64, 128) X(2, 16, 256, 128) X(3, 64, 64, 0) X(4, 128, 32, 0) \
    X(5, 32, 128, 0) X(6, 32, 32, 0) X(7, 16, 64, 0)
#define HPTT_MATRIX_SHAPES_F64(X) \
    X(0, 32, 64, 128) X(1, 16, 64, 128) X(2, 8, 128, 128) X(3, 32, 64, 0) X(4, 32, 32, 0) \
    X(5, 16, 64, 0)

// Byte offset of flattened position x.
__host__ __device__ __forceinline__ uint32_t matrix_offset(const FastDiv* ext, const uint32_t* stride,
                                                           int n, uint32_t x) {
    if (n == 1) return x * stride[0];
    uint32_t off = 0;
    for (int k = 0; k < n; ++k) {
        const uint32_t q = fast_div(x, ext[k]);
        off += (x - q * ext[k].d) * stride[k];
        x = q;
    }
    return off;
}

// Tables of one tile: rowA[R] = A offset of staged row R (run position row0 +
// R - S, or the nearest that exists), and for each column q its B offset
// colB, its shift colD below the tile's first row, and colL = q - colD * pitch.
template <class Mem, typename T, class SH>
__host__ __device__ inline void matrix_tables(const MatrixArgs& g, const MatrixTile& m, int tid,
                                              uint32_t* rowA, uint32_t* colB, int32_t* colL,
                                              int32_t* colD) {
    for (int i = tid; i < SH::rows + SH::TC; i += kBlock) {
        if (i < SH::rows) {
            int32_t p = m.row0 + i - SH::S;
            p = p < 0 ? 0 : imin(p, int32_t(g.rowsB) - 1);
            Mem::template lds_st<uint32_t>(rowA, i,
                                           matrix_offset(g.rExt, g.rStrideA, g.nR, uint32_t(p)));
        } else {
            const int q = i - SH::rows;
            const int32_t c = imin(m.col0 + q, int32_t(g.colsA) - 1);
            const uint32_t off = matrix_offset(g.cExt, g.cStrideB, g.nC, uint32_t(c));
            int32_t d = 0;
            if (SH::S)
                d = int32_t((uint32_t(m.b) + off) / sizeof(T) + uint32_t(m.row0) +
                            uint32_t(g.misLine)) & SH::S;
            Mem::template lds_st<uint32_t>(colB, q, off);
            Mem::template lds_st<int32_t>(colL, q, q - d * SH::pitch);
            Mem::template lds_st<int32_t>(colD, q, d);
        }
    }
}

// Load phase: vector c of each staged row, at any element boundary of A.
template <class Mem, typename T, int HINT, class SH>
__host__ __device__ inline void matrix_load(const MatrixArgs& g, const MatrixTile& m, int tid,
                                            const T* A, T* lds, const uint32_t* rowA) {
    const int r = tid / SH::laneC;
    // a matrix with fewer columns than the tile: its last vector twice
    const int c = imin((tid % SH::laneC) * SH::V, imin(SH::TC, int(g.colsA)) - SH::V);
    const T* base = Mem::template at_bytes<const T>(A, m.a + int64_t(m.col0) * int64_t(sizeof(T)));
    Vec<T, SH::V> v[SH::loads];
#pragma unroll
    for (int u = 0; u < SH::loads; ++u)
        v[u] = Mem::template ldub<T, SH::V, (HINT & kNtLoad) != 0>(
            base, Mem::template lds_ld<uint32_t>(rowA, r + u * SH::rowStep) +
                      uint32_t(c) * uint32_t(sizeof(T)));
#pragma unroll
    for (int u = 0; u < SH::loads; ++u)
#pragma unroll
        for (int e = 0; e < SH::V; ++e)
            Mem::template lds_st<T>(lds, (r + u * SH::rowStep) * SH::pitch + c + e, v[u].v[e]);
}

// Store phase.  Tiles whose runs lie inside the rows take whole vectors; at
// the ends of the row range vectors are checked one by one.
template <class Mem, typename T, int MODE, int HINT, class SH, bool EDGE>
__host__ __device__ inline void matrix_store_part(const MatrixArgs& g, const MatrixTile& m, int tid,
                                                  T* B, const T* lds, const uint32_t* colB,
                                                  const int32_t* colL, const int32_t* colD, T alpha,
                                                  T beta) {
    constexpr int V = SH::V, NB = SH::stores < 4 ? SH::stores : 4;
    const int s = tid % SH::laneR * V, q0 = tid / SH::laneR;
    // offsets count from S + 1 rows before the tile, so that they are not negative
    constexpr int back = SH::S ? SH::S + 1 : 0;
    T* base = Mem::template at_bytes<T>(B, m.b + (int64_t(m.row0) - back) * int64_t(sizeof(T)));
    const int at = (SH::S + s) * SH::pitch;
#pragma unroll
    for (int u0 = 0; u0 < SH::stores; u0 += NB) {
        Vec<T, V> x[NB], y[NB];
        uint32_t off[NB];
        int lo[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int q = q0 + (u0 + u) * SH::colStep;
            const int l = Mem::template lds_ld<int32_t>(colL, q);
            const int d = SH::S ? Mem::template lds_ld<int32_t>(colD, q) : 0;
            off[u] = Mem::template lds_ld<uint32_t>(colB, q) +
                     uint32_t(back + s - d) * uint32_t(sizeof(T));
            lo[u] = m.row0 + s - d;
#pragma unroll
            for (int e = 0; e < V; ++e)
                x[u].v[e] = Mem::template lds_any<T>(
                    lds, at + l + e * SH::pitch,
                    q >= m.qLo && q < m.qHi &&
                        (!EDGE || (lo[u] + e >= 0 && lo[u] + e < int(g.rowsB))));
            if (MODE == kAxpby && q >= m.qLo && q < m.qHi) {
                if (!EDGE || (lo[u] >= 0 && lo[u] + V <= int(g.rowsB))) {
                    y[u] = SH::S ? Mem::template ldb<T, V, (HINT & kNtStore) != 0>(base, off[u])
                                 : Mem::template ldub<T, V, (HINT & kNtStore) != 0>(base, off[u]);
                } else {
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        if (lo[u] + e >= 0 && lo[u] + e < int(g.rowsB))
                            y[u].v[e] = Mem::template ldb<T, 1, false>(
                                            base, off[u] + uint32_t(e) * uint32_t(sizeof(T))).v[0];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int q = q0 + (u0 + u) * SH::colStep;
            if (q < m.qLo || q >= m.qHi) continue;
            Vec<T, V> z;
#pragma unroll
            for (int e = 0; e < V; ++e)
                z.v[e] = update<MODE>(x[u].v[e], MODE == kAxpby ? y[u].v[e] : T(0), alpha, beta);
            if (!EDGE || (lo[u] >= 0 && lo[u] + V <= int(g.rowsB))) {
                if (SH::S) Mem::template stb<(HINT & kNtStore) != 0, T, V>(base, off[u], z);
                else Mem::template stub<(HINT & kNtStore) != 0, T, V>(base, off[u], z);
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (lo[u] + e >= 0 && lo[u] + e < int(g.rowsB)) {
                        Vec<T, 1> w;
                        w.v[0] = z.v[e];
                        Mem::template stb<false, T, 1>(
                            base, off[u] + uint32_t(e) * uint32_t(sizeof(T)), w);
                    }
            }
        }
    }
}

template <class Mem, typename T, int MODE, int HINT, class SH>
__host__ __device__ inline void matrix_store(const MatrixArgs& g, const MatrixTile& m, int tid,
                                             T* B, const T* lds, const uint32_t* colB,
                                             const int32_t* colL, const int32_t* colD, T alpha,
                                             T beta) {
    if (m.row0 >= SH::S && m.row0 + SH::TR <= int(g.rowsB))
        matrix_store_part<Mem, T, MODE, HINT, SH, false>(g, m, tid, B, lds, colB, colL, colD, alpha,
                                                         beta);
    else
        matrix_store_part<Mem, T, MODE, HINT, SH, true>(g, m, tid, B, lds, colB, colL, colD, alpha,
                                                        beta);
}

}  // namespace hptt
