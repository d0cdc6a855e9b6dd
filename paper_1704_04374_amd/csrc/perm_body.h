// Kernel P: tiles whose A run and B run share indices, permuted inside LDS by
// workgroups that take several tiles.  What a lane does in a tile -- where its
// vectors lie in A, in LDS and in B, and which LDS elements make up a B
// vector -- is the same in every tile, so it is worked out once per workgroup
// and kept in registers; a tile then costs its scalar base and, per vector,
// the access and its LDS words.
//
// Kernel T's shared tiles are bound by issue, not by HBM: 2925x1207x2x7
// [2,0,3,1] fp32 takes 38 M vector instructions, 62 of its 91 us at one per SIMD
// and 4 cycles, most of them for these numbers; here 6.8 M and 81 us.  Over 60
// drawn fp32 problems of 2 x 120 to 2 x 260 MB 2.9-4.5 TB/s become 3.8-5.3 (0.84
// of the time; the copy kernel moves 6.7), and 7-12 us below 1 MB become 4-6.
// One-element LDS stores and loads, because a row's start in LDS and a B
// vector's elements lie anywhere; the next tile's A is fetched while this one is
// written.
#pragma once

#include "kernel_body.h"

namespace hptt {

template <typename T, int N>
struct PermLane {
    static constexpr int V = int(16 / sizeof(T));
    uint32_t offA[N];         // byte offset of load vector u in the tile's A
    uint32_t rc[N];           // its row and column (16 bits each)
    uint32_t offB[N];         // byte offset of store vector u in the tile's B
    uint32_t qb[N];           // its column and position in the B run
    uint32_t src[N][V / 2];   // LDS elements of its V elements (16 bits each)
};

struct PermTile {
    int64_t a, b;  // byte offsets
    int32_t cols, rows, colsS, runB;  // valid A run, load rows, store columns, B run
    bool whole;
};

__host__ __device__ inline PermTile perm_tile(const PermArgs& g, uint32_t t) {
    if (g.xcdGroupLog) t = xcd_group_map(t, g.numTiles, uint32_t(g.xcdGroupLog));
    PermTile p;
    p.a = p.b = 0;
    p.cols = g.runA;
    p.rows = g.rows;
    p.colsS = g.colsS;
    p.runB = g.runB;
    uint32_t j0 = 0;
    for (int k = 0; k < g.nG; ++k) {
        const uint32_t q = fast_div(t, g.gExt[k]);
        uint32_t j = t - q * g.gExt[k].d;
        t = q;
        if (k == 0) j0 = j;
        if (k == 1 && g.skew) {
            j += j0 - fast_div(j0, g.gExt[1]) * g.gExt[1].d;
            if (j >= g.gExt[1].d) j -= g.gExt[1].d;
        }
        p.a += int64_t(j) * g.gStrideA[k];
        p.b += int64_t(j) * g.gStrideB[k];
        if (k == g.gChunkC) {
            const int32_t m = imin(g.cChunk, g.cLast - int32_t(j) * g.cChunk);
            p.cols = g.cInner * m;
            if (g.cInnerS) p.colsS = g.cInnerS * m;
        }
        if (k == g.gChunkR) {
            const int32_t m = imin(g.rChunk, g.rLast - int32_t(j) * g.rChunk);
            p.runB = g.rInner * m;
            if (g.rInnerL) p.rows = g.rInnerL * m;
        }
    }
    p.whole = p.cols == g.runA && p.rows == g.rows && p.colsS == g.colsS && p.runB == g.runB;
    return p;
}

// Digits of x over ext, weighted.
__host__ __device__ __forceinline__ uint32_t perm_weigh(const FastDiv* ext, const uint32_t* w, int n,
                                                        uint32_t x) {
    uint32_t s = 0;
    for (int k = 0; k < n; ++k) {
        const uint32_t q = fast_div(x, ext[k]);
        s += (x - q * ext[k].d) * w[k];
        x = q;
    }
    return s;
}

template <typename T, int N>
__host__ __device__ inline void perm_setup(const PermArgs& g, int tid, PermLane<T, N>& l) {
    constexpr int V = PermLane<T, N>::V;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const uint32_t i = uint32_t(u * kBlock + tid);
        const uint32_t r = fast_div(i, g.vecsA);
        // the last vector of a row ends with it
        const uint32_t c = imin((i - r * g.vecsA.d) * uint32_t(V), uint32_t(g.runA - V));
        l.offA[u] = perm_weigh(g.rExt, g.rStrideA, g.nR, r) + c * uint32_t(sizeof(T));
        l.rc[u] = (r << 16) | c;
        const uint32_t q = fast_div(i, g.vecsB), b = (i - q * g.vecsB.d) * uint32_t(V);
        l.offB[u] = perm_weigh(g.cExt, g.cStrideB, g.nC, q) + b * uint32_t(sizeof(T));
        l.qb[u] = (q << 16) | b;
        const uint32_t col = perm_weigh(g.cExt, g.cLds, g.nC, q);
        uint32_t pos[V];
#pragma unroll
        for (int e = 0; e < V; ++e)
            pos[e] = col + perm_weigh(g.oExt, g.oLds, g.nO, imin(b + uint32_t(e), uint32_t(g.runB) - 1));
#pragma unroll
        for (int e = 0; e < V / 2; ++e) l.src[u][e] = (pos[2 * e] & 0xffff) | (pos[2 * e + 1] << 16);
    }
}

// A into registers.
template <class Mem, typename T, int N, int HINT>
__host__ __device__ inline void perm_load(const PermArgs& g, const PermTile& p, int tid,
                                          const PermLane<T, N>& l, const T* A,
                                          Vec<T, PermLane<T, N>::V> (&x)[N]) {
    constexpr int V = PermLane<T, N>::V;
    const T* base = Mem::template at_bytes<const T>(A, p.a);
    if (p.whole) {
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (u * kBlock + tid < g.loads)
                x[u] = Mem::template ldub<T, V, (HINT & kNtLoad) != 0>(base, l.offA[u]);
        return;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int r = int(l.rc[u] >> 16), c = int(l.rc[u] & 0xffff);
        if (u * kBlock + tid >= g.loads || r >= p.rows) continue;
        if (c + V <= p.cols) {
            x[u] = Mem::template ldub<T, V, false>(base, l.offA[u]);
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (c + e < p.cols)
                    x[u].v[e] = Mem::template ldub<T, 1, false>(
                                    base, l.offA[u] + uint32_t(e) * uint32_t(sizeof(T))).v[0];
        }
    }
}

template <class Mem, typename T, int N>
__host__ __device__ inline void perm_stage(const PermArgs& g, int tid, const PermLane<T, N>& l,
                                           T* lds, const Vec<T, PermLane<T, N>::V> (&x)[N]) {
    constexpr int V = PermLane<T, N>::V;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (u * kBlock + tid >= g.loads) continue;
        const int at = int(l.rc[u] >> 16) * g.pitch + int(l.rc[u] & 0xffff);
#pragma unroll
        for (int e = 0; e < V; ++e) Mem::template lds_st<T>(lds, at + e, x[u].v[e]);
    }
}

// Elements of store vector u that exist in this tile.
template <int V>
__host__ __device__ __forceinline__ int perm_count(const PermTile& p, uint32_t qb) {
    const int q = int(qb >> 16), b = int(qb & 0xffff);
    return q < p.colsS ? imin(V, p.runB - b) : 0;
}

// B into registers, where it is read.
template <class Mem, typename T, int N, int HINT>
__host__ __device__ inline void perm_prior(const PermArgs& g, const PermTile& p, int tid,
                                           const PermLane<T, N>& l, const T* B,
                                           Vec<T, PermLane<T, N>::V> (&y)[N]) {
    constexpr int V = PermLane<T, N>::V;
    const T* base = Mem::template at_bytes<const T>(B, p.b);
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (u * kBlock + tid >= g.stores) continue;
        const int n = perm_count<V>(p, l.qb[u]);
        if (n == V) {
            y[u] = Mem::template ldub<T, V, (HINT & kNtStore) != 0>(base, l.offB[u]);
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (e < n)
                    y[u].v[e] = Mem::template ldub<T, 1, false>(
                                    base, l.offB[u] + uint32_t(e) * uint32_t(sizeof(T))).v[0];
        }
    }
}

// LDS to B.
template <class Mem, typename T, int N, int MODE, int HINT>
__host__ __device__ inline void perm_store(const PermArgs& g, const PermTile& p, int tid,
                                           const PermLane<T, N>& l, T* B, const T* lds,
                                           const Vec<T, PermLane<T, N>::V> (&y)[N], T alpha,
                                           T beta) {
    constexpr int V = PermLane<T, N>::V;
    T* base = Mem::template at_bytes<T>(B, p.b);
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (u * kBlock + tid >= g.stores) continue;
        Vec<T, V> z;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const uint32_t two = l.src[u][e / 2];
            const T x = Mem::template lds_any<T>(lds, int(e % 2 ? two >> 16 : two & 0xffff),
                                                 e < perm_count<V>(p, l.qb[u]));
            z.v[e] = update<MODE>(x, MODE == kAxpby ? y[u].v[e] : T(0), alpha, beta);
        }
        const int n = perm_count<V>(p, l.qb[u]);
        if (n == V) {
            Mem::template stub<(HINT & kNtStore) != 0, T, V>(base, l.offB[u], z);
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (e < n) {
                    Vec<T, 1> w;
                    w.v[0] = z.v[e];
                    Mem::template stub<false, T, 1>(
                        base, l.offB[u] + uint32_t(e) * uint32_t(sizeof(T)), w);
                }
        }
    }
}

}  // namespace hptt
