// Kernel P instantiations: shared-run tiles permuted in LDS (perm_body.h).
#include "device_mem.h"
#include "perm_body.h"

namespace hptt {
namespace {

template <typename T, int N, int MODE, int HINT>
__global__ __launch_bounds__(kBlock) void perm_kernel(const T* __restrict__ A, T* __restrict__ B,
                                                      const PermArgs g, T alpha, T beta) {
    extern __shared__ int64_t smem[];
    T* lds = reinterpret_cast<T*>(smem);
    const int tid = int(threadIdx.x);
    uint32_t t = blockIdx.x;
    if (t >= g.numTiles) return;
    PermLane<T, N> l;
    perm_setup<T, N>(g, tid, l);
    Vec<T, PermLane<T, N>::V> x[N];
    PermTile p = perm_tile(g, t);
    perm_load<DeviceMem, T, N, HINT>(g, p, tid, l, A, x);
    for (;;) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            DeviceMem::opaque(l.rc[u]);
            DeviceMem::opaque(l.qb[u]);
            DeviceMem::opaque(l.offA[u]);
            DeviceMem::opaque(l.offB[u]);
#pragma unroll
            for (int e = 0; e < PermLane<T, N>::V / 2; ++e) DeviceMem::opaque(l.src[u][e]);
        }
        // in the order they are waited for: this tile's B, the next tile's A
        Vec<T, PermLane<T, N>::V> y[N];
        if (MODE == kAxpby) perm_prior<DeviceMem, T, N, HINT>(g, p, tid, l, B, y);
        perm_stage<DeviceMem, T, N>(g, tid, l, lds, x);
        __syncthreads();
        const PermTile now = p;
        t += gridDim.x;
        const bool more = t < g.numTiles;
        if (more) {  // the next tile's A while this one is written
            p = perm_tile(g, t);
            perm_load<DeviceMem, T, N, HINT>(g, p, tid, l, A, x);
        }
        perm_store<DeviceMem, T, N, MODE, HINT>(g, now, tid, l, B, lds, y, alpha, beta);
        if (!more) break;
        __syncthreads();  // this tile's LDS reads are done
    }
}

template <typename T, int N, int MODE>
const void* by_hint(int hints) {
    if (hints == (kNtStore | kNtLoad))
        return reinterpret_cast<const void*>(&perm_kernel<T, N, MODE, kNtStore | kNtLoad>);
    if (hints == kNtStore) return reinterpret_cast<const void*>(&perm_kernel<T, N, MODE, kNtStore>);
    return reinterpret_cast<const void*>(&perm_kernel<T, N, MODE, 0>);
}

template <typename T, int N>
const void* by_mode(int mode, int hints) {
    switch (mode) {
        case kCopy: return by_hint<T, N, kCopy>(hints);
        case kScale: return by_hint<T, N, kScale>(hints);
        default: return by_hint<T, N, kAxpby>(hints);
    }
}

template <typename T>
const void* by_vectors(int n, int mode, int hints) {
    switch (n) {
        case 1: return by_mode<T, 1>(mode, hints);
        case 2: return by_mode<T, 2>(mode, hints);
        case 3: return by_mode<T, 3>(mode, hints);
        case 5: return by_mode<T, 5>(mode, hints);
    }
    return nullptr;
}

}  // namespace

const void* perm_kernel_f32(int vectors, int mode, int hints) {
    return by_vectors<float>(vectors, mode, hints);
}

const void* perm_kernel_f64(int vectors, int mode, int hints) {
    return by_vectors<double>(vectors, mode, hints);
}

}  // namespace hptt
