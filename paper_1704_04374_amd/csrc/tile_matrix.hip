// Kernel M instantiations: flattened two-dimensional tiles (matrix_body.h).
#include "device_mem.h"
#include "matrix_body.h"

namespace hptt {
namespace {

// One tile per workgroup: tables, A runs into LDS, B runs out of it.  Kernel T
// was bound by its instructions where runs start off the vector grid: 615
// VALU and 560 scalar instructions per wave on 2193 x 22800 fp32, 50 of its 80
// us at one VALU instruction per SIMD and 4 cycles (rocprofv3 SQ_INSTS_VALU),
// spent on run-time divisions, vector checks and the shift of every vector.
// Here the tile's size is a compile-time constant, A is read with 16-byte
// vectors from any element boundary, and one table pass per tile holds every
// row's and column's offset, so a vector costs a table read, one addition,
// the access and its LDS words.  MI355X, kernel T -> kernel M: 2193 x 22800
// 80.4 -> 75.6 us (5.3 TB/s), 427x110x3x355 reversed with beta = 1 143.7 ->
// 121.6, an fp64 block of 65x33x64x9 15.5 -> 7, 64 x 3136 x 64 [1,0,2]
// 22.5 -> 19.1, fp64 8192 x 4096 with beta = 1 190 -> 136.
template <typename T, int MODE, int HINT, class SH>
__global__ __launch_bounds__(kBlock) void matrix_kernel(const T* __restrict__ A, T* __restrict__ B,
                                                        const MatrixArgs g, T alpha, T beta) {
    __shared__ __align__(16) char smem[SH::ldsBytes];
    uint32_t* rowA = reinterpret_cast<uint32_t*>(smem);
    uint32_t* colB = rowA + SH::rows;
    int32_t* colL = reinterpret_cast<int32_t*>(colB + SH::TC);
    int32_t* colD = colL + SH::TC;
    T* lds = reinterpret_cast<T*>(smem + (SH::tableBytes + 15) / 16 * 16);
    const int tid = int(threadIdx.x);
    const MatrixTile m = matrix_tile<SH>(g, blockIdx.x);
    matrix_tables<DeviceMem, T, SH>(g, m, tid, rowA, colB, colL, colD);
    __syncthreads();
    matrix_load<DeviceMem, T, HINT, SH>(g, m, tid, A, lds, rowA);
    __syncthreads();
    matrix_store<DeviceMem, T, MODE, HINT, SH>(g, m, tid, B, lds, colB, colL, colD, alpha, beta);
}

template <typename T, int MODE, class SH>
const void* by_hint(int hints) {
    // non-temporal loads only where a tile's rows are whole lines and start on
    // them (choose_matrix), which sheared and narrower tiles never have
    if constexpr (SH::S == 0 && SH::TC * sizeof(T) % 128 == 0)
        if (hints == (kNtStore | kNtLoad))
            return reinterpret_cast<const void*>(&matrix_kernel<T, MODE, kNtStore | kNtLoad, SH>);
    return hints == kNtStore ? reinterpret_cast<const void*>(&matrix_kernel<T, MODE, kNtStore, SH>)
           : hints == 0      ? reinterpret_cast<const void*>(&matrix_kernel<T, MODE, 0, SH>)
                             : nullptr;
}

template <typename T, class SH>
const void* by_mode(int mode, int hints) {
    switch (mode) {
        case kCopy: return by_hint<T, kCopy, SH>(hints);
        case kScale: return by_hint<T, kScale, SH>(hints);
        default: return by_hint<T, kAxpby, SH>(hints);
    }
}

}  // namespace

const void* matrix_kernel_f32(int shape, int mode, int hints) {
    switch (shape) {
#define X(id, tc, tr, line) \
    case id: return by_mode<float, MatrixShape<float, tc, tr, line>>(mode, hints);
        HPTT_MATRIX_SHAPES_F32(X)
#undef X
    }
    return nullptr;
}

const void* matrix_kernel_f64(int shape, int mode, int hints) {
    switch (shape) {
#define X(id, tc, tr, line) \
    case id: return by_mode<double, MatrixShape<double, tc, tr, line>>(mode, hints);
        HPTT_MATRIX_SHAPES_F64(X)
#undef X
    }
    return nullptr;
}

}  // namespace hptt
