// The direct contraction kernel (contract_direct.h).
#include <hip/hip_runtime.h>

#include "contract_direct.h"
#include "kernel_body.h"

namespace hptt {
namespace {

template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
    typedef double acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mac(double a, double b, acc c) {
#if defined(__HIP_DEVICE_COMPILE__)
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
#else
        return c;
#endif
    }
    // row of the 16x16 product that register r of a lane holds
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }
};
template <>
struct Mfma<float> {
    typedef float acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mac(float a, float b, acc c) {
#if defined(__HIP_DEVICE_COMPILE__)
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
#else
        return c;
#endif
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// The element at a byte offset from a base that the whole wave shares.
template <typename T>
__device__ __forceinline__ T at_bytes(const T* base, uint32_t off) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + off);
}

// One 128 x 64 block of C per workgroup.  Per slice each thread holds the next
// slice's elements in registers while the waves multiply the staged one (one
// LDS buffer, two barriers); offsets come from LDS tables computed once per
// block, the contracted positions' per slice.  fp64 takes slices of 8 and is held
// to 128 registers (4 waves per SIMD): against slices of 16 and 3 waves, abcd =
// dbea.ec (64 contracted) 207 -> 175 us, abc = bda.dc 96 -> 87; a long
// contraction, bound by the chain of slices, loses 3 to 9 %.  fp32 is held to 96
// (5 waves): with 98, at 4 waves, many small products took up to 1.19x as long
// (cdahb = eghaf.fcbdehg, 213 batches of 341 x 12 x 10: 10.3 -> 12.3 us).
// With few contracted elements the kernel is bound by the traffic of C: fp64
// abcde = efbad.cf (340 MB of tensors, 2.0 GFLOP) takes 73 us, 4.7 TB/s,
// where transposition - GEMM - transposition moves 1.0 GB in 235 us.  Lanes
// store 16 rows of 4 columns at a time, 128-byte (fp64) pieces of C.
template <typename T, bool BETA, bool NT>
__global__ __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 4 : 5))) void direct_kernel(
        const T* __restrict__ P0, const T* __restrict__ Q0, T* __restrict__ C0, const DirectArgs g,
        T alpha, T beta) {
    typedef typename Mfma<T>::acc acc;
    constexpr int kBK = direct_slice(sizeof(T));
    constexpr int kSlotsP = kBM * kBK / kBlock;  // elements a thread stages per slice
    constexpr int kSlotsQ = kBN * kBK / kBlock;
    __shared__ T ldsP[kBK * kPitchP];
    __shared__ T ldsQ[kBK * kPitchQ];
    __shared__ uint32_t rowP[kBM], rowC[kBM], colQ[kBN], colC[kBN];
    __shared__ uint32_t kP[2][kBK], kQ[2][kBK];
    const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    const DirectTile d = direct_tile(g, xcd_group_map(blockIdx.x, g.numTiles, 4));
    const T* P = reinterpret_cast<const T*>(reinterpret_cast<const char*>(P0) + d.offP);
    const T* Q = reinterpret_cast<const T*>(reinterpret_cast<const char*>(Q0) + d.offQ);
    T* C = reinterpret_cast<T*>(reinterpret_cast<char*>(C0) + d.offC);
    direct_tables<kBK>(g, d, tid, rowP, rowC, colQ, colC, kP[0], kQ[0]);
    __syncthreads();
    // this thread's staging slots: offset of the row or column, place in LDS
    // and position in the slice (two 16-bit numbers)
    uint32_t inP[kSlotsP], inQ[kSlotsQ];
    int toP[kSlotsP], toQ[kSlotsQ];
#pragma unroll
    for (int u = 0; u < kSlotsP; ++u) {
        const DirectSlot s = direct_slot_p(g, u * kBlock + tid, kBK);
        inP[u] = rowP[s.row];
        toP[u] = (s.k << 16) | (s.k * kPitchP + s.at);
    }
#pragma unroll
    for (int u = 0; u < kSlotsQ; ++u) {
        const DirectSlot s = direct_slot_q(g, u * kBlock + tid, kBK);
        inQ[u] = colQ[s.row];
        toQ[u] = (s.k << 16) | (s.k * kPitchQ + s.at);
    }
    T vp[kSlotsP], vq[kSlotsQ];
    auto fetch = [&](int kb) {
        const int which = kb & 1, left = g.k.total - kb * kBK;
#pragma unroll
        for (int u = 0; u < kSlotsP; ++u)  // always inside P
            vp[u] = at_bytes(P, inP[u] + kP[which][toP[u] >> 16]);
#pragma unroll
        for (int u = 0; u < kSlotsQ; ++u) vq[u] = at_bytes(Q, inQ[u] + kQ[which][toQ[u] >> 16]);
        if (left < kBK) {
#pragma unroll
            for (int u = 0; u < kSlotsP; ++u) vp[u] = (toP[u] >> 16) < left ? vp[u] : T(0);
#pragma unroll
            for (int u = 0; u < kSlotsQ; ++u) vq[u] = (toQ[u] >> 16) < left ? vq[u] : T(0);
        }
    };
    // wave w computes rows [32w, 32w + 32) by all columns: 2 x 4 products of
    // 16 x 16, transposed (the lane's low four bits are the row in C, along
    // which C is contiguous)
    acc sum[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[i][j] = acc{0, 0, 0, 0};
    int base[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        base[i] = direct_rows_at(g, wave * 32 + i * 16) + (lane & 15) + (lane >> 4) * kPitchP;
    const int baseQ = (lane & 15) + (lane >> 4) * kPitchQ;
    const int cols = (imin(kBN, g.y.total - d.y) + 15) / 16;  // 16-column products with work
    const int slices = (g.k.total + kBK - 1) / kBK;
    fetch(0);
    for (int kb = 0;; ++kb) {
#pragma unroll
        for (int u = 0; u < kSlotsP; ++u) ldsP[toP[u] & 0xffff] = vp[u];
#pragma unroll
        for (int u = 0; u < kSlotsQ; ++u) ldsQ[toQ[u] & 0xffff] = vq[u];
        const bool more = kb + 1 < slices;
        const int next = (kb + 1) & 1;
        if (more && tid < kBK) direct_position(g, kBK, kb + 1, tid, &kP[next][tid], &kQ[next][tid]);
        __syncthreads();
        if (more) fetch(kb + 1);
#pragma unroll
        for (int k4 = 0; k4 < kBK; k4 += 4) {
            T p[2], q[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) p[i] = ldsP[k4 * kPitchP + base[i]];
#pragma unroll
            for (int j = 0; j < 4; ++j) q[j] = ldsQ[k4 * kPitchQ + j * 16 + baseQ];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < cols) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) sum[i][j] = Mfma<T>::mac(q[j], p[i], sum[i][j]);
                }
        }
        if (!more) break;
        __syncthreads();
    }
    uint32_t inC[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) inC[i] = rowC[wave * 32 + i * 16 + (lane & 15)];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t cc[4];
        T old[4][2];
#pragma unroll
        for (int r = 0; r < 4; ++r) cc[r] = colC[j * 16 + Mfma<T>::row(lane, r)];
        if (BETA) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (inC[i] != kOutside && cc[r] != kOutside) {
                        const T* at = reinterpret_cast<const T*>(reinterpret_cast<const char*>(C) +
                                                                 (inC[i] + cc[r]));
                        old[r][i] = NT ? __builtin_nontemporal_load(at) : *at;
                    }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (inC[i] != kOutside && cc[r] != kOutside) {
                    T* at = reinterpret_cast<T*>(reinterpret_cast<char*>(C) + (inC[i] + cc[r]));
                    T x = alpha * sum[i][j][r];
                    if (BETA) x += beta * old[r][i];
                    if (NT) __builtin_nontemporal_store(x, at);
                    else *at = x;
                }
    }
}

template <typename T>
const void* kernel_of(bool beta, bool nt) {
    if constexpr (sizeof(T) == 8)  // (plan_direct: never in fp32)
        if (nt)
            return beta ? reinterpret_cast<const void*>(&direct_kernel<T, true, true>)
                        : reinterpret_cast<const void*>(&direct_kernel<T, false, true>);
    return beta ? reinterpret_cast<const void*>(&direct_kernel<T, true, false>)
                : reinterpret_cast<const void*>(&direct_kernel<T, false, false>);
}

}  // namespace

bool launch_direct(const DirectArgs& g, bool f64, const void* P, const void* Q, void* C,
                   double alpha, double beta, hipStream_t stream, hipError_t* err) {
    // C off the lines: its runs are not whole lines in memory
    const bool nt = g.streamC && reinterpret_cast<uintptr_t>(C) % 128 == 0;
    const void* fn =
        f64 ? kernel_of<double>(beta != 0, nt) : kernel_of<float>(float(beta) != 0.f, nt);
    DirectArgs args = g;
    float af = float(alpha), bf = float(beta);
    double ad = alpha, bd = beta;
    void* a = f64 ? static_cast<void*>(&ad) : &af;
    void* b = f64 ? static_cast<void*>(&bd) : &bf;
    void* params[6] = {&P, &Q, &C, &args, a, b};
    *err = hipLaunchKernel(fn, dim3(g.numTiles), dim3(kBlock), params, 0, stream);
    return *err == hipSuccess;
}

}  // namespace hptt
