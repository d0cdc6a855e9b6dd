// Direct contraction: C = alpha * A . B + beta * C in one pass, the operands
// read and the product written where they lie, whatever the order of their
// modes.  This header holds the argument block, its planner (host only) and
// the index arithmetic that the kernel (contract_direct.hip) and the CPU
// tests share.
//
// With the roles of contract.hip (P and Q are A and B, or B and A) the
// contraction is C[X, Y, L] = sum over K of P[X, K, L] Q[K, Y, L].  A
// workgroup computes one kBM x kBN block of C for one batch index: kBM
// combinations of X modes by kBN combinations of Y modes, over all of K in
// slices of direct_slice.  Where each row, column and contracted position lies in its
// two tensors comes from offset tables in LDS, so no mode order needs a
// transposition.
#pragma once

#include <string>

#include "hptt.h"
#include "hptt_args.h"

namespace hptt {

constexpr int kBM = 128;               // rows (X) of a block
constexpr int kBN = 64;                // columns (Y) of a block
// contracted positions per slice, 16 (fp32) or 8 (fp64)
constexpr int direct_slice(int elem) { return elem == 4 ? 16 : 8; }
// LDS pitches: k rows 16 elements apart modulo the 64 banks, so that the four
// k rows (fp32) or two (fp64) of one operand read fall on different banks.
constexpr int kPitchP = kBM + 16;
constexpr int kPitchQ = kBN + 16;

// A group of modes flattened into one index (first mode fastest), with the
// modes' strides, in bytes, in two tensors.  Offsets inside a batch are 32-bit:
// no tensor is larger than 2^32 - 1 bytes, so that a lane's address is a
// 64-bit base in scalar registers plus one 32-bit register.
struct ModeGroup {
    int32_t n;
    int32_t total;  // product of the extents
    FastDiv ext[kMaxDims];
    uint32_t s0[kMaxDims], s1[kMaxDims];
};
constexpr uint32_t kOutside = 0xffffffffu;  // C offset of a row or column that does not exist

struct DirectArgs {
    // X is split in two groups: x2 are the modes that P's memory starts with
    // when those are not C's stride-1 mode (x2.total = 1 otherwise), x1 the
    // others in C's order.  A block's rows are t1 consecutive positions of x1
    // by t2 of x2, row = i1 + t1 * i2 (t1 * t2 = kBM, t1 >= 16), so that
    // P is read and C written in runs.  s0: strides in P, s1: in C.
    ModeGroup x1, x2;
    ModeGroup y;  // s0: strides in Q, s1: in C
    ModeGroup k;  // s0: strides in P, s1: in Q
    int32_t t1log, t2log;
    // a thread's staging slot s is split by shifts: position in x1
    // (s >> sh1) & (t1 - 1), in x2 (s >> sh2) & (t2 - 1), in the slice
    // (s >> shk) & (slice - 1), the direction that is contiguous in P first
    int32_t sh1, sh2, shk;
    int32_t shn, shq;  // the same for Q: column (s >> shn) & (kBN - 1), slice (s >> shq)
    int32_t streamC;  // C, if it starts on a line, written (and read) non-temporally
    // the grid: column blocks first, then x2, x1, batch
    FastDiv tilesY, tiles2, tiles1;
    uint32_t numTiles;
    int32_t nL;
    FastDiv eL[kMaxDims];
    int64_t sLP[kMaxDims], sLQ[kMaxDims], sLC[kMaxDims];
};

// Offsets of position x of a group in its two tensors.
__host__ __device__ __forceinline__ void group_offsets(const ModeGroup& g, uint32_t x, uint32_t& o0,
                                                       uint32_t& o1) {
    o0 = o1 = 0;
    for (int j = 0; j < g.n; ++j) {
        const uint32_t q = fast_div(x, g.ext[j]);
        const uint32_t d = x - q * g.ext[j].d;
        o0 += d * g.s0[j];
        o1 += d * g.s1[j];
        x = q;
    }
}

struct DirectTile {
    int32_t y, i2, i1;       // first column, first position in x2 and x1
    int64_t offP, offQ, offC;  // the batch's offsets (bytes)
};

__host__ __device__ __forceinline__ DirectTile direct_tile(const DirectArgs& g, uint32_t t) {
    DirectTile d;
    uint32_t q = fast_div(t, g.tilesY);
    d.y = int32_t(t - q * g.tilesY.d) * kBN;
    t = q;
    q = fast_div(t, g.tiles2);
    d.i2 = int32_t(t - q * g.tiles2.d) << g.t2log;
    t = q;
    q = fast_div(t, g.tiles1);
    d.i1 = int32_t(t - q * g.tiles1.d) << g.t1log;
    t = q;
    d.offP = d.offQ = d.offC = 0;
    for (int j = 0; j < g.nL; ++j) {
        q = fast_div(t, g.eL[j]);
        const int64_t x = int64_t(t - q * g.eL[j].d);
        d.offP += x * g.sLP[j];
        d.offQ += x * g.sLQ[j];
        d.offC += x * g.sLC[j];
        t = q;
    }
    return d;
}

// Row r of a block: its offsets in P and C; outside the tensor C's is kOutside
// and P's that of the first element.
__host__ __device__ __forceinline__ void direct_row(const DirectArgs& g, const DirectTile& d, int r,
                                                    uint32_t& inP, uint32_t& inC) {
    const int32_t i1 = d.i1 + (r & ((1 << g.t1log) - 1)), i2 = d.i2 + (r >> g.t1log);
    inP = 0;
    inC = kOutside;
    if (i1 >= g.x1.total || i2 >= g.x2.total) return;
    uint32_t p1, c1, p2, c2;
    group_offsets(g.x1, uint32_t(i1), p1, c1);
    group_offsets(g.x2, uint32_t(i2), p2, c2);
    inP = p1 + p2;
    inC = c1 + c2;
}

__host__ __device__ __forceinline__ void direct_column(const DirectArgs& g, const DirectTile& d,
                                                       int c, uint32_t& inQ, uint32_t& inC) {
    inQ = 0;
    inC = kOutside;
    if (d.y + c < g.y.total) group_offsets(g.y, uint32_t(d.y + c), inQ, inC);
}

// Offsets of slice kb's position j, to *inP and *inQ; beyond the contraction those
// of its first element, whose products are left out.
__host__ __device__ __forceinline__ void direct_position(const DirectArgs& g, int slice, int kb,
                                                         int j, uint32_t* inP, uint32_t* inQ) {
    uint32_t p = 0, q = 0;
    if (kb * slice + j < g.k.total) group_offsets(g.k, uint32_t(kb * slice + j), p, q);
    *inP = p;
    *inQ = q;
}

// A block's tables, one entry per thread: rows, columns, and slice 0 (which
// is table 0 of two: slice kb + 1 goes to table (kb + 1) & 1 while the waves
// are still to multiply slice kb, whose offsets have all been used by then).
template <int SLICE>
__host__ __device__ __forceinline__ void direct_tables(const DirectArgs& g, const DirectTile& d,
                                                       int tid, uint32_t* rowP, uint32_t* rowC,
                                                       uint32_t* colQ, uint32_t* colC,
                                                       uint32_t* kP, uint32_t* kQ) {
    static_assert(kBM + kBN + SLICE <= kBlock, "every entry has a thread");
    static_assert(kBM == 32 * (kBlock / 64) && kBN == 64, "wave w takes rows 32 w to 32 w + 31");
    if (tid < kBM) direct_row(g, d, tid, rowP[tid], rowC[tid]);
    else if (tid < kBM + kBN) direct_column(g, d, tid - kBM, colQ[tid - kBM], colC[tid - kBM]);
    else if (tid < kBM + kBN + SLICE)
        direct_position(g, SLICE, 0, tid - kBM - kBN, &kP[tid - kBM - kBN], &kQ[tid - kBM - kBN]);
}

// Staging slot s of P: row, slice position and place in a slice's LDS row.
// Each step of x2 is padded by one element, so that lanes that walk x2
// write different banks.
struct DirectSlot {
    int row, k, at;
};
__host__ __device__ __forceinline__ DirectSlot direct_slot_p(const DirectArgs& g, int s,
                                                             int slice) {
    const int t1 = 1 << g.t1log;
    const int i1 = (s >> g.sh1) & (t1 - 1), i2 = (s >> g.sh2) & ((1 << g.t2log) - 1);
    DirectSlot x;
    x.row = i1 + (i2 << g.t1log);
    x.k = (s >> g.shk) & (slice - 1);
    x.at = i1 + i2 * (t1 + 1);
    return x;
}
__host__ __device__ __forceinline__ DirectSlot direct_slot_q(const DirectArgs& g, int s,
                                                             int slice) {
    DirectSlot x;
    x.row = (s >> g.shn) & (kBN - 1);
    x.k = (s >> g.shq) & (slice - 1);
    x.at = x.row;
    return x;
}

// Place in a slice's LDS row of the 16 rows from r on (a multiple of 16).
__host__ __device__ __forceinline__ int direct_rows_at(const DirectArgs& g, int r) {
    const int t1 = 1 << g.t1log;
    return (r & (t1 - 1)) + (r >> g.t1log) * (t1 + 1);
}

// Fill *g for C[modesC] = P[modesP] . Q[modesQ] (extents by mode).  Returns
// false where the kernel does not serve the problem: C's stride-1 mode is not
// one of X, a tensor of 2^32 bytes or more, too many blocks.
bool plan_direct(const std::string& modesP, const std::string& modesQ, const std::string& modesC,
                 const int64_t* ext, int elem, DirectArgs* g);

// Estimated time in microseconds (MI355X) of the kernel on a planned problem,
// and of `transposes` transpositions of `bytesMoved` bytes in all around a GEMM of
// m x n x k, `batch` times, that reads its C or does not.
double direct_us(const DirectArgs& g, int elem, bool beta);
double transposed_us(double m, double n, double k, double batch, int elem, int transposes,
                     double bytesMoved, bool readC);

// In libhptt.so: a failed launch's error, for hptt_last_hip_error; and a plan
// whose result is read next, so that nothing of it is stored non-temporally.
void record_hip_error(hipError_t err);
void keep_cached(hptt_plan_t plan);

// Queue the kernel; false (and the HIP error) if the launch failed.
bool launch_direct(const DirectArgs& g, bool f64, const void* P, const void* Q, void* C,
                   double alpha, double beta, hipStream_t stream, hipError_t* err);

}  // namespace hptt
