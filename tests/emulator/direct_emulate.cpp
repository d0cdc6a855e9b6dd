// Host emulation of the direct contraction kernel, for CPU tests only: its
// planner and the index code of contract_direct.h in the kernel's order, block by
// block, with every offset checked against its tensor, every table entry and LDS
// place written before it is read, and every LDS place once per slice.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "contract_direct.h"
#include "kernel_body.h"

namespace {

struct Check {
    long errors = 0;
    char msg[256] = "";
    void fail(const char* what, long long a, long long b) {
        if (errors++ == 0) snprintf(msg, sizeof(msg), "%s (%lld, %lld)", what, a, b);
    }
};

// A table entry that no thread has written; no offset of a tensor below 2^32
// bytes is odd.
constexpr uint32_t kUnwritten = 0xfffffffdu;

// Products are summed in double, whatever T: the tests take whole numbers.
template <typename T>
int64_t emulate(const char* mA, const char* mB, const char* mC, const int64_t* ext256,
                double alpha, double beta, const T* A, const T* B, T* C, uint8_t* counts,
                int64_t blockStride, char* msg, size_t msglen) {
    using namespace hptt;
    constexpr int elem = int(sizeof(T)), kBK = direct_slice(elem);
    constexpr int kSlotsP = kBM * kBK / kBlock, kSlotsQ = kBN * kBK / kBlock;
    DirectArgs g;
    const T *P = A, *Q = B;
    std::string mP = mA, mQ = mB;
    if (!plan_direct(mA, mB, mC, ext256, elem, &g)) {
        if (!plan_direct(mB, mA, mC, ext256, elem, &g)) return -1;
        P = B;
        Q = A;
        std::swap(mP, mQ);
    }
    auto volume = [&](const std::string& m) {
        int64_t v = 1;
        for (char c : m) v *= ext256[static_cast<unsigned char>(c)];
        return v;
    };
    const int64_t nP = volume(mP), nQ = volume(mQ), nC = volume(mC);
    Check ck;
    std::vector<double> ldsP(kBK * kPitchP), ldsQ(kBK * kPitchQ);
    std::vector<int> seenP(kBK * kPitchP), seenQ(kBK * kPitchQ);
    std::vector<double> vp(kSlotsP * kBlock), vq(kSlotsQ * kBlock), sum(kBM * kBN);
    const int64_t last = int64_t(g.numTiles) - 1;  // (a sample has the last block too)
    for (int64_t blk = 0;; blk = std::min(blk + blockStride, last)) {
        const DirectTile d = direct_tile(g, xcd_group_map(uint32_t(blk), g.numTiles, 4));
        uint32_t rowP[kBM], rowC[kBM], colQ[kBN], colC[kBN], kP[2][kBK], kQ[2][kBK];
        for (auto* t : {rowP, rowC}) std::fill(t, t + kBM, kUnwritten);
        for (auto* t : {colQ, colC}) std::fill(t, t + kBN, kUnwritten);
        for (auto* t : {kP[0], kP[1], kQ[0], kQ[1]}) std::fill(t, t + kBK, kUnwritten);
        for (int tid = 0; tid < kBlock; ++tid)
            direct_tables<kBK>(g, d, tid, rowP, rowC, colQ, colC, kP[0], kQ[0]);
        std::fill(sum.begin(), sum.end(), 0.0);
        // what the threads' slots hold of slice kb
        auto fetch = [&](int kb, bool p) {
            const int which = kb & 1, left = g.k.total - kb * kBK;
            for (int s = 0; s < (p ? kSlotsP : kSlotsQ) * kBlock; ++s) {
                const DirectSlot x = p ? direct_slot_p(g, s, kBK) : direct_slot_q(g, s, kBK);
                if (x.row < 0 || x.row >= (p ? kBM : kBN) || x.k < 0 || x.k >= kBK) {
                    ck.fail("slot out of range", s, x.row);
                    continue;
                }
                const uint32_t row = p ? rowP[x.row] : colQ[x.row];
                const uint32_t pos = p ? kP[which][x.k] : kQ[which][x.k];
                if (row == kUnwritten || pos == kUnwritten) ck.fail("table read before write", s, kb);
                const uint32_t off = row + pos;  // 32 bits, as in the kernel
                const int64_t at = (p ? d.offP : d.offQ) + int64_t(off), end = (p ? nP : nQ) * elem;
                if (int64_t(row) + int64_t(pos) != int64_t(off) || off % elem || at < 0 ||
                    at + elem > end) {
                    ck.fail(p ? "P offset out of range" : "Q offset out of range", at, blk);
                    continue;
                }
                (p ? vp : vq)[s] = A && x.k < left ? double((p ? P : Q)[at / elem]) : 0.0;
            }
        };
        auto stage = [&](bool p) {
            auto& seen = p ? seenP : seenQ;
            const int pitch = p ? kPitchP : kPitchQ;
            std::fill(seen.begin(), seen.end(), 0);
            for (int s = 0; s < (p ? kSlotsP : kSlotsQ) * kBlock; ++s) {
                const DirectSlot x = p ? direct_slot_p(g, s, kBK) : direct_slot_q(g, s, kBK);
                if (x.at < 0 || x.at >= pitch || x.k * pitch + x.at >= (1 << 16)) {
                    ck.fail("LDS place out of range", s, x.at);
                    continue;
                }
                (p ? ldsP : ldsQ)[x.k * pitch + x.at] = (p ? vp : vq)[s];
                if (seen[x.k * pitch + x.at]++) ck.fail("LDS place written twice", x.k, x.at);
            }
        };
        const int slices = (g.k.total + kBK - 1) / kBK;
        fetch(0, true);
        fetch(0, false);
        for (int kb = 0;; ++kb) {
            stage(true);
            stage(false);
            const bool more = kb + 1 < slices;
            const int next = (kb + 1) & 1;
            if (more) {
                for (int j = 0; j < kBK; ++j)
                    direct_position(g, kBK, kb + 1, j, &kP[next][j], &kQ[next][j]);
                fetch(kb + 1, true);
                fetch(kb + 1, false);
                // stale from here on: the next entries go there
                std::fill(kP[kb & 1], kP[kb & 1] + kBK, kUnwritten);
                std::fill(kQ[kb & 1], kQ[kb & 1] + kBK, kUnwritten);
            }
            for (int k = 0; k < kBK; ++k)
                for (int r = 0; r < kBM; ++r) {
                    const int at = k * kPitchP + direct_rows_at(g, r & ~15) + (r & 15);
                    if (at >= kBK * kPitchP || !seenP[at]) ck.fail("P read before write", k, r);
                    for (int c = 0; A && c < kBN; ++c)
                        sum[r * kBN + c] += ldsP[at] * ldsQ[k * kPitchQ + c];
                }
            if (!more) break;
        }
        for (int r = 0; r < kBM; ++r)
            for (int c = 0; c < kBN; ++c) {
                if (rowC[r] == kOutside || colC[c] == kOutside) continue;
                const uint32_t off = rowC[r] + colC[c];
                const int64_t at = (d.offC + int64_t(off)) / elem;
                if (int64_t(rowC[r]) + int64_t(colC[c]) != int64_t(off) || off % elem || at < 0 ||
                    at >= nC) {
                    ck.fail("C offset out of range", at, blk);
                    continue;
                }
                if (counts) counts[at]++;
                if (A) {
                    const double v = alpha * sum[r * kBN + c];
                    C[at] = T(v + (beta != 0 ? beta * double(C[at]) : 0.0));
                }
            }
        if (blk == last) break;
    }
    if (msg && msglen) snprintf(msg, msglen, "%s", ck.msg);
    return ck.errors;
}

}  // namespace

extern "C" {

// C = alpha * A . B + beta * C in fp64 (elem 8) or fp32 (elem 4).  Returns -1
// where the planner refuses, else the number of index errors.  counts: how often
// each C element is written.  blockStride > 1 runs a sample of the blocks; A
// NULL: indexes only.
int64_t direct_emulate(const char* mA, const char* mB, const char* mC, const int64_t* ext256,
                       int32_t elem, double alpha, double beta, const void* A, const void* B,
                       void* C, uint8_t* counts, int64_t blockStride, char* msg, size_t msglen) {
    if (elem == 4)
        return emulate<float>(mA, mB, mC, ext256, alpha, beta, static_cast<const float*>(A),
                              static_cast<const float*>(B), static_cast<float*>(C), counts,
                              blockStride, msg, msglen);
    return emulate<double>(mA, mB, mC, ext256, alpha, beta, static_cast<const double*>(A),
                           static_cast<const double*>(B), static_cast<double*>(C), counts,
                           blockStride, msg, msglen);
}

}  // extern "C"
