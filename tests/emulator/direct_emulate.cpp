// Host emulation of the direct contraction kernel, for CPU tests only: its
// planner and the index arithmetic of contract_direct.h, block by block, with
// every offset checked against its tensor, every LDS place written exactly
// once per slice, and every read of a row that C keeps preceded by a write.
#include <math.h>
#include <stdio.h>
#include <string.h>

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

}  // namespace

extern "C" {

// C = alpha * A . B + beta * C in fp64.  Returns -1 where the planner refuses,
// else the number of index errors.  counts: how often each C element is
// written.  blockStride > 1 runs a sample of the blocks; A NULL: indexes only.
int64_t direct_emulate(const char* mA, const char* mB, const char* mC, const int64_t* ext256,
                       double alpha, double beta, const double* A, const double* B, double* C,
                       uint8_t* counts, int64_t blockStride, char* msg, size_t msglen) {
    using namespace hptt;
    constexpr int kBK = direct_slice(8), kSlotsP = kBM * kBK / kBlock, kSlotsQ = kBN * kBK / kBlock;
    DirectArgs g;
    const double *P = A, *Q = B;
    std::string mP = mA, mQ = mB;
    if (!plan_direct(mA, mB, mC, ext256, 8, &g)) {
        if (!plan_direct(mB, mA, mC, ext256, 8, &g)) return -1;
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
    std::vector<double> sum(kBM * kBN);
    for (int64_t blk = 0; blk < int64_t(g.numTiles); blk += blockStride) {
        const DirectTile d = direct_tile(g, xcd_group_map(uint32_t(blk), g.numTiles, 4));
        uint32_t rowP[kBM], rowC[kBM], colQ[kBN], colC[kBN];
        for (int r = 0; r < kBM; ++r) direct_row(g, d, r, rowP[r], rowC[r]);
        for (int c = 0; c < kBN; ++c) direct_column(g, d, c, colQ[c], colC[c]);
        std::fill(sum.begin(), sum.end(), 0.0);
        for (int kb = 0; kb < (g.k.total + kBK - 1) / kBK; ++kb) {
            uint32_t kP[kBK] = {0}, kQ[kBK] = {0};
            for (int j = 0; j < kBK; ++j)
                if (kb * kBK + j < g.k.total)
                    group_offsets(g.k, uint32_t(kb * kBK + j), kP[j], kQ[j]);
            std::fill(seenP.begin(), seenP.end(), 0);
            std::fill(seenQ.begin(), seenQ.end(), 0);
            auto stage = [&](bool p) {
                for (int s = 0; s < (p ? kSlotsP : kSlotsQ) * kBlock; ++s) {
                    const DirectSlot x = p ? direct_slot_p(g, s, kBK) : direct_slot_q(g, s, kBK);
                    const int pitch = p ? kPitchP : kPitchQ, rows = p ? kBM : kBN;
                    if (x.row < 0 || x.row >= rows || x.k < 0 || x.k >= kBK || x.at < 0 ||
                        x.at >= pitch) {
                        ck.fail("slot out of range", s, x.at);
                        continue;
                    }
                    const int64_t off = p ? int64_t(rowP[x.row]) + kP[x.k]
                                          : int64_t(colQ[x.row]) + kQ[x.k];
                    if (off % 8 || off >= (p ? nP : nQ) * 8) {
                        ck.fail(p ? "P offset out of range" : "Q offset out of range", off, blk);
                        continue;
                    }
                    const bool in = kb * kBK + x.k < g.k.total;
                    const double v = A && in ? (p ? P[(d.offP + off) / 8] : Q[(d.offQ + off) / 8]) : 0.0;
                    if ((p ? d.offP : d.offQ) + off >= (p ? nP : nQ) * 8)
                        ck.fail("batch offset out of range", off, blk);
                    (p ? ldsP : ldsQ)[x.k * pitch + x.at] = v;
                    if ((p ? seenP : seenQ)[x.k * pitch + x.at]++)
                        ck.fail("LDS place written twice", x.k, x.at);
                }
            };
            stage(true);
            stage(false);
            for (int k = 0; k < kBK; ++k)
                for (int r = 0; r < kBM; ++r) {
                    const int at = k * kPitchP + direct_rows_at(g, r & ~15) + (r & 15);
                    if (at >= kBK * kPitchP || !seenP[at]) ck.fail("P read before write", k, r);
                    for (int c = 0; A && c < kBN; ++c)
                        sum[r * kBN + c] += ldsP[at] * ldsQ[k * kPitchQ + c];
                }
        }
        for (int r = 0; r < kBM; ++r)
            for (int c = 0; c < kBN; ++c) {
                if (rowC[r] == kOutside || colC[c] == kOutside) continue;
                const int64_t at = (d.offC + int64_t(rowC[r]) + colC[c]) / 8;
                if (at < 0 || at >= nC) {
                    ck.fail("C offset out of range", at, blk);
                    continue;
                }
                if (counts) counts[at]++;
                if (A) C[at] = alpha * sum[r * kBN + c] + (beta != 0 ? beta * C[at] : 0.0);
            }
    }
    if (msg && msglen) snprintf(msg, msglen, "%s", ck.msg);
    return ck.errors;
}

}  // extern "C"
