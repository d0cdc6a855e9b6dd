// Planner of the direct contraction kernel (contract_direct.h): host code
// only, no HIP call.
#include <string.h>

#include <algorithm>
#include <cmath>

#include "contract_direct.h"

namespace hptt {

namespace {

constexpr int64_t kLimit = int64_t(1) << 31;

int64_t stride_of(const std::string& modes, char m, const int64_t* ext) {
    int64_t s = 1;
    for (char c : modes) {
        if (c == m) return s;
        s *= ext[static_cast<unsigned char>(c)];
    }
    return 0;
}

bool has(const std::string& s, char c) { return s.find(c) != std::string::npos; }

int ceil_log2(int64_t v) {
    int l = 0;
    while ((int64_t(1) << l) < v) ++l;
    return l;
}

void set_group(ModeGroup& g, const std::string& modes, const std::string& t0,
               const std::string& t1, const int64_t* ext, int elem) {
    g.n = 0;
    int64_t total = 1;
    for (char c : modes) {
        const int64_t e = ext[static_cast<unsigned char>(c)];
        g.ext[g.n] = make_fastdiv(uint32_t(e));
        g.s0[g.n] = uint32_t(stride_of(t0, c, ext) * elem);
        g.s1[g.n] = uint32_t(stride_of(t1, c, ext) * elem);
        total *= e;
        ++g.n;
    }
    g.total = int32_t(total);
}

// Bytes of C that x1's positions fill from C's first one on: every run of rows
// in C starts at a multiple of it.
int64_t run_c(const DirectArgs& g, int elem) {
    int64_t run = elem;
    for (int j = 0; j < g.x1.n && int64_t(g.x1.s1[j]) == run; ++j) run *= g.x1.ext[j].d;
    return run;
}

}  // namespace

bool plan_direct(const std::string& modesP, const std::string& modesQ, const std::string& modesC,
                 const int64_t* ext, int elem, DirectArgs* g) {
    memset(g, 0, sizeof(*g));
    // extent-1 modes move nothing
    std::string P, Q, C;
    auto keep = [&](const std::string& from, std::string& to) {
        int64_t v = 1;
        for (char c : from) {
            const int64_t e = ext[static_cast<unsigned char>(c)];
            if (e > 1) to += c;
            v *= e;
            if (v * elem >= (int64_t(1) << 32) || v >= kLimit) return false;
        }
        return true;
    };
    if (!keep(modesP, P) || !keep(modesQ, Q) || !keep(modesC, C)) return false;
    if (C.empty() || !has(P, C[0]) || has(Q, C[0])) return false;
    std::string X, Y, K, L;
    for (char c : C) (has(P, c) ? (has(Q, c) ? L : X) : Y) += c;
    // the contracted modes in the order of the operand that starts with one
    const std::string& kFrom = !P.empty() && !has(C, P[0]) ? P : !Q.empty() && !has(C, Q[0]) ? Q : P;
    for (char c : kFrom)
        if (!has(C, c)) K += c;
    // Y in Q's order when Q starts with one of its modes (runs of Q), else C's
    if (!Q.empty() && has(Y, Q[0])) {
        Y.clear();
        for (char c : Q)
            if (has(C, c) && !has(P, c)) Y += c;
    }
    // x2: the X modes P starts with, until they make a run of 8 elements,
    // unless P starts with C's stride-1 mode (or with a contracted one)
    std::string x2;
    int64_t e2 = 1;
    size_t lead = 0;
    while (lead < P.size() && has(X, P[lead]) && P[lead] != C[0] && e2 < 8) {
        e2 *= ext[static_cast<unsigned char>(P[lead])];
        x2 += P[lead++];
    }
    std::string x1;
    for (char c : X)
        if (!has(x2, c)) x1 += c;
    set_group(g->x1, x1, P, C, ext, elem);
    set_group(g->x2, x2, P, C, ext, elem);
    set_group(g->y, Y, Q, C, ext, elem);
    set_group(g->k, K, P, Q, ext, elem);
    const int logM = ceil_log2(kBM), logN = ceil_log2(kBN), logK = ceil_log2(direct_slice(elem));
    // Up to 8 positions of x2 (MI355X, fp64 abcde = efbad.cf, runs of 8, 4 and 2
    // elements in P against runs of 16, 32 and 64 in C: 99, 113 and 132 us).
    g->t2log = ceil_log2(e2 < 8 ? e2 : 8);
    g->t1log = logM - g->t2log;
    if (!x2.empty()) {
        g->sh2 = 0;
        if (lead < P.size() && !has(C, P[lead])) {  // then a contracted mode
            g->shk = g->t2log;
            g->sh1 = g->t2log + logK;
        } else {
            g->sh1 = g->t2log;
            g->shk = logM;
        }
    } else if (!P.empty() && !has(C, P[0])) {  // P starts with a contracted mode
        g->shk = 0;
        g->sh1 = logK;
        g->sh2 = logK + g->t1log;
    } else {
        g->sh1 = 0;
        g->sh2 = g->t1log;
        g->shk = logM;
    }
    if (!Q.empty() && !has(C, Q[0])) {
        g->shq = 0;
        g->shn = logK;
    } else {
        g->shn = 0;
        g->shq = logN;
    }
    const int64_t t1 = int64_t(1) << g->t1log, t2 = int64_t(1) << g->t2log;
    const int64_t ny = (g->y.total + kBN - 1) / kBN, n2 = (g->x2.total + t2 - 1) / t2,
                  n1 = (g->x1.total + t1 - 1) / t1;
    g->tilesY = make_fastdiv(uint32_t(ny));
    g->tiles2 = make_fastdiv(uint32_t(n2));
    g->tiles1 = make_fastdiv(uint32_t(n1));
    int64_t tiles = ny * n2 * n1;
    for (char c : L) {
        const int64_t e = ext[static_cast<unsigned char>(c)];
        g->eL[g->nL] = make_fastdiv(uint32_t(e));
        g->sLP[g->nL] = stride_of(P, c, ext) * elem;
        g->sLQ[g->nL] = stride_of(Q, c, ext) * elem;
        g->sLC[g->nL] = stride_of(C, c, ext) * elem;
        ++g->nL;
        tiles *= e;
    }
    if (tiles >= (int64_t(1) << 32) / kBlock) return false;  // a launch counts threads in 32 bits
    g->numTiles = uint32_t(tiles);
    // Non-temporal stores of C where it will not stay in the 256 MiB last-level
    // cache anyway, sooner where its 16-element runs are written by distant
    // blocks -- in fp64, whose stores are whole lines where C's runs are
    // (MI355X, 70 contractions of 64 MiB of C and more: 1.03x on average, 0.90 to
    // 1.11; abcde = efbad.cf 91.8 -> 87.9 us).  A line written in parts that way
    // goes to memory in parts: runs off the lines lose up to 4x (fp32
    // adgihcb = eihgfab.egfchid 127 us, 529 non-temporal), and so does fp32,
    // whose stores are half lines (0.83 to 1.07x on whole-line runs).
    int64_t bytesC = elem;
    for (char c : C) bytesC *= ext[static_cast<unsigned char>(c)];
    g->streamC = elem == 8 && run_c(*g, elem) % 128 == 0 &&
                 bytesC >= ((x2.empty() ? 128 : 64) << 20);
    return true;
}

namespace {

// Two overlapping costs: the larger, and a part of the smaller.
double overlap(double a, double b, double part) { return a > b ? a + part * b : b + part * a; }

double batches(const DirectArgs& g) {
    double v = 1;
    for (int j = 0; j < g.nL; ++j) v *= double(g.eL[j].d);
    return v;
}

// Bytes of P, Q and C.
void tensor_bytes(const DirectArgs& g, int elem, double* P, double* Q, double* C) {
    const double m = double(g.x1.total) * double(g.x2.total), n = g.y.total, k = g.k.total;
    *P = m * k * batches(g) * elem;
    *Q = n * k * batches(g) * elem;
    *C = m * n * batches(g) * elem;
}

// How many times over the 64 bytes around an element of an operand are read:
// a block reads one batch index, so where a batch mode lies within those 64
// bytes the rest of them is another block's.
double spread(const DirectArgs& g, const int64_t* strides) {
    double s = 1;
    for (int j = 0; j < g.nL; ++j)
        if (strides[j] < 64) s = std::max(s, 64.0 / double(strides[j]));
    return s;
}

}  // namespace

// The constants are fitted to 5,789 random contractions on MI355X and, for what
// large operands read again, 1,920 more (fp64 and fp32, 3,228 with batch modes,
// 2,576 with beta = 1; tensors to 300 MB, most read from memory), each timed both
// ways: the logarithms of both estimates are within 0.18 (one standard
// deviation) of the measured ones.  With the margin that use_direct asks for the
// calls take 0.714 of transposition - GEMM - transposition on average and 1.010 of
// the faster of the two; 103 of the 7,709 are more than 3 % slower than that path,
// 57 more than 10 %, the worst 1.62x.  With estimates that knew of neither the batch
// modes' spread, nor the read of C, nor the GEMM's padding, and no margin, it was
// 0.718 and 1.016; 199, 138 and up to 4.4x.
double direct_us(const DirectArgs& g, int elem, bool beta) {
    const bool f64 = elem == 8;
    double P, Q, C;
    tensor_bytes(g, elem, &P, &Q, &C);
    // runs of C below 64 bytes write parts of its lines, at a greater cost where
    // the lines have been read before
    const double parts = std::min(4.0, std::max(1.0, 64.0 / double(run_c(g, elem)))) - 1;
    const double out =
        beta ? C * (2.5 + parts) : C + parts * (0.4 * C + 0.2 * std::max(0.0, C - 30e6));
    const int bk = direct_slice(elem);
    const double slices = (g.k.total + bk - 1) / bk;
    const double rows = double(g.tiles1.d) * g.tiles2.d * kBM;
    const double cols = (g.y.total + 15) / 16 * 16.0;  // products of 16 columns are left out
    const double flops = 2.0 * rows * cols * slices * bk * batches(g);
    // what is read again: the operands by other blocks, and the other parts of
    // lines that hold several batches, the more of these the larger the tensor
    const double ny = g.tilesY.d, nx = double(g.tiles1.d) * g.tiles2.d;
    auto again = [](double bytes, double parts, double times) {
        return (parts - 1) * (0.21 + bytes / 200e6) * bytes * std::pow(times, 0.6) +
               0.25 * bytes * (times - 1);
    };
    const double moved = P + again(P, spread(g, g.sLP), ny) + Q + again(Q, spread(g, g.sLQ), nx);
    const double stream = overlap(flops / (f64 ? 86e6 : 143e6), (moved + out) / 4.85e6, 0.84);
    // a block's slices follow each other; about 1024 blocks run at one time
    const double rounds = (g.numTiles + 1023) / 1024;
    const double chain = rounds * (slices * (f64 ? 1.0 : 1.2) + (beta ? 2.0 : 0.0) + 0.84);
    return 3.8 + overlap(stream, chain, 0.84);
}

// The GEMM works on padded tiles, several rounds of them where it has many
// batches, and a long contraction is a chain for it too.
double transposed_us(double m, double n, double k, double batch, int elem, int transposes,
                     double bytesMoved, bool readC) {
    const bool f64 = elem == 8;
    const double tiles = std::ceil(m / 64) * std::ceil(n / 32) * batch;
    const double flops = 2.0 * tiles * 64 * 32 * k;
    const double bytes = (m * k + n * k + m * n * (readC ? 2 : 1)) * batch * elem;
    const double gemm = overlap(overlap(flops / (f64 ? 98e6 : 110e6), bytes / 8.5e6, 1.1),
                                std::min(k, 700.0) * (f64 ? 0.029 : 0.0063), 1.1);
    return 6.6 + 3.0 * transposes + bytesMoved / 5.7e6 + gemm + 0.7 * std::ceil(tiles / 256);
}

}  // namespace hptt
