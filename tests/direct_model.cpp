// Host model of the direct contraction's work lists (csrc/cgtp_direct.h): runs
// every item of every group as the kernel does, with every index checked
// against its buffer, and compares the outputs with the plain double sum over
// the oracle's Racah-formula coefficients.
//   usage: direct_model fp32|fp64 L
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "cgtp_direct_plan.h"

extern "C" double oracle_cg(int j1, int m1, int j2, int m2, int j, int m);

using namespace cgtp;

static void need(bool ok, const char* what) {
    if (!ok) {
        std::printf("direct_model: %s\n", what);
        std::exit(1);
    }
}

template <typename T>
static double run(int L) {
    DirHost<T> h;
    dir_build<T>(L, h);
    constexpr int HM = dir_orders<T>(), KC = dir_kc<T>(), RS = dir_row<T>();
    const int nin = (L + 1) * (L + 1), nout = nin * nin;
    std::vector<double> x[2], out(nout, NAN);
    for (auto& r : x) {
        r.resize(nin);
        for (auto& v : r) v = drand48() - 0.5;
    }
    for (const auto& g : h.groups) {
        std::vector<double> tile[2];   // orders as given and reversed
        for (int s = 0; s < 2; ++s) {
            tile[s].assign((size_t)g.tile_len, 0.0);
            for (int in = 0; in < 2; ++in) {
                const int la = in ? g.l2a : g.l1a, lb = in ? g.l2b : g.l1b, base = in ? g.x2tile : 0;
                const int end = in ? g.tile_len : g.x2tile;
                for (int l = la; l <= lb; ++l)
                    for (int m = -l; m <= l; ++m) {
                        const int e = base + (dir_tile_row<T>(l, la) + l + m) * RS;
                        need(e >= base && e + RS - 1 <= end, "tile row outside its tile");
                        tile[s][(size_t)e] = x[in][(size_t)(l * l + l + (s ? -m : m))];
                    }
            }
        }
        for (int si = g.stage0; si < g.stage0 + g.nstages; ++si) {
            const DirStage& st = h.stages[(size_t)si];
            std::vector<double> buf((size_t)st.len, NAN);
            need(((size_t)g.tile_len + (size_t)dir_pairs<T>() * (st.len | 1)) * sizeof(T) <= (size_t)h.lds_bytes,
                 "stage larger than the LDS of the launch");
            for (int ii = st.item0; ii < st.item0 + st.nitems; ++ii) {
                const DirItem& it = h.items[(size_t)ii];
                const int lt = it.code & 255, lmin = it.code >> 8 & 255, m0 = it.code >> 16 & 255;
                const int swap = it.code >> 24;
                for (int s = 0; s < 2; ++s)
                    for (int o = 0; o < HM; ++o)
                        for (int r = 0; r < kDirRows; ++r) {
                            const int M = m0 + o, l3 = lt - r;
                            double acc = 0;
                            for (int k = 0; k < it.nk; ++k) {
                                const int ea = it.xa - k * RS, eb = it.xb + (k + o) * RS;
                                const size_t ci = (size_t)(it.chunk0 + k / KC) * kDirChunk +
                                                  (size_t)dir_coef_index<T>(k % KC, o, r);
                                need(ea >= 0 && ea < g.tile_len && eb >= 0 && eb < g.tile_len, "read past the tiles");
                                need(ci < h.coef.size(), "read past the coefficients");
                                acc += (double)h.coef[ci] * tile[s][(size_t)ea] * tile[s][(size_t)eb];
                            }
                            if (M > l3 || l3 < lmin || (s && !M)) continue;
                            const int q = it.c + l3 * l3 + l3 + (s ? -M : M);
                            need(q >= 0 && q < st.len, "write outside the stage");
                            need(std::isnan(buf[(size_t)q]), "output written twice");
                            buf[(size_t)q] = ((r & 1) && s != swap) ? -acc : acc;
                        }
            }
            for (int i = 0; i < st.len; ++i) {
                need(!std::isnan(buf[(size_t)i]), "output of a stage not written");
                need(std::isnan(out[(size_t)(st.off + i)]), "stages overlap");
                out[(size_t)(st.off + i)] = buf[(size_t)i];
            }
        }
    }
    double num = 0, den = 0;
    int off = 0;
    for (int l1 = 0; l1 <= L; ++l1)
        for (int l2 = 0; l2 <= L; ++l2)
            for (int l3 = std::abs(l1 - l2); l3 <= l1 + l2; ++l3)
                for (int m3 = -l3; m3 <= l3; ++m3, ++off) {
                    double a = 0;
                    for (int m1 = std::max(-l1, m3 - l2); m1 <= std::min(l1, m3 + l2); ++m1)
                        a += oracle_cg(l1, m1, l2, m3 - m1, l3, m3) * x[0][(size_t)(l1 * l1 + l1 + m1)] *
                             x[1][(size_t)(l2 * l2 + l2 + m3 - m1)];
                    num += (a - out[(size_t)off]) * (a - out[(size_t)off]);
                    den += a * a;
                }
    return std::sqrt(num / den);
}

// Largest error of the plan's coefficients against the oracle's.
static double coefficients(int L) {
    double worst = 0;
    std::vector<std::vector<double>> cg;
    for (int la = 0; la <= L; la += 4)
        for (int lb = la; lb <= L; lb += 3) {
            dir_cg_block(la, lb, cg);
            for (int M = 0; M <= la + lb; ++M) {
                const int n = std::min(2 * la + 1, la + lb - M + 1);
                for (int r = 0; r < n; ++r)
                    for (int k = 0; k < n; ++k)
                        worst = std::max(worst, std::fabs(cg[(size_t)M][(size_t)r * n + k] -
                                                          oracle_cg(la, la - k, lb, M - la + k, la + lb - r, M)));
            }
        }
    return worst;
}

int main(int argc, char** argv) {
    need(argc == 3, "usage: direct_model fp32|fp64|cg L");
    const int L = std::atoi(argv[2]);
    const double e = !std::strcmp(argv[1], "cg") ? coefficients(L) : !std::strcmp(argv[1], "fp64") ? run<double>(L) : run<float>(L);
    std::printf("%.17g\n", e);
    return 0;
}
