// Host model of the direct contraction's work lists (csrc/cgtp_direct.h): runs
// every item of every group as the kernel does, with every index checked
// against its buffer, and compares the outputs with the plain double sum over
// the oracle's Racah-formula coefficients.
//   usage: direct_model fp32|fp64|backward|cg|launches L
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
static double run(int L, const DirHost<T>& h, const DirList& list) {
    constexpr int HM = dir_orders<T>(), KC = dir_kc<T>(), RS = dir_row<T>();
    const int nin = (L + 1) * (L + 1), nout = nin * nin;
    need(list.lds_bytes <= kLdsBudget, "more LDS than a CU has");
    std::vector<double> x[2], out(nout, NAN);
    for (auto& r : x) {
        r.resize(nin);
        for (auto& v : r) v = drand48() - 0.5;
    }
    for (int gi = list.group0; gi < list.group0 + list.ngroups; ++gi) {
        const DirGroup& g = h.groups[(size_t)gi];
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
            need(((size_t)g.tile_len + (size_t)dir_pairs<T>() * (st.len | 1)) * sizeof(T) <= (size_t)list.lds_bytes,
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

// Both lists of the plan; the outputs of one seed are the same to the last bit.
template <typename T>
static double forward(int L) {
    DirHost<T> h;
    dir_build<T>(L, h);
    srand48(1);
    const double e = run<T>(L, h, h.lists[0]);
    srand48(1);
    need(run<T>(L, h, h.lists[1]) == e, "the lists differ");
    return e;
}

// The gradient kernel's lists (fp32), run task by task in the same way.
static double backward(int L, const DgHost& h, const DgList& list) {
    const int nin = (L + 1) * (L + 1), nout = nin * nin;
    std::vector<double> x[2], grad[2], ref[2], g(nout);
    for (int i = 0; i < 2; ++i) {
        x[i].resize(nin);
        grad[i].assign(nin, 0.0);
        ref[i].assign(nin, 0.0);
        for (auto& v : x[i]) v = drand48() - 0.5;
    }
    for (auto& v : g) v = drand48() - 0.5;
    int si = list.stage0, covered = 0;
    for (int cls = 0; cls < kDgClasses; ++cls)
        for (int i = 0; i < list.nstages[cls]; ++i, ++si) {
            const DgStage& st = h.stages[(size_t)si];
            const int G = dg_groups(cls), P = dg_pairs(G), RS = dg_row(G), HM = dg_orders(G), KC = dg_kc(G);
            need(list.lds_bytes[cls] <= kLdsBudget, "more LDS than a CU has");
            need(4 * (st.acc0 + st.acc_len) <= list.lds_bytes[cls] && st.acc0 % 4 == 0 && st.acc_len % 4 == 0,
                 "stage larger than the LDS of the launch");
            need((st.l1b + 1) * (st.l1b + 1) - st.l1a * st.l1a + (st.l2b + 1) * (st.l2b + 1) - st.l2a * st.l2a <= kDgMaxInputs,
                 "more inputs than the threads of a pair hold");
            std::vector<double> tile[2];
            for (int s = 0; s < 2; ++s) {
                tile[s].assign((size_t)st.tile_len, 0.0);
                for (int in = 0; in < 2; ++in)
                    for (int l = in ? st.l2a : st.l1a; l <= (in ? st.l2b : st.l1b); ++l)
                        for (int m = -l; m <= l; ++m) {
                            const int e = (in ? st.x2tile : 0) + (dg_tile_row(l, in ? st.l2a : st.l1a) + l + m) * RS;
                            need(e >= 0 && e + RS - 1 <= (in ? st.tile_len : st.x2tile), "tile row outside its tile");
                            tile[s][(size_t)e] = x[in][(size_t)(l * l + l + (s ? -m : m))];
                        }
            }
            std::vector<double> sums[2];   // by sign of the order; element / (2 P) is the row
            for (auto& v : sums) v.assign((size_t)st.acc_len, 0.0);
            auto at = [&](int s, int e) -> double& {
                need(e >= st.acc0 && e + P <= st.acc0 + st.acc_len, "sum outside the sums");
                return sums[s][(size_t)(e - st.acc0)];
            };
            for (int pi = st.part0; pi < st.part0 + st.nparts; ++pi) {
                const DgPart& part = h.parts[(size_t)pi];
                need(st.tile_len + P * dir_run<float>(part.len) <= st.acc0, "run overlaps the sums");
                need(part.s0 % KC == 0, "a part starts inside a chunk");
                covered += part.len;
                for (int ti = st.task0; ti < st.task0 + st.ntasks; ++ti) {
                    const DgTask& t = h.tasks[(size_t)ti];
                    const int la = t.code & 255, lb = t.code >> 8 & 255, k0 = t.code >> 16 & 255, rgs = t.code >> 24 & 15;
                    const int swap = t.code >> 28 & 1, lt = la + lb;
                    size_t ck = (size_t)t.chunk0;
                    for (int m0 = 0; m0 <= lt; m0 += HM) {
                        const int nk = std::min(2 * la + 1, lt - m0 + 1), s1 = std::min(nk, part.s1);
                        if (nk <= k0 || nk <= part.s0) break;
                        for (int s = 0; s < 2; ++s)
                            for (int o = 0; o < HM; ++o)
                                for (int r = 0; r < 4 * rgs; ++r) {
                                    double T = 0;
                                    for (int k = part.s0; k < s1; ++k) {
                                        const size_t ci = (ck + (size_t)(k / KC) * rgs + r / 4) * kDirChunk +
                                                          (size_t)dg_coef_index(G, k % KC, o, r % 4);
                                        need(ci < h.coef.size(), "read past the coefficients");
                                        const int l3 = lt - k, M = m0 + o;
                                        if (M > l3 || (s && !M)) continue;
                                        const int q = t.goff + l3 * (l3 + 1) + (s ? -M : M) - (part.off - st.off);
                                        need(q >= 0 && q < part.len, "gradient read outside the run");
                                        T += ((k & 1) && s != swap ? -1.0 : 1.0) * (double)h.coef[ci] *
                                             g[(size_t)(part.off + q)];
                                    }
                                    const int d = std::min(lb - la + k0 + m0 + o + r, 2 * lb + 1);
                                    const int ea = t.xa - r * RS, eb = t.xb + d * RS;
                                    need(ea >= 0 && ea + 2 * P <= st.tile_len && eb >= 0 && eb + 2 * P <= st.tile_len,
                                         "read past the tiles");
                                    if (m0 + o > lt) need(T == 0, "order past the block");
                                    at(s, t.acca + r * RS + s * P) += T * tile[s][(size_t)eb];
                                    at(s, t.accb + d * RS + s * P) += T * tile[s][(size_t)ea];
                                }
                        ck += (size_t)((nk + KC - 1) / KC * rgs);
                        need((ck + (size_t)rgs) * kDirChunk <= h.coef.size(), "read ahead past the coefficients");
                    }
                }
            }
            for (int oi = st.out0; oi < st.out0 + st.nouts; ++oi) {
                const DgOut& o = h.outs[(size_t)oi];
                const int nt = o.code & 15, stride = o.code >> 4 & 0xffff, e = o.code >> 20, nrow = o.ws >> 20;
                double v = 0;
                for (int t = 0; t < nt; ++t) v += at(0, o.plus + t * stride) + at(1, o.minus + t * stride);
                // the block from its place in the workspace
                int l1 = 0, l2 = 0;
                while ((int)bwd_block_off(L, l1, l2) != (o.ws & 0xfffff))
                    if (++l2 > L) l2 = 0, need(++l1 <= L, "no such block");
                need(nrow == 2 * (l1 + l2 + 1) && e < nrow, "wrong component");
                if (e < 2 * l1 + 1)
                    grad[0][(size_t)(l1 * l1 + e)] += v;
                else
                    grad[1][(size_t)(l2 * l2 + e - (2 * l1 + 1))] += v;
            }
        }
    need(covered == nout, "stages do not cover the outputs");
    int off = 0;
    for (int l1 = 0; l1 <= L; ++l1)
        for (int l2 = 0; l2 <= L; ++l2)
            for (int l3 = std::abs(l1 - l2); l3 <= l1 + l2; ++l3)
                for (int m3 = -l3; m3 <= l3; ++m3, ++off)
                    for (int m1 = std::max(-l1, m3 - l2); m1 <= std::min(l1, m3 + l2); ++m1) {
                        const double c = oracle_cg(l1, m1, l2, m3 - m1, l3, m3) * g[(size_t)off];
                        const size_t i1 = (size_t)(l1 * l1 + l1 + m1), i2 = (size_t)(l2 * l2 + l2 + m3 - m1);
                        ref[0][i1] += c * x[1][i2];
                        ref[1][i2] += c * x[0][i1];
                    }
    double num = 0, den = 0;
    for (int in = 0; in < 2; ++in)
        for (int i = 0; i < nin; ++i) {
            num += (grad[in][(size_t)i] - ref[in][(size_t)i]) * (grad[in][(size_t)i] - ref[in][(size_t)i]);
            den += ref[in][(size_t)i] * ref[in][(size_t)i];
        }
    return std::sqrt(num / den);
}

static double gradients(int L) {
    DirHost<float> f;
    DgHost h;
    dir_build<float>(L, f, &h);
    srand48(1);
    const double a = backward(L, h, h.lists[0]);
    srand48(1);
    return std::max(a, backward(L, h, h.lists[1]));
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

// Launches of a call of about 2^L work-groups: below 2^32 work-items each, whole
// rounds, every work-group once.  Returns how many there are.
static double launches(int L) {
    int n = 0;
    for (int64_t total : {((int64_t)1 << L) - 1, (int64_t)1 << L, ((int64_t)1 << L) + 5})
        for (int threads : {256, 512})
            for (int64_t per : {8, 64, 512}) {
                int64_t next = 0;
                n = 0;
                const int err = dir_launches(total, per, threads, [&](int64_t first, unsigned grid) {
                    need(first == next && first % per == 0 && grid > 0 && grid % per == 0, "not whole rounds in order");
                    need((uint64_t)grid * (uint64_t)threads < ((uint64_t)1 << 32), "too many work-items in a launch");
                    next = first + grid;
                    ++n;
                    return 0;
                });
                need(err == 0 && next >= total && next < total + per, "work-groups left out");
                need(dir_launches(total, per, threads, [&](int64_t, unsigned) { return 7; }) == 7, "a failure is lost");
            }
    return n;
}

int main(int argc, char** argv) {
    need(argc == 3, "usage: direct_model fp32|fp64|backward|cg|launches L");
    const int L = std::atoi(argv[2]);
    const bool fp64 = !std::strcmp(argv[1], "fp64"), bwd = !std::strcmp(argv[1], "backward");
    if (!std::strcmp(argv[1], "launches")) return std::printf("%.17g\n", launches(L)), 0;
    const double e = !std::strcmp(argv[1], "cg") ? coefficients(L) : bwd ? gradients(L) : fp64 ? forward<double>(L) : forward<float>(L);
    std::printf("%.17g\n", e);
    return 0;
}
