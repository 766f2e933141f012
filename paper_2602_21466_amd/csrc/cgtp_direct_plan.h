// Plan of the direct contraction (host): the Clebsch-Gordan matrices of every
// block and the lists of items, stages and groups (cgtp_direct.h).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <map>
#include <utility>
#include <vector>

#include "cgtp_direct.h"
#include "cgtp_internal.h"

namespace cgtp {

template <typename T>
struct DirHost {
    std::vector<T> coef;
    std::vector<DirItem> items;
    std::vector<DirStage> stages;
    std::vector<DirGroup> groups;
    DirList lists[2] = {};   // long, short
};

// For fixed (la, lb, M) the coefficients of l3 are the eigenvector of
// J^2 = (Ja + Jb)^2 with eigenvalue l3 (l3 + 1) in the basis |ma, M - ma>, where
// J^2 is tridiagonal: diagonal la (la+1) + lb (lb+1) + 2 ma mb, off-diagonal
// sqrt((la - ma)(la + ma + 1)) sqrt((lb + mb)(lb - mb + 1)) between ma and ma + 1.
// The three-term recurrence is run from both ends, where it grows, and joined
// at the first maximum seen from the upper end, so neither run enters a region
// in which it would amplify rounding.  Signs: the coefficient at the largest
// ma (ma = la, or mb = -lb) is positive in the Condon-Shortley convention (it
// is a single positive term of the Racah sum).
// out[M][r n + k] = C^{l3 M}_{la ma, lb M-ma}, l3 = la + lb - r, ma = la - k,
// n = min(2 la + 1, la + lb - M + 1).
inline void dir_cg_block(int la, int lb, std::vector<std::vector<double>>& out) {
    out.assign((size_t)(la + lb + 1), {});
    std::vector<double> dg, of, up, dn;
    for (int M = 0; M <= la + lb; ++M) {
        const int n = std::min(2 * la + 1, la + lb - M + 1);
        auto& o = out[(size_t)M];
        o.assign((size_t)n * n, 0.0);
        dg.assign(n, 0.0);
        of.assign(n, 0.0);   // of[k]: between k and k + 1
        for (int k = 0; k < n; ++k) {
            const int ma = la - k, mb = M - ma;
            dg[k] = (double)(la * (la + 1) + lb * (lb + 1) + 2 * ma * mb);
            // ma -> ma - 1, mb -> mb + 1
            of[k] = std::sqrt((double)(la + ma) * (la - ma + 1) * (double)(lb - mb) * (lb + mb + 1));
        }
        up.assign(n, 0.0);
        dn.assign(n, 0.0);
        for (int r = 0; r < n; ++r) {
            const int l3 = la + lb - r;
            const double ev = (double)l3 * (l3 + 1);
            up[0] = 1.0;
            int join = n - 1;
            for (int k = 0; k + 1 < n; ++k) {
                up[k + 1] = ((ev - dg[k]) * up[k] - (k ? of[k - 1] * up[k - 1] : 0.0)) / of[k];
                if (std::fabs(up[k + 1]) < std::fabs(up[k])) {
                    join = k;
                    break;
                }
            }
            dn[n - 1] = 1.0;
            for (int k = n - 1; k > join; --k)
                dn[k - 1] = ((ev - dg[k]) * dn[k] - (k + 1 < n ? of[k] * dn[k + 1] : 0.0)) / of[k - 1];
            const double s = up[join] / dn[join];
            double norm = 0;
            for (int k = 0; k < n; ++k) {
                const double v = k <= join ? up[k] : s * dn[k];
                o[(size_t)r * n + k] = v;
                norm += v * v;
            }
            const double f = 1.0 / std::sqrt(norm);
            for (int k = 0; k < n; ++k) o[(size_t)r * n + k] *= f;
        }
    }
}

// First coefficient chunk of each (row group, first order) of the blocks la <= lb.
using DirFirst = std::map<std::pair<int, int>, std::vector<std::vector<int>>>;

// One list of groups: stages of up to max_len outputs per pair; a group takes
// blocks together up to group_len outputs, or with `split` is a single stage.
template <typename T>
void dir_list(int L, const DirFirst& first, int max_len, int group_len, bool split, DirHost<T>& h, DirList& list) {
    constexpr int P = dir_pairs<T>(), HM = dir_orders<T>();
    const int max_tile = sizeof(T) == 4 ? 6144 : 7680;   // elements: 24 KiB (fp32)
    struct Piece {   // one row group of one block, in output order
        int l1, l2, rg, off, len;
    };
    struct Cost {
        DirGroup g;
        int64_t cost;
    };
    std::vector<Cost> groups;
    const int nblk = (L + 1) * (L + 1);
    int off = 0, path = 0;
    std::vector<int> boff(nblk), bpath(nblk);
    for (int b = 0; b < nblk; ++b) {
        const int l1 = b / (L + 1), l2 = b % (L + 1);
        boff[b] = off;
        bpath[b] = path;
        off += (2 * l1 + 1) * (2 * l2 + 1);
        path += 2 * std::min(l1, l2) + 1;
    }
    size_t lds = 0;
    for (int b0 = 0; b0 < nblk;) {
        // blocks b0 .. b1-1 of the group
        DirGroup g{};
        int b1 = b0, outs = 0;
        g.l1a = g.l1b = b0 / (L + 1);
        g.l2a = g.l2b = b0 % (L + 1);
        while (b1 < nblk) {
            const int l1 = b1 / (L + 1), l2 = b1 % (L + 1);
            const int sz = (2 * l1 + 1) * (2 * l2 + 1);
            const int l1b = std::max(g.l1b, l1), l2a = std::min(g.l2a, l2), l2b = std::max(g.l2b, l2);
            const int rows = dir_tile_row<T>(l1b + 1, g.l1a) + dir_tile_row<T>(l2b + 1, l2a);
            if (b1 > b0 && (outs + sz > group_len || rows * dir_row<T>() > max_tile)) break;
            outs += sz;
            g.l1b = l1b;
            g.l2a = l2a;
            g.l2b = l2b;
            ++b1;
        }
        const int rows1 = dir_tile_row<T>(g.l1b + 1, g.l1a), rows2 = dir_tile_row<T>(g.l2b + 1, g.l2a);
        g.x2tile = rows1 * dir_row<T>();
        g.tile_len = ((rows1 + rows2) * dir_row<T>() + 3) & ~3;
        g.stage0 = (int)h.stages.size();
        std::vector<Piece> pieces;
        for (int b = b0; b < b1; ++b) {
            const int l1 = b / (L + 1), l2 = b % (L + 1), la = std::min(l1, l2), d = std::abs(l1 - l2);
            for (int rg = (2 * la + kDirRows) / kDirRows - 1; rg >= 0; --rg) {
                const int hi = l1 + l2 - kDirRows * rg, lo = std::max(d, hi - kDirRows + 1);
                pieces.push_back({l1, l2, rg, boff[b] + lo * lo - d * d, (hi + 1) * (hi + 1) - lo * lo});
            }
        }
        int64_t cost = 0;
        for (size_t i = 0; i < pieces.size();) {
            if (split) cost = 0;
            DirStage st{(int)h.items.size(), 0, pieces[i].off, 0};
            size_t j = i;
            for (; j < pieces.size() && (j == i || st.len + pieces[j].len <= max_len); ++j) {
                const Piece& q = pieces[j];
                st.len += q.len;
                const int la = std::min(q.l1, q.l2), lb = std::max(q.l1, q.l2), d = lb - la;
                const bool swap = q.l1 > q.l2;
                const int b = q.l1 * (L + 1) + q.l2, lt = q.l1 + q.l2 - kDirRows * q.rg;
                const int t1 = dir_tile_row<T>(q.l1, g.l1a) * dir_row<T>();
                const int t2 = g.x2tile + dir_tile_row<T>(q.l2, g.l2a) * dir_row<T>();
                const auto& f = first.at({la, lb})[(size_t)q.rg];
                for (int m0 = 0; m0 <= lt; m0 += HM) {
                    DirItem it{};
                    it.chunk0 = f[(size_t)(m0 / HM)];
                    it.nk = std::min(2 * la + 1, la + lb - m0 + 1);
                    it.xa = (swap ? t2 : t1) + 2 * la * dir_row<T>();
                    it.xb = (swap ? t1 : t2) + (lb + m0 - la) * dir_row<T>();
                    it.code = lt | d << 8 | m0 << 16 | (swap ? 1 << 24 : 0);
                    it.c = boff[b] - d * d - st.off;
                    it.path = bpath[b] - d;
                    h.items.push_back(it);
                    cost += it.nk + 6;
                }
            }
            st.nitems = (int)h.items.size() - st.item0;
            std::stable_sort(h.items.begin() + st.item0, h.items.end(),
                             [](const DirItem& x, const DirItem& y) { return x.nk > y.nk; });
            lds = std::max(lds, ((size_t)g.tile_len + (size_t)P * (st.len | 1)) * sizeof(T));
            h.stages.push_back(st);
            i = j;
            if (split || i == pieces.size()) {
                g.nstages = (int)h.stages.size() - g.stage0;
                groups.push_back({g, cost});
                g.stage0 += g.nstages;
            }
        }
        b0 = b1;
    }
    std::stable_sort(groups.begin(), groups.end(), [](const Cost& x, const Cost& y) { return x.cost > y.cost; });
    list = {(int)h.groups.size(), (int)groups.size(), (int)lds};
    for (const auto& c : groups) h.groups.push_back(c.g);
}

// Coefficients of block (la, lb), la <= lb, for the forward; first chunk of (row
// group, orders m0..).
template <typename T>
void dir_coefs(int la, int lb, const std::vector<std::vector<double>>& cg, DirHost<T>& h,
               std::vector<std::vector<int>>& f) {
    constexpr int KC = dir_kc<T>(), HM = dir_orders<T>();
    f.resize((size_t)(2 * la + 1 + kDirRows - 1) / kDirRows);
    for (int rg = 0; rg < (int)f.size(); ++rg) {
        const int lt = la + lb - kDirRows * rg;
        for (int m0 = 0; m0 <= lt; m0 += HM) {
            const int nk = std::min(2 * la + 1, la + lb - m0 + 1);
            const int nch = (nk + KC - 1) / KC;
            const size_t at = h.coef.size();
            f[(size_t)rg].push_back((int)(at / kDirChunk));
            h.coef.resize(at + (size_t)nch * kDirChunk, (T)0);
            for (int o = 0; o < HM && m0 + o <= lt; ++o) {
                const int n = std::min(2 * la + 1, la + lb - m0 - o + 1);
                const auto& a = cg[(size_t)(m0 + o)];
                for (int r = 0; r < kDirRows && kDirRows * rg + r < n; ++r)
                    for (int k = 0; k < n; ++k)
                        h.coef[at + (size_t)(k / KC) * kDirChunk + dir_coef_index<T>(k % KC, o, r)] =
                            (T)a[(size_t)(kDirRows * rg + r) * n + k];
            }
        }
    }
}

struct DgHost {
    std::vector<float> coef;
    std::vector<DgTask> tasks;
    std::vector<DgOut> outs;
    std::vector<DgPart> parts;
    std::vector<DgStage> stages;
    DgList lists[2] = {};   // long, short
};

using DgFirst = std::map<std::pair<int, int>, std::vector<int>>;   // (la, lb) -> first chunk of each task

// One list of stages; several blocks share a stage up to max_len outputs.
inline void dg_list(int L, const DgFirst& first, int max_len, DgHost& h, DgList& list) {
    const int max_lds_of[kDgClasses] = {52 * 1024, 52 * 1024, 79 * 1024};   // three, three, two work-groups per CU
    const int nblk = (L + 1) * (L + 1);
    std::vector<int> boff(nblk);
    for (int b = 0, off = 0; b < nblk; ++b) {
        boff[b] = off;
        off += (2 * (b / (L + 1)) + 1) * (2 * (b % (L + 1)) + 1);
    }
    // stages: consecutive blocks of one class while their LDS fits
    struct Cost {
        DgStage s;
        int64_t cost;
    };
    std::vector<Cost> by_class[kDgClasses];
    for (int b0 = 0; b0 < nblk;) {
        const int cls = dg_class(b0 / (L + 1), b0 % (L + 1)), G = dg_groups(cls), P = dg_pairs(G), RS = dg_row(G);
        const int max_lds = max_lds_of[cls];
        DgStage st{};
        st.off = boff[b0];
        st.l1a = st.l1b = b0 / (L + 1);
        st.l2a = st.l2b = b0 % (L + 1);
        int b1 = b0, acc_rows = 0, len = 0;
        auto tile = [&](int l1b, int l2a, int l2b) {
            return (dg_tile_row(l1b + 1, st.l1a) + dg_tile_row(l2b + 1, l2a)) * RS;
        };
        auto lds = [&](int tile_len, int n, int rows) {
            return 4 * (((tile_len + 3) & ~3) + P * dir_run<float>(n) + rows * RS + 4);
        };
        while (b1 < nblk) {
            const int l1 = b1 / (L + 1), l2 = b1 % (L + 1), la = std::min(l1, l2), lb = std::max(l1, l2);
            if (dg_class(l1, l2) != cls) break;
            const int nrg = (2 * la + 4) / 4, nt = (nrg + kDgRows - 1) / kDgRows;
            const int rows = 4 * nrg + nt * (2 * lb + 2);
            const int n = len + (2 * l1 + 1) * (2 * l2 + 1);
            const int l1b = std::max(st.l1b, l1), l2a = std::min(st.l2a, l2), l2b = std::max(st.l2b, l2);
            const int reads = (l1b + 1) * (l1b + 1) - st.l1a * st.l1a + (l2b + 1) * (l2b + 1) - l2a * l2a;
            if (b1 > b0 && (n > max_len || lds(tile(l1b, l2a, l2b), n, acc_rows + rows) > max_lds ||
                            reads > kDgMaxInputs))
                break;
            len = n;
            st.l1b = l1b;
            st.l2a = l2a;
            st.l2b = l2b;
            acc_rows += rows;
            ++b1;
        }
        st.x2tile = dg_tile_row(st.l1b + 1, st.l1a) * RS;
        st.tile_len = (tile(st.l1b, st.l2a, st.l2b) + 3) & ~3;
        // parts: one, or for a single large block as many as it takes to keep to the
        // LDS of the class (their steps start at whole chunks)
        st.part0 = (int)h.parts.size();
        int run = 0;
        if (b1 > b0 + 1) {
            h.parts.push_back({st.off, len, 0, 4 * L + 4});
            run = dir_run<float>(len);
        } else {
            const int l1 = st.l1a, l2 = st.l2a, lt = l1 + l2, d = std::abs(l1 - l2), n = lt - d + 1, KC = dg_kc(G);
            int np = 1, per = n;
            for (;; ++np) {
                per = ((n + np - 1) / np + KC - 1) / KC * KC;
                run = 0;
                for (int s0 = 0; s0 < n; s0 += per) {
                    const int hi = lt - s0, lo = std::max(d, hi - per + 1);
                    run = std::max(run, dir_run<float>((hi + 1) * (hi + 1) - lo * lo));
                }
                if (per <= KC || 4 * (st.tile_len + P * run + acc_rows * RS + 4) <= max_lds) break;
            }
            for (int s0 = 0; s0 < n; s0 += per) {
                const int hi = lt - s0, lo = std::max(d, hi - per + 1);
                h.parts.push_back({st.off + lo * lo - d * d, (hi + 1) * (hi + 1) - lo * lo, s0, s0 + hi - lo + 1});
            }
        }
        st.nparts = (int)h.parts.size() - st.part0;
        st.acc0 = st.tile_len + P * run;
        st.acc_len = (acc_rows * RS + 3) & ~3;
        list.lds_bytes[cls] = std::max(list.lds_bytes[cls], 4 * (st.acc0 + st.acc_len));
        st.task0 = (int)h.tasks.size();
        st.out0 = (int)h.outs.size();
        int64_t cost = 0;
        int acc = st.acc0;
        for (int b = b0; b < b1; ++b) {
            const int l1 = b / (L + 1), l2 = b % (L + 1), la = std::min(l1, l2), lb = std::max(l1, l2);
            const bool swap = l1 > l2;
            const int t1 = dg_tile_row(l1, st.l1a) * RS, t2 = st.x2tile + dg_tile_row(l2, st.l2a) * RS;
            const int nrg = (2 * la + 4) / 4, nt = (nrg + kDgRows - 1) / kDgRows;
            const int stride = (2 * lb + 2) * RS, accb = acc + 4 * nrg * RS;
            const int n1 = 2 * l1 + 1, n2 = 2 * l2 + 1;
            for (int e = 0; e < n1 + n2; ++e) {
                const bool first_in = e < n1;
                const int l = first_in ? l1 : l2, m = (first_in ? e : e - n1) - l;
                DgOut o{};
                if (first_in != swap) {   // the smaller degree's input (x1 if equal)
                    o.plus = acc + (l - m) * RS;
                    o.minus = acc + (l + m) * RS + P;
                    o.code = 1;
                } else {
                    o.plus = accb + (l + m) * RS;
                    o.minus = accb + (l - m) * RS + P;
                    o.code = nt | stride << 4;
                }
                o.code |= e << 20;
                o.ws = (int)bwd_block_off(L, l1, l2) | (n1 + n2) << 20;
                h.outs.push_back(o);
            }
            for (int t = 0; t < nt; ++t) {
                DgTask k{};
                const int k0 = 4 * kDgRows * t, rgs = std::min(kDgRows, nrg - kDgRows * t);
                k.chunk0 = first.at({la, lb})[(size_t)t];
                k.code = la | lb << 8 | k0 << 16 | rgs << 24 | (swap ? 1 << 28 : 0);
                k.xa = (swap ? t2 : t1) + (2 * la - k0) * RS;
                k.xb = swap ? t1 : t2;
                const int d = lb - la;
                k.goff = boff[b] - st.off - d * d;
                k.acca = acc + k0 * RS;
                k.accb = accb + t * stride;
                h.tasks.push_back(k);
                for (int m0 = 0; m0 <= la + lb; m0 += dg_orders(G)) {
                    const int nk = std::min(2 * la + 1, la + lb - m0 + 1);
                    if (nk > k0) cost += (int64_t)rgs * nk + 8;
                }
            }
            acc = accb + nt * stride;
        }
        st.ntasks = (int)h.tasks.size() - st.task0;
        st.nouts = (int)h.outs.size() - st.out0;
        std::stable_sort(h.tasks.begin() + st.task0, h.tasks.end(), [](const DgTask& x, const DgTask& y) {
            auto w = [](const DgTask& t) {   // rows x steps of the first orders, as a measure
                const int la = t.code & 255, lb = t.code >> 8 & 255;
                return ((t.code >> 24) & 15) * (2 * la + 1) * (la + lb + 1 - (t.code >> 16 & 255));
            };
            return w(x) > w(y);
        });
        by_class[cls].push_back({st, cost});
        b0 = b1;
    }
    list.stage0 = (int)h.stages.size();
    for (int c = 0; c < kDgClasses; ++c) {
        std::stable_sort(by_class[c].begin(), by_class[c].end(), [](const Cost& x, const Cost& y) { return x.cost > y.cost; });
        for (const auto& s : by_class[c]) h.stages.push_back(s.s);
        list.nstages[c] = (int)by_class[c].size();
    }
}

// The same for the gradients; first chunk of each task.
inline void dg_coefs(int la, int lb, const std::vector<std::vector<double>>& cg, DgHost& h, std::vector<int>& first) {
    const int G = dg_groups(dg_class(la, lb)), HM = dg_orders(G), KC = dg_kc(G);
    const int nrg = (2 * la + 1 + 3) / 4;
    for (int rg0 = 0; rg0 < nrg; rg0 += kDgRows) {
        const int rgs = std::min(kDgRows, nrg - rg0);
        first.push_back((int)(h.coef.size() / kDirChunk));
        for (int m0 = 0; m0 <= la + lb; m0 += HM) {
            const int nk = std::min(2 * la + 1, la + lb - m0 + 1);
            if (nk <= 4 * rg0) break;
            const int nch = (nk + KC - 1) / KC;
            const size_t at = h.coef.size();
            h.coef.resize(at + (size_t)nch * rgs * kDirChunk, 0.0f);
            for (int o = 0; o < HM && m0 + o <= la + lb; ++o) {
                const int n = std::min(2 * la + 1, la + lb - m0 - o + 1);
                const auto& a = cg[(size_t)(m0 + o)];
                for (int s = 0; s < n; ++s)
                    for (int r = 0; r < 4 * rgs && 4 * rg0 + r < n; ++r)
                        h.coef[at + ((size_t)(s / KC) * rgs + r / 4) * kDirChunk + dg_coef_index(G, s % KC, o, r % 4)] =
                            (float)a[(size_t)s * n + 4 * rg0 + r];
            }
        }
    }
}

// The coefficient table and the work lists of degree L, and with `g` the
// gradient kernel's.
template <typename T>
void dir_build(int L, DirHost<T>& h, DgHost* g = nullptr) {
    DirFirst first;
    DgFirst gfirst;
    std::vector<std::vector<double>> cg;
    for (int la = 0; la <= L; ++la)
        for (int lb = la; lb <= L; ++lb) {
            dir_cg_block(la, lb, cg);
            dir_coefs<T>(la, lb, cg, h, first[{la, lb}]);
            if (g) dg_coefs(la, lb, cg, *g, gfirst[{la, lb}]);
        }
    // long: a stage's run, per pair, takes up to 40 KiB (fp32) of LDS for the pairs
    // of a work-group, so that two work-groups share a CU, and at least the largest
    // block's four largest degrees, (2 L + 1)^2 - (2 L - 3)^2 outputs.  A group takes blocks together until one filling of
    // the input tiles serves about four stages' worth of outputs (two stages: 1147 us
    // instead of 1105 at L = 16, N = 8192; 164 instead of 155 in the real basis at
    // L = 11, N = 4001; one stage 1211 and 185)
    const int max_len = std::max(40 * 1024 / (dir_pairs<T>() * 4) - 1, 16 * L - 8);
    dir_list<T>(L, first, max_len, 4 * max_len, false, h, h.lists[0]);
    // short: single stages of 256 (fp64: 128) outputs where that many are more than
    // four degrees of a block (half as many: 12.0 instead of 9.4 us in the real basis
    // at L = 16, N = 16; twice as many: 11.0 instead of 7.8 in fp64 at L = 4, N = 100)
    const int short_len = 4096 / dir_pairs<T>();
    dir_list<T>(L, first, short_len, short_len, true, h, h.lists[1]);
    if (!g) return;
    g->coef.resize(g->coef.size() + (size_t)kDgRows * kDirChunk, 0.0f);   // read ahead of the last chunk
    dg_list(L, gfirst, INT32_MAX, *g, g->lists[0]);
    // (128 outputs: 16.5 instead of 14.3 us at L = 3, N = 100)
    dg_list(L, gfirst, 64, *g, g->lists[1]);
}

}  // namespace cgtp
