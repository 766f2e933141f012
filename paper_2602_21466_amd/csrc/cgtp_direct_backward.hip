// Gradients of the CGTP by the direct contraction, transposed (cgtp_direct.h
// has the scheme and the work lists), fp32.
//
// Per stage and tile of pairs: the input tiles and the stage's runs of the
// upstream gradient go to LDS; each wave takes its tasks through all orders
// (per k step four LDS reads feed 4 x (row groups) MFMAs); the sums of a block
// are then put together over its tasks and order signs and written to the
// workspace, which launch_backward_sums adds up over the other degree.
//
// Bound by the phases of a work-group, which follow one another and which two
// or three work-groups per CU overlap only in part: of 2692 us at L = 16, 8192
// pairs (an earlier version), 1469 were left without the tasks, 1998 without the
// loads of the gradient, 768 without both; the sums take 135.  Measured (us,
// sphere-grid kernels before / now): L = 16, 4000 pairs 16150 / 1055; L = 32, 226
// pairs 11889 / 1115.  grad_b by LDS float atomics 4107 at L = 16, 8192 pairs, by
// ordered plain reads and writes 2707.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "cgtp_direct.h"
#include "cgtp_internal.h"
#include "device_common.h"

namespace cgtp {
namespace {

using namespace ::cgtp::dev;

struct DgArgs {
    const float* __restrict__ coef;
    const DgTask* __restrict__ tasks;
    const DgOut* __restrict__ outs;
    const DgPart* __restrict__ parts;
    const DgStage* __restrict__ stages;
    const float* __restrict__ x1;
    const float* __restrict__ x2;
    const float* __restrict__ g;
    float* __restrict__ ws;
    int64_t N;
    // the classes of one launch
    int32_t ncls;
    int32_t G[2], stage0[2];
    int64_t nunits[2];       // stages x tiles of pairs
    int64_t wg0[3];          // first work-group of each class, counted from the launch's first
    int32_t chunk[2];        // consecutive units given to one XCD
    int32_t L;
};

template <int G, int J> __device__ __forceinline__ f32x4 dg_mfma(float a, float b, f32x4 c) {
    // the coefficients of step J, four rows, broadcast to the columns of each group of orders
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, G == 2 ? 3 : 2, J, 0);
}

// Steps J .. of one chunk.  MASK: some orders may exceed the degree, or the
// block ends within the chunk (`left` steps; the others read its last degree
// and count nothing).
template <int G, int RG, int J, bool MASK>
__device__ __forceinline__ void dg_steps(const f32x4 (&a)[RG], const float* const (&gp)[4], int l3, int left, int mlane,
                                         float f_odd, f32x4 (&acc)[RG][4]) {
    constexpr int KC = dg_kc(G);
    if constexpr (J < KC) {
        if (MASK && J == 4 && left <= 4) return;
        const int l = MASK ? max(l3 - J, l3 - left + 1) : l3 - J, ro = l * (l + 1);
        const int lim = MASK && J >= left ? -1 : l;
        float b[4];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
            b[mi] = gp[mi][ro];
            if (MASK) b[mi] = mlane + mi <= lim ? b[mi] : 0.0f;
            if (J & 1) b[mi] *= f_odd;
        }
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) acc[r][mi] = dg_mfma<G, J>(a[r][mi], b[mi], acc[r][mi]);
        if (J & 1) __builtin_amdgcn_sched_barrier(0);   // keeps the loads of later steps from holding registers
        dg_steps<G, RG, J + 1, MASK>(a, gp, l3, left, mlane, f_odd, acc);
    }
}

template <int G, int RG>
__device__ __forceinline__ void dg_task(const DgTask& t, const DgPart& part, const float* __restrict__ coef, float* smem,
                                        const float* run, int lane) {
    constexpr int P = dg_pairs(G), KC = dg_kc(G), RS = dg_row(G), HM = dg_orders(G), NR = 4 * RG;
    static_assert(KC % 2 == 0, "a chunk starts at an even step");
    const int col = lane & (2 * P - 1), gm = 4 * (lane / (2 * P));
    const bool neg = col >= P;
    const int la = t.code & 255, lb = (t.code >> 8) & 255, k0 = (t.code >> 16) & 255;
    const bool swap = (t.code >> 28) & 1;
    const float f_odd = neg != swap ? -1.0f : 1.0f;
    const int lt = la + lb, sg = neg ? -1 : 1;
    float ga[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) ga[i] = 0.0f;
    const float* xa = smem + t.xa + col;   // row i at -i RS
    const float* cf0 = coef + (size_t)t.chunk0 * kDirChunk + 4 * lane;
    float* accb = smem + t.accb + col;
    for (int m0 = 0; m0 <= lt; m0 += HM) {
        const int nk = min(2 * la + 1, lt - m0 + 1);
        if (nk <= k0 || nk <= part.s0) break;   // (nk falls with m0)
        const int s1 = min(nk, part.s1);        // the part's steps
        const float* cf = cf0 + (size_t)(part.s0 / KC) * RG * kDirChunk;
        cf0 += (size_t)((nk + KC - 1) / KC) * RG * kDirChunk;
        f32x4 acc[RG][4];
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) acc[r][mi] = f32x4(0);
        const float* gp[4];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) gp[mi] = run + t.goff + sg * (m0 + gm + mi);
        // chunks in which every order of the item has its degrees, then the others; the
        // next chunk's coefficients are loaded a chunk ahead (the table ends in spare ones)
        const int nfull = part.s0 + max(min(s1, lt - (m0 + HM - 1) + 1) - part.s0, 0) / KC * KC;
        f32x4 a[RG], an[RG];
#pragma unroll
        for (int r = 0; r < RG; ++r) a[r] = *reinterpret_cast<const f32x4*>(cf + r * kDirChunk);
        int s = part.s0;
        for (; s < nfull; s += KC) {
            cf += RG * kDirChunk;
#pragma unroll
            for (int r = 0; r < RG; ++r) an[r] = *reinterpret_cast<const f32x4*>(cf + r * kDirChunk);
            dg_steps<G, RG, 0, false>(a, gp, lt - s, KC, 0, f_odd, acc);
#pragma unroll
            for (int r = 0; r < RG; ++r) a[r] = an[r];
        }
        for (; s < s1; s += KC) {
            cf += RG * kDirChunk;
#pragma unroll
            for (int r = 0; r < RG; ++r) an[r] = *reinterpret_cast<const f32x4*>(cf + r * kDirChunk);
            dg_steps<G, RG, 0, true>(a, gp, lt - s, s1 - s, m0 + gm, f_odd, acc);
#pragma unroll
            for (int r = 0; r < RG; ++r) a[r] = an[r];
        }
        if (m0 == 0 && neg && gm == 0) {   // order 0 counts once
#pragma unroll
            for (int r = 0; r < RG; ++r) acc[r][0] = f32x4(0);
        }
        // ---- T[k0 + i][m0 + gm + mi] = acc[i / 4][mi][i % 4]: both gradients
        const float* xb = smem + t.xb + col;
        const int d0 = lb - la + k0 + m0 + gm;   // row lb + mb of i = mi = 0
        // grad_b is added to four rows at a time: within four, the groups of orders
        // add to different rows (except past the degree, in the spare one), and a
        // wave's LDS accesses are in order.  (Plain reads and writes: an LDS float
        // atomic takes about as long as ten of them.)
#pragma unroll
        for (int i0 = 0; i0 < NR + 3; i0 += 4) {
            float v[4], *dst[4];
#pragma unroll
            for (int u = 0; u < 4 && i0 + u < NR + 3; ++u) {
                const int i = i0 + u;
                const int d = min(d0 + i, 2 * lb + 1);   // (past the degree: the zero and spare row)
                const float xbv = xb[d * RS];
                dst[u] = accb + d * RS;
                v[u] = *dst[u];
#pragma unroll
                for (int mi = 0; mi < 4; ++mi) {
                    const int k = i - mi;
                    if (k < 0 || k >= NR) continue;
                    const float tv = acc[k >> 2][mi][k & 3];
                    ga[k] = fmaf(tv, xbv, ga[k]);
                    v[u] = fmaf(tv, xa[-k * RS], v[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4 && i0 + u < NR + 3; ++u) *dst[u] = v[u];
            asm volatile("" ::: "memory");   // the next four rows are read after these are written
        }
    }
    // grad_a: summed over the groups of orders (and the parts)
#pragma unroll
    for (int i = 0; i < NR; ++i) {
#pragma unroll
        for (int o = 2 * P; o < 64; o *= 2) ga[i] += __shfl_xor(ga[i], o);
        if (gm == 0) smem[t.acca + i * RS + col] += ga[i];
    }
}

template <int G>
__device__ __forceinline__ void dg_stage(const DgArgs& ar, const DgStage& st, int64_t p0, float* smem) {
    constexpr int P = dg_pairs(G), RS = dg_row(G);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int np = (int)(ar.N - p0 < P ? ar.N - p0 : P);
    const int nin = (ar.L + 1) * (ar.L + 1);
    const int64_t nout = (int64_t)nin * nin;
    float* run = smem + st.tile_len;
    constexpr int TP = kDgThreads / P;   // threads per pair that load its inputs and runs
    const int xp = tid / TP, xi = tid & (TP - 1);
    // the run of a part, 16 bytes at a time, eight loads in flight per thread: it starts
    // as far from a 16-byte boundary in LDS as in memory.  (Threads of its own for each
    // pair; with the waves taking the pairs in turn L = 4, 16 pairs took 15.8 us instead
    // of 14.3, L = 16, 4000 pairs 1207 instead of 1055; four loads in flight 1091.)
    constexpr int kLoads = 8;
    auto load_run = [&](const DgPart& part, int ps) {
        const int64_t o = (p0 + xp) * nout + part.off;
        const int sh = (int)(o & 3), end = xp < np ? sh + part.len : 0;
        const float* src = ar.g + (o - sh);
        float* dst = run + xp * ps;
        const int full = end & ~3, e = full + xi;   // (the last elements one by one)
        const float last = e < end ? src[e] : 0.0f;
        for (int i0 = 4 * xi; i0 < full; i0 += 4 * kLoads * TP) {
            f32x4 v[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int i = i0 + 4 * TP * u;
                if (i < full) v[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + i));
            }
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int i = i0 + 4 * TP * u;
                if (i < full) *reinterpret_cast<f32x4*>(dst + i) = v[u];
            }
        }
        if (e < end) dst[e] = last;
    };
    // ---- input tiles (all of a thread's loads in flight), zero rows around the
    // degrees, cleared sums
    {
        constexpr int kX = (kDgMaxInputs + TP - 1) / TP;
        const int e1 = (st.l1b + 1) * (st.l1b + 1) - st.l1a * st.l1a, e2 = (st.l2b + 1) * (st.l2b + 1) - st.l2a * st.l2a;
        const int64_t row = p0 + xp < ar.N ? p0 + xp : ar.N - 1;   // (columns past N are not written out)
        const float* r1 = ar.x1 + row * nin + st.l1a * st.l1a;
        const float* r2 = ar.x2 + row * nin + st.l2a * st.l2a - e1;
        float xv[kX];
#pragma unroll
        for (int u = 0; u < kX; ++u) {
            const int i = xi + u * TP;
            if (i < e1 + e2) xv[u] = (i < e1 ? r1 : r2)[i];
        }
        for (int e = st.acc0 + tid * 4; e < st.acc0 + st.acc_len; e += kDgThreads * 4)
            *reinterpret_cast<f32x4*>(smem + e) = f32x4(0);
        for (int s = 0; s < 2; ++s) {
            const int la = s ? st.l2a : st.l1a, lb = s ? st.l2b : st.l1b;
            float* t0 = smem + (s ? st.x2tile : 0);
            for (int l = la; l <= lb + 1; ++l)   // the rows before degree l
                for (int e = tid; e < kDgPad * RS; e += kDgThreads) t0[(dg_tile_row(l, la) - kDgPad) * RS + e] = 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kX; ++u) {
            const int i = xi + u * TP;
            if (i >= e1 + e2) break;
            const int l0 = i < e1 ? st.l1a : st.l2a, ci = i < e1 ? i + l0 * l0 : i - e1 + l0 * l0;
            const int l = (int)__builtin_sqrtf((float)ci + 0.5f);   // exact for ci < 2^20
            const int m = ci - l * l - l;
            float* t0 = smem + (i < e1 ? 0 : st.x2tile) + (dg_tile_row(l, l0) + l) * RS + xp;   // order 0
            t0[m * RS] = xv[u];
            t0[-m * RS + P] = xv[u];   // the second set of columns: orders reversed
        }
    }
    const int pr = lane & (P - 1);
    for (int pi = 0; pi < st.nparts; ++pi) {
        const DgPart part = ar.parts[st.part0 + pi];
        const int ps = dir_run<float>(part.len);
        load_run(part, ps);
        lds_barrier();
        // the lane's pair's run, from the stage's first output
        const float* lrun = run + pr * ps + (int)(((p0 + pr) * nout + part.off) & 3) - (part.off - st.off);
        for (int ti = wave; ti < st.ntasks; ti += kDgWaves) {
            const DgTask t = ar.tasks[st.task0 + ti];
            switch ((t.code >> 24) & 15) {
                case 1: dg_task<G, 1>(t, part, ar.coef, smem, lrun, lane); break;
                case 2: dg_task<G, 2>(t, part, ar.coef, smem, lrun, lane); break;
                default: dg_task<G, 3>(t, part, ar.coef, smem, lrun, lane); break;
            }
        }
        lds_barrier();
    }
    // ---- the blocks' gradient rows: both order signs, grad_b over the tasks in order
    for (int r = tid; r < st.nouts; r += kDgThreads) {
        const DgOut o = ar.outs[st.out0 + r];
        const int nt = o.code & 15, stride = (o.code >> 4) & 0xffff, e = (o.code >> 20) & 0xff;
        const int nrow = o.ws >> 20;
        float* dst = ar.ws + (int64_t)(o.ws & 0xfffff) * ar.N + p0 * nrow + e;
        for (int p = 0; p < np; ++p) {
            float v = 0.0f;
            for (int t = 0; t < nt; ++t) v += smem[o.plus + t * stride + p] + smem[o.minus + t * stride + p];
            dst[(int64_t)p * nrow] = v;
        }
    }
}

__global__ __launch_bounds__(kDgThreads, 3) void direct_backward_kernel(const DgArgs ar) {
    extern __shared__ __align__(16) unsigned char dg_smem[];
    float* smem = reinterpret_cast<float*>(dg_smem);
    const int c = ar.ncls > 1 && (int64_t)blockIdx.x >= ar.wg0[1] ? 1 : 0;
    // (work-groups of a class start at a multiple of 8: work-group i runs on XCD i mod 8)
    const int64_t i = blockIdx.x - ar.wg0[c], xcd = i & 7, j = i >> 3, ck = j / ar.chunk[c];
    const int64_t unit = (ck * 8 + xcd) * ar.chunk[c] + (j - ck * ar.chunk[c]);
    if (unit >= ar.nunits[c]) return;
    const int P = dg_pairs(ar.G[c]);
    const int64_t ntiles = (ar.N + P - 1) / P, si = unit / ntiles;
    const DgStage st = ar.stages[ar.stage0[c] + si];
    const int64_t p0 = (unit - si * ntiles) * P;
    if (ar.G[c] == 2)
        dg_stage<2>(ar, st, p0, smem);
    else
        dg_stage<4>(ar, st, p0, smem);
}

}  // namespace

int launch_direct_backward(const DgTables& tb, const float* x1, const float* x2, const float* g, float* gx1, float* gx2,
                           float* ws, int64_t N, int L, void* stream) {
    DgArgs ar{};
    ar.coef = tb.coef;
    ar.tasks = tb.tasks;
    ar.outs = tb.outs;
    ar.parts = tb.parts;
    ar.stages = tb.stages;
    ar.x1 = x1;
    ar.x2 = x2;
    ar.g = g;
    ar.ws = ws;
    ar.N = N;
    ar.L = L;
    int64_t units = 0;
    for (int c = 0; c < kDgClasses; ++c) {
        const int P = dg_pairs(dg_groups(c));
        units += (N + P - 1) / P * tb.lists[1].nstages[c];
    }
    const DgList& ls = tb.lists[units <= kDgShortMax ? 1 : 0];
    // classes 0 and 1 in one launch, class 2 in its own with more LDS
    for (int c0 = 0; c0 < kDgClasses; c0 += 2) {
        ar.ncls = c0 == 0 ? 2 : 1;
        ar.wg0[0] = 0;
        int lds = 0;
        for (int i = 0; i < ar.ncls; ++i) {
            const int c = c0 + i, P = dg_pairs(dg_groups(c));
            ar.G[i] = dg_groups(c);
            ar.stage0[i] = ls.stage0;
            for (int k = 0; k < c; ++k) ar.stage0[i] += ls.nstages[k];
            ar.nunits[i] = (N + P - 1) / P * ls.nstages[c];
            ar.chunk[i] = ar.nunits[i] >= 96 * 32 ? 96 : ar.nunits[i] >= 256 ? 8 : 1;
            const int64_t per = 8LL * ar.chunk[i];
            ar.wg0[i + 1] = ar.wg0[i] + (ar.nunits[i] + per - 1) / per * per;
            lds = std::max(lds, ls.lds_bytes[c]);
        }
        if (ar.wg0[ar.ncls] == 0) continue;
        if (lds > 64 * 1024) {   // (always the same limit, as for the forward)
            const hipError_t e = hipFuncSetAttribute((const void*)direct_backward_kernel,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBudget);
            if (e != hipSuccess) return (int)e;
        }
        const int err = dir_launches(ar.wg0[ar.ncls], 8, kDgThreads, [&](int64_t first, unsigned grid) {
            DgArgs al = ar;
            for (int i = 0; i <= ar.ncls; ++i) al.wg0[i] -= first;
            hipLaunchKernelGGL(direct_backward_kernel, dim3(grid), dim3(kDgThreads), lds, (hipStream_t)stream, al);
            return (int)hipGetLastError();
        });
        if (err) return err;
    }
    return launch_backward_sums(ws, gx1, gx2, N, L, stream);
}

}  // namespace cgtp
