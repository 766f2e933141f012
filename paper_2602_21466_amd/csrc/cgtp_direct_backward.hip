// Gradients of the CGTP by the direct contraction, transposed (cgtp_direct.h
// has the scheme and the work lists), fp32.
//
// Per stage and tile of pairs: the input tiles and the stage's runs of the
// upstream gradient go to LDS; each wave takes its tasks through all orders
// (per k step four LDS reads feed 4 x (row groups) MFMAs); the sums of a block
// are then put together over its tasks and order signs and written to the
// workspace, which launch_backward_sums adds up over the other degree.

#include <hip/hip_runtime.h>

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
    const DgBlock* __restrict__ blocks;
    const DgStage* __restrict__ stages;
    const float* __restrict__ x1;
    const float* __restrict__ x2;
    const float* __restrict__ g;
    float* __restrict__ ws;
    int64_t N;
    int64_t nunits[kDgClasses];       // stages x tiles of pairs
    int64_t wg0[kDgClasses + 1];      // first work-group of each class
    int32_t stage0[kDgClasses];
    int32_t chunk[kDgClasses];        // consecutive units given to one XCD
    int32_t L;
};

template <int G, int J> __device__ __forceinline__ f32x4 dg_mfma(float a, float b, f32x4 c) {
    // the coefficients of step J, four rows, broadcast to the columns of each group of orders
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, G == 2 ? 3 : G == 4 ? 2 : 1, J, 0);
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
__device__ __forceinline__ void dg_task(const DgTask& t, const float* __restrict__ coef, float* smem, const float* run,
                                        int ps, int lane) {
    constexpr int P = dg_pairs(G), KC = dg_kc(G), RS = dg_row(G), HM = dg_orders(G), NR = 4 * RG;
    static_assert(KC % 2 == 0, "a chunk starts at an even step");
    const int col = lane & (2 * P - 1), gm = 4 * (lane / (2 * P)), pr = col & (P - 1);
    const bool neg = col >= P;
    const int la = t.code & 255, lb = (t.code >> 8) & 255, k0 = (t.code >> 16) & 255;
    const bool swap = (t.code >> 28) & 1;
    const float f_odd = neg != swap ? -1.0f : 1.0f;
    const int lt = la + lb, sg = neg ? -1 : 1;
    float ga[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) ga[i] = 0.0f;
    const float* xa = smem + t.xa + col;   // row i at -i RS
    const float* cf = coef + (size_t)t.chunk0 * kDirChunk + 4 * lane;
    float* accb = smem + t.accb + col;
    for (int m0 = 0; m0 <= lt; m0 += HM) {
        const int nk = min(2 * la + 1, lt - m0 + 1);
        if (nk <= k0) break;
        f32x4 acc[RG][4];
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) acc[r][mi] = f32x4(0);
        const float* gp[4];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) gp[mi] = run + pr * ps + t.goff + sg * (m0 + gm + mi);
        // chunks in which every order of the item has its degrees, then the others; the
        // next chunk's coefficients are loaded a chunk ahead (the table ends in spare ones)
        const int nfull = max(min(nk, lt - (m0 + HM - 1) + 1), 0) / KC * KC;
        f32x4 a[RG], an[RG];
#pragma unroll
        for (int r = 0; r < RG; ++r) a[r] = *reinterpret_cast<const f32x4*>(cf + r * kDirChunk);
        int s = 0;
        for (; s < nfull; s += KC) {
            cf += RG * kDirChunk;
#pragma unroll
            for (int r = 0; r < RG; ++r) an[r] = *reinterpret_cast<const f32x4*>(cf + r * kDirChunk);
            dg_steps<G, RG, 0, false>(a, gp, lt - s, KC, 0, f_odd, acc);
#pragma unroll
            for (int r = 0; r < RG; ++r) a[r] = an[r];
        }
        for (; s < nk; s += KC) {
            cf += RG * kDirChunk;
#pragma unroll
            for (int r = 0; r < RG; ++r) an[r] = *reinterpret_cast<const f32x4*>(cf + r * kDirChunk);
            dg_steps<G, RG, 0, true>(a, gp, lt - s, nk - s, m0 + gm, f_odd, acc);
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
                dst[u] = accb + d * 2 * P;
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
    // grad_a: summed over the groups of orders
#pragma unroll
    for (int i = 0; i < NR; ++i) {
#pragma unroll
        for (int o = 2 * P; o < 64; o *= 2) ga[i] += __shfl_xor(ga[i], o);
        if (gm == 0) smem[t.acca + i * 2 * P + col] = ga[i];
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
    const int ps = st.len | 1;
    float* run = smem + st.tile_len;
    for (int e = tid * 4; e < st.tile_len; e += kDgThreads * 4) *reinterpret_cast<f32x4*>(smem + e) = f32x4(0);
    for (int e = st.acc0 + tid * 4; e < st.acc0 + st.acc_len; e += kDgThreads * 4)
        *reinterpret_cast<f32x4*>(smem + e) = f32x4(0);
    lds_barrier();
    for (int p = wave; p < np; p += kDgWaves) {
        const float* src = ar.g + (p0 + p) * nout + st.off;
        float* dst = run + p * ps;
        for (int i0 = 0; i0 < st.len; i0 += 8 * 64) {   // eight loads in flight per lane
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + 64 * u + lane;
                v[u] = i < st.len ? __builtin_nontemporal_load(src + i) : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + 64 * u + lane;
                if (i < st.len) dst[i] = v[u];
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int la = s ? st.l2a : st.l1a, lb = s ? st.l2b : st.l1b;
            const float* xs = (s ? ar.x2 : ar.x1) + (p0 + p) * nin;
            float* tile = smem + (s ? st.x2tile : 0);
            for (int i = la * la + lane; i < (lb + 1) * (lb + 1); i += 64) {
                const int l = (int)__builtin_sqrtf((float)i + 0.5f);   // exact for i < 2^20
                const int m = i - l * l - l;
                const float v = xs[i];
                float* t0 = tile + (dg_tile_row(l, la) + l) * RS + p;   // order 0
                t0[m * RS] = v;
                t0[-m * RS + P] = v;   // the second set of columns: orders reversed
            }
        }
    }
    lds_barrier();
    for (int ti = wave; ti < st.ntasks; ti += kDgWaves) {
        const DgTask t = ar.tasks[st.task0 + ti];
        switch ((t.code >> 24) & 15) {
            case 1: dg_task<G, 1>(t, ar.coef, smem, run, ps, lane); break;
            case 2: dg_task<G, 2>(t, ar.coef, smem, run, ps, lane); break;
            default: dg_task<G, 3>(t, ar.coef, smem, run, ps, lane); break;
        }
    }
    lds_barrier();
    // ---- per block: both order signs, grad_b over the tasks in order
    for (int b = st.block0; b < st.block0 + st.nblocks; ++b) {
        const DgBlock bl = ar.blocks[b];
        const int n1 = 2 * bl.l1 + 1, n2 = 2 * bl.l2 + 1, nrow = n1 + n2;
        const bool swap = bl.l1 > bl.l2;
        float* dst = ar.ws + bwd_block_off(ar.L, bl.l1, bl.l2) * ar.N + p0 * nrow;
        for (int e = tid; e < np * nrow; e += kDgThreads) {
            const int p = e / nrow, ee = e - p * nrow;
            const bool first = ee < n1;
            const int l = first ? bl.l1 : bl.l2, m = (first ? ee : ee - n1) - l;
            float v;
            if (first != swap) {   // the smaller degree's input (x1 if equal)
                const float* a = smem + bl.acca + p;
                v = a[(l - m) * 2 * P] + a[(l + m) * 2 * P + P];
            } else {
                v = 0.0f;
                for (int t = 0; t < bl.ntasks; ++t) {
                    const float* a = smem + bl.accb + t * bl.stride + p;
                    v += a[(l + m) * 2 * P] + a[(l - m) * 2 * P + P];
                }
            }
            dst[e] = v;
        }
    }
}

__global__ __launch_bounds__(kDgThreads, 3) void direct_backward_kernel(const DgArgs ar) {
    extern __shared__ __align__(16) unsigned char dg_smem[];
    float* smem = reinterpret_cast<float*>(dg_smem);
    int c = 0;
    while (c + 1 < kDgClasses && (int64_t)blockIdx.x >= ar.wg0[c + 1]) ++c;
    // (work-groups of a class start at a multiple of 8: work-group i runs on XCD i mod 8)
    const int64_t i = blockIdx.x - ar.wg0[c], xcd = i & 7, j = i >> 3, ck = j / ar.chunk[c];
    const int64_t unit = (ck * 8 + xcd) * ar.chunk[c] + (j - ck * ar.chunk[c]);
    if (unit >= ar.nunits[c]) return;
    const int P = dg_pairs(dg_groups(c));
    const int64_t ntiles = (ar.N + P - 1) / P, si = unit / ntiles;
    const DgStage st = ar.stages[ar.stage0[c] + si];
    const int64_t p0 = (unit - si * ntiles) * P;
    if (c == 0)
        dg_stage<2>(ar, st, p0, smem);
    else if (c == 1)
        dg_stage<4>(ar, st, p0, smem);
    else
        dg_stage<8>(ar, st, p0, smem);
}

}  // namespace

int launch_direct_backward(const DgTables& tb, const float* x1, const float* x2, const float* g, float* gx1, float* gx2,
                           float* ws, int64_t N, int L, void* stream) {
    DgArgs ar{};
    ar.coef = tb.coef;
    ar.tasks = tb.tasks;
    ar.blocks = tb.blocks;
    ar.stages = tb.stages;
    ar.x1 = x1;
    ar.x2 = x2;
    ar.g = g;
    ar.ws = ws;
    ar.N = N;
    ar.L = L;
    int s0 = 0;
    for (int c = 0; c < kDgClasses; ++c) {
        const int P = dg_pairs(dg_groups(c));
        ar.stage0[c] = s0;
        s0 += tb.nstages[c];
        ar.nunits[c] = (N + P - 1) / P * tb.nstages[c];
        ar.chunk[c] = ar.nunits[c] >= 96 * 32 ? 96 : ar.nunits[c] >= 256 ? 8 : 1;
        const int64_t per = 8LL * ar.chunk[c];
        ar.wg0[c + 1] = ar.wg0[c] + (ar.nunits[c] + per - 1) / per * per;
    }
    if (ar.wg0[kDgClasses] > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    if (tb.lds_bytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)direct_backward_kernel,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, tb.lds_bytes);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL(direct_backward_kernel, dim3((unsigned)ar.wg0[kDgClasses]), dim3(kDgThreads), tb.lds_bytes,
                       (hipStream_t)stream, ar);
    const int err = (int)hipGetLastError();
    return err ? err : launch_backward_sums(ws, gx1, gx2, N, L, stream);
}

}  // namespace cgtp
