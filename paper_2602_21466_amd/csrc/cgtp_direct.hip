// Direct contraction of the CGTP on the matrix cores (cgtp_direct.h has the
// scheme and the work lists).
//
// One work-group of 8 waves makes the stages of one group for a tile of pairs:
// it fills the input tiles once; per stage its waves take the items in turn
// (coefficients from the plan's table in L2, one 16-byte load per lane for 8 k
// steps; the products x_a x_b formed from two LDS reads per step, the second
// input's values shared by four consecutive orders), put the results together
// in LDS in output order, and then write them as whole runs.
//
// Bound by instruction issue: the vector units issue in 59 % of the SIMD cycles
// at L = 16 (54 % at L = 32), the matrix cores work in 19 % (25 %).  Most of it
// is not the k loop: per item and wave 286 (352) vector instructions besides the
// MFMAs, of which 54 (105) are the products and the other 230 to 250 the item's
// fixed cost: 16 accumulators cleared, 16 results each compared, masked, signed,
// addressed and stored.  Two work-groups per CU, so that one computes while the
// other stores.  Measured (us, sphere-grid kernels before / now): L = 16, 8192
// pairs 13467 / 1053; L = 32, 1024 pairs 22259 / 2175 (2.2 TB/s of outputs); real
// basis L = 11, 4001 pairs 2412 / 157; 16 weighted channels, L = 16, 8192 rows
// 14582 / 1171; one pair, fp64, L = 16 36 / 24.
// The 16x16x4 instruction takes 1948 us at L = 32, but 258 against 117 at L = 4
// (100000 pairs) and 191 against 162 in the real basis at L = 11.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "cgtp_direct.h"
#include "cgtp_internal.h"
#include "device_common.h"

namespace cgtp {
namespace {

using namespace ::cgtp::dev;

enum DirMode { kDirPlain = 0, kDirWeighted = 1, kDirReal = 2 };

constexpr double kSqrt2 = 1.41421356237309504880168872420970;
constexpr double kInvSqrt2 = 0.70710678118654752440084436210485;

template <typename T>
struct DirArgs {
    const T* __restrict__ coef;
    const DirItem* __restrict__ items;
    const DirStage* __restrict__ stages;
    const DirGroup* __restrict__ groups;
    const T* __restrict__ x1;
    const T* __restrict__ x2;
    T* __restrict__ out;
    const T* __restrict__ w;
    int64_t N;
    // units (group, tile of pairs), the tiles of a group in turn
    uint32_t ntiles;          // tiles of pairs
    uint32_t group0, tile0;   // first unit of the launch
    uint32_t nunits;          // units of the launch
    uint32_t chunk;           // consecutive units given to one XCD
    int32_t L;
    int32_t channels, flags, npaths;
};

// Coefficients of one chunk and the k step that uses them.
template <typename T> struct DirCoef;

template <> struct DirCoef<float> {
    f32x4 a;   // the lane's coefficient for each of the four orders
    __device__ __forceinline__ void load(const float* __restrict__ coef, int chunk, int lane) {
        a = *reinterpret_cast<const f32x4*>(coef + (size_t)chunk * kDirChunk + 4 * lane);
    }
    template <int J> __device__ __forceinline__ void step(const float (&b)[4], f32x4 (&acc)[4]) const {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) acc[mi] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[mi], b[mi], acc[mi], 3, J, 0);
    }
};

template <> struct DirCoef<double> {
    const double* a;
    __device__ __forceinline__ void load(const double* __restrict__ coef, int chunk, int) {
        a = coef + (size_t)chunk * kDirChunk;
    }
    template <int J> __device__ __forceinline__ void step(const double (&b)[4], f64x4 (&acc)[4]) const {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int r = 0; r < kDirRows; ++r) acc[mi][r] = fma(a[16 * J + 4 * mi + r], b[mi], acc[mi][r]);
    }
};

// k steps J .. of one chunk: the factors of step J and the multiply-adds.
// TAIL: only the first `cnt` steps.
template <typename T, int MODE, int J, bool TAIL>
__device__ __forceinline__ void dir_steps(const DirCoef<T>& cf, const T* pa, const T* pb, int part, T im_sign, int cnt,
                                          T (&w)[2][3], typename Cplx<T>::acc4 (&acc)[4]) {
    constexpr int KC = dir_kc<T>(), RS = dir_row<T>(), P = dir_pairs<T>();
    if constexpr (J < KC) {
        if (TAIL && J >= cnt) return;
        T b[4];
        if constexpr (MODE == kDirReal) {
            // (a1 + i b1)(a2 + i b2): the lane's part is a1 own + (-b1 or b1) other
            const T a1 = pa[-J * RS], b1 = im_sign * pa[P - J * RS];
            const T own = pb[(J + 3) * RS + part], oth = pb[(J + 3) * RS + (P - part)];
            const T wo[4] = {w[0][0], w[0][1], w[0][2], own}, wt[4] = {w[1][0], w[1][1], w[1][2], oth};
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) b[mi] = a1 * wo[mi] + b1 * wt[mi];
            w[0][0] = w[0][1];
            w[0][1] = w[0][2];
            w[0][2] = own;
            w[1][0] = w[1][1];
            w[1][1] = w[1][2];
            w[1][2] = oth;
        } else {
            const T xa = pa[-J * RS], xb = pb[(J + 3) * RS];
            b[0] = xa * w[0][0];
            b[1] = xa * w[0][1];
            b[2] = xa * w[0][2];
            b[3] = xa * xb;
            w[0][0] = w[0][1];
            w[0][1] = w[0][2];
            w[0][2] = xb;
        }
        cf.template step<J>(b, acc);
        dir_steps<T, MODE, J + 1, TAIL>(cf, pa, pb, part, im_sign, cnt, w, acc);
    }
}

template <typename T, int MODE>
__global__ __launch_bounds__(kDirThreads, 4) void direct_kernel(const DirArgs<T> ar) {
    using Acc = typename Cplx<T>::acc4;
    constexpr int P = dir_pairs<T>(), KC = dir_kc<T>(), RS = dir_row<T>();
    extern __shared__ __align__(16) unsigned char smem[];
    T* tile = reinterpret_cast<T*>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // work-group -> unit (group, tile of pairs): work-group i runs on XCD i mod 8;
    // an XCD takes `chunk` consecutive units at a time, so the work-groups that
    // read the same coefficients share its L2
    const uint32_t xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const uint32_t ck = j / ar.chunk, unit = (ck * 8 + xcd) * ar.chunk + (j - ck * ar.chunk);
    if (unit >= ar.nunits) return;
    const uint32_t tu = ar.tile0 + unit, dgi = tu / ar.ntiles, gi = ar.group0 + dgi;
    const int64_t p0 = (int64_t)(tu - dgi * ar.ntiles) * P;
    const int np = (int)(ar.N - p0 < P ? ar.N - p0 : P);
    const DirGroup g = ar.groups[gi];
    const int nin = (ar.L + 1) * (ar.L + 1);
    const int64_t nout = (int64_t)nin * nin;
    T* st_buf = tile + g.tile_len;

    // ---- input tiles: zero (padding rows, pairs past N), then the columns
    for (int e = tid * 4; e < g.tile_len; e += kDirThreads * 4)
        *reinterpret_cast<Acc*>(tile + e) = Acc(0);
    lds_barrier();
    for (int p = wave; p < np; p += kDirWaves) {
        const int64_t row = p0 + p;
        const int64_t row2 = (MODE == kDirWeighted && (ar.flags & kX2Shared)) ? row / ar.channels : row;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int la = s ? g.l2a : g.l1a, lb = s ? g.l2b : g.l1b;
            const T* src = s ? ar.x2 + row2 * nin : ar.x1 + row * nin;
            T* dst = tile + (s ? g.x2tile : 0);
            for (int i = la * la + lane; i < (lb + 1) * (lb + 1); i += 64) {
                int l = (int)__builtin_sqrtf((float)i + 0.5f);   // exact for i < 2^20
                const int m = i - l * l - l;
                const T v = src[i];
                T* t0 = dst + (dir_tile_row<T>(l, la) + l) * RS + p;   // order 0
                if constexpr (MODE == kDirReal) {
                    // complex coefficients of a real-basis row: c_0 = r_0,
                    // c_m = (-1)^m (r_m - i r_-m) / sqrt 2, c_-m = (r_m + i r_-m) / sqrt 2
                    const T h = (T)kInvSqrt2 * v;
                    const T hs = (m & 1) ? -h : h;
                    if (m == 0) {
                        t0[0] = v;
                    } else if (m > 0) {
                        t0[m * RS] = hs;
                        t0[-m * RS] = h;
                    } else {
                        t0[-m * RS + P] = -hs;
                        t0[m * RS + P] = h;
                    }
                } else {
                    // the second set of columns holds the orders reversed
                    t0[m * RS] = v;
                    t0[-m * RS + P] = v;
                }
            }
        }
    }
    lds_barrier();

    // The instructions from here on start 4 bytes past a multiple of 8, whatever is
    // before them (real basis, L = 11, 4001 pairs: 150.5 us, at a multiple of 8 152.4;
    // the other modes do not care)
    asm volatile(".p2align 3\n\ts_nop 0");

    // the lane's column: pair, half (order sign or part) and group of orders
    const int col = lane & (2 * P - 1), gm = 4 * (lane / (2 * P)), pr = col & (P - 1), half = col / P;
    // (real basis: even rows go to +M from the real part, odd rows to -M)
    const int sg_even = half ? -1 : 1, sg_odd = MODE == kDirReal ? -sg_even : sg_even;
    const T* colp = tile + (MODE == kDirReal ? pr : col);
    const T im_sign = half ? (T)1 : (T)-1;
    const T* wrow = nullptr;
    if constexpr (MODE == kDirWeighted) {
        if (ar.w) {
            const int64_t r = p0 + (pr < np ? pr : 0);
            wrow = ar.w + ((ar.flags & kWeightsPerRow) ? r : r % ar.channels) * ar.npaths;
        }
    }

    for (int si = g.stage0; si < g.stage0 + g.nstages; ++si) {
        const DirStage st = ar.stages[si];
        const int ps = st.len | 1;   // odd: pairs start on different banks
        for (int t = 0, ii = wave; ii < st.nitems; ++t, ii = t * kDirWaves + ((t & 1) ? kDirWaves - 1 - wave : wave)) {
            const DirItem it = ar.items[st.item0 + ii];
            const int lt = it.code & 0xff, lmin = (it.code >> 8) & 0xff, m0 = (it.code >> 16) & 0xff;
            const bool swap = it.code >> 24;
            Acc acc[4];
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) acc[mi] = Acc(0);
            DirCoef<T> cf, cfn;
            cf.load(ar.coef, it.chunk0, lane);
            const T* pa = colp + it.xa;
            const T* pb = colp + it.xb + gm * RS;
            const int part = MODE == kDirReal ? half * P : 0;
            T w[2][3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                w[0][i] = pb[i * RS + part];
                w[1][i] = MODE == kDirReal ? pb[i * RS + (P - part)] : (T)0;
            }
            int k = 0;
            for (; k + KC <= it.nk; k += KC) {
                cfn = cf;
                if (k + KC < it.nk) cfn.load(ar.coef, it.chunk0 + k / KC + 1, lane);
                dir_steps<T, MODE, 0, false>(cf, pa - k * RS, pb + k * RS, part, im_sign, KC, w, acc);
                cf = cfn;
            }
            if (k < it.nk) dir_steps<T, MODE, 0, true>(cf, pa - k * RS, pb + k * RS, part, im_sign, it.nk - k, w, acc);

            // ---- results of degree lt - r, order m0 + gm + mi, into the stage's run
            const T f_odd = ((MODE != kDirReal && half) != swap) ? (T)-1 : (T)1;
            T* o0 = st_buf + pr * ps + it.c;
            const int mg = m0 + gm;
#pragma unroll
            for (int r = 0; r < kDirRows; ++r) {
                const int l3 = lt - r;
                if (l3 < lmin) break;
                T* orow = o0 + l3 * (l3 + 1);
                T f = (r & 1) ? f_odd : (T)1;
                if constexpr (MODE == kDirWeighted) {
                    if (ar.w) f *= wrow[it.path + l3];
                }
                const int sg = (r & 1) ? sg_odd : sg_even;
#pragma unroll
                for (int mi = 0; mi < 4; ++mi) {
                    const int M = mg + mi;
                    T v = acc[mi][r];
                    bool ok = M <= l3;
                    if constexpr (MODE == kDirReal) {
                        // with z the path at order M: even paths r_M = sqrt 2 (-1)^M Re z,
                        // r_-M = -sqrt 2 (-1)^M Im z; odd ones r_M = -sqrt 2 (-1)^M Im z,
                        // r_-M = -sqrt 2 (-1)^M Re z; order 0: Re z and -Im z
                        T fr = (mi & 1) ? (T)-kSqrt2 : (T)kSqrt2;
                        if ((r & 1) || half) fr = -fr;
                        if (M == 0) {
                            fr = (r & 1) ? (T)-1 : (T)1;
                            ok = ok && half == (r & 1);
                        }
                        v *= f * fr;
                    } else {
                        ok = ok && (M > 0 || !half);
                        v *= f;
                    }
                    if (ok) orow[sg * M] = v;
                }
            }
        }
        lds_barrier();
        for (int p = wave; p < np; p += kDirWaves) {
            T* dst = ar.out + (p0 + p) * nout + st.off;
            const T* src = st_buf + p * ps;
            for (int i = lane; i < st.len; i += 64) __builtin_nontemporal_store(src[i], dst + i);
        }
        lds_barrier();
    }
}

template <typename T, int MODE>
int launch_mode(int lds_bytes, int64_t nunits, DirArgs<T>& ar, void* stream) {
    const void* kern = (const void*)direct_kernel<T, MODE>;
    if (lds_bytes > 64 * 1024) {
        // (always the same limit: threads that launch different lists cannot lower it for each other)
        const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBudget);
        if (e != hipSuccess) return (int)e;
    }
    return dir_launches(nunits, 8LL * ar.chunk, kDirThreads, [&](int64_t first, unsigned grid) {
        ar.group0 = (uint32_t)(first / ar.ntiles);
        ar.tile0 = (uint32_t)(first % ar.ntiles);
        ar.nunits = (uint32_t)std::min<int64_t>(grid, nunits - first);
        hipLaunchKernelGGL((direct_kernel<T, MODE>), dim3(grid), dim3(kDirThreads), lds_bytes, (hipStream_t)stream,
                           ar);
        return (int)hipGetLastError();
    });
}

template <typename T>
int launch(const DirTables<T>& tb, const T* x1, const T* x2, T* out, int64_t N, int L, const ChanArgs<T>* ch,
           bool real_basis, void* stream) {
    DirArgs<T> ar{};
    ar.coef = tb.coef;
    ar.items = tb.items;
    ar.stages = tb.stages;
    ar.x1 = x1;
    ar.x2 = x2;
    ar.out = out;
    ar.N = N;
    const int64_t ntiles = (N + dir_pairs<T>() - 1) / dir_pairs<T>();
    if (ntiles > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;   // (more pairs than memory holds)
    const DirList& ls = tb.lists[ntiles * tb.lists[1].ngroups <= kDirShortMax ? 1 : 0];
    const int64_t nunits = ntiles * ls.ngroups;
    ar.groups = tb.groups + ls.group0;
    ar.ntiles = (uint32_t)ntiles;
    // 64 units at a time (the work-groups an XCD runs at once) where every XCD
    // gets several such chunks, else fewer
    ar.chunk = nunits >= 64 * 32 ? 64 : nunits >= 256 ? 8 : 1;
    ar.L = L;
    if (real_basis) return launch_mode<T, kDirReal>(ls.lds_bytes, nunits, ar, stream);
    if (!ch) return launch_mode<T, kDirPlain>(ls.lds_bytes, nunits, ar, stream);
    ar.w = ch->w;
    ar.channels = ch->channels;
    ar.flags = ch->flags;
    ar.npaths = ch->npaths;
    return launch_mode<T, kDirWeighted>(ls.lds_bytes, nunits, ar, stream);
}

}  // namespace

int launch_direct_f32(const DirTables<float>& tb, const float* x1, const float* x2, float* out, int64_t N, int L,
                      const ChanArgs<float>* ch, bool real_basis, void* stream) {
    return launch<float>(tb, x1, x2, out, N, L, ch, real_basis, stream);
}
int launch_direct_f64(const DirTables<double>& tb, const double* x1, const double* x2, double* out, int64_t N, int L,
                      const ChanArgs<double>* ch, bool real_basis, void* stream) {
    return launch<double>(tb, x1, x2, out, N, L, ch, real_basis, stream);
}

}  // namespace cgtp
