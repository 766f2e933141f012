// Internal layout of the direct contraction, shared by its plan
// (cgtp_direct_plan.h) and its kernels (cgtp_direct.hip,
// cgtp_direct_backward.hip).  Not part of the
// public ABI.
//
// Every (l1, l2) block of the CGTP is, per order M >= 0 of the output, one
// square orthogonal matrix of Clebsch-Gordan coefficients
//   A_M[l3][k] = C^{l3 M}_{la ma, lb M-ma},  ma = la - k,
// (la <= lb the block's degrees, n(M) = min(2 la + 1, la + lb - M + 1) rows and
// columns) applied to the products x_a[ma] x_b[M - ma] of every pair; orders
// -M use the same matrix on the reversed products, up to the sign
// (-1)^(l1+l2-l3), and block (lb, la) the same up to that sign.  Per block that
// is 2 n^2 multiply-adds per M for 2 n outputs: at L = 32 31 M per pair, a
// fifth of the arithmetic of the sphere-grid method, all of it contraction.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace cgtp {

// A wave works on 64 columns at once: kDirPairs pairs x 2 (orders +M and -M;
// real basis: real and imaginary part) x G groups of four consecutive orders.
// fp32: G = 2 groups on v_mfma_f32_4x4x1_16b (16 blocks of 4 rows x 4 columns;
// the coefficients of 8 k steps x 4 rows of each group fill one operand
// register, and the instruction broadcasts the step's block to its group).
// fp64: G = 1, vector multiply-adds with the coefficient in scalar registers.
template <typename T> struct DirGeom;
template <> struct DirGeom<float> {
    static constexpr int G = 2;
};
template <> struct DirGeom<double> {
    static constexpr int G = 1;
};
template <typename T> __host__ __device__ constexpr int dir_pairs() { return 32 / DirGeom<T>::G; }
template <typename T> __host__ __device__ constexpr int dir_kc() { return 16 / DirGeom<T>::G; }       // k steps per coefficient chunk
template <typename T> __host__ __device__ constexpr int dir_orders() { return 4 * DirGeom<T>::G; }    // orders M per item
constexpr int kDirThreads = 512;
constexpr int kDirWaves = kDirThreads / 64;
constexpr int kDirRows = 4;        // output degrees l3 per item
constexpr int kDirChunk = 256;     // coefficients per chunk

// LDS tile of one input: per degree l, 2 l + 1 rows (order m = row - l) and
// dir_orders - 1 zero rows, which the last orders of an item read past the
// degree; a row holds the 2 dir_pairs columns and one element of padding.
template <typename T> __host__ __device__ constexpr int dir_row() { return 2 * dir_pairs<T>() + 1; }
template <typename T> __host__ __device__ constexpr int dir_pad() { return dir_orders<T>() - 1; }
template <typename T> __host__ __device__ inline int dir_tile_row(int l, int l0) {
    return l * l - l0 * l0 + dir_pad<T>() * (l - l0);
}

// One item: 4 output degrees lt, lt-1, lt-2, lt-3 (those >= lmin) of one block
// for the orders m0 .. m0 + dir_orders - 1 (those <= the degree).
struct alignas(16) DirItem {
    int32_t chunk0;   // first coefficient chunk
    int32_t nk;       // k steps: n(m0)
    int32_t xa;       // tile element of (la, ma = la); step k is k rows further down
    int32_t xb;       // tile element of (lb, mb = m0 - la); step k is k rows further up
    int32_t code;     // lt | lmin << 8 | m0 << 16 | (l1 > l2) << 24
    int32_t c;        // output (l3, M) sits at c + l3^2 + l3 + M of the stage's run
    int32_t path;     // path (l1, l2, l3) has index path + l3
    int32_t pad;
};

// One stage: a run of consecutive outputs of every pair, small enough to be
// put together in LDS and written as whole lines.
struct DirStage {
    int32_t item0, nitems;   // heaviest items first
    int32_t off, len;        // run of one pair's output
};

// One group: the consecutive stages a work-group makes from one filling of the
// input tiles (x1 degrees l1a..l1b, x2 degrees l2a..l2b).
struct DirGroup {
    int32_t stage0, nstages;
    int32_t l1a, l1b, l2a, l2b;
    int32_t x2tile;      // first element of the x2 tile (x1's is at 0)
    int32_t tile_len;    // elements of both tiles, a multiple of 4
};

// One way to cut the outputs into groups.  The long list's groups share the
// filling of their input tiles over several stages; the short list's are one
// short stage each, for calls whose pairs give the long list too few work-groups
// to fill the chip, so that each is a long chain of stages.  The items are the
// same, so the outputs do not depend on the list, to the last bit.
struct DirList {
    int32_t group0, ngroups;
    int32_t lds_bytes;
};

template <typename T>
struct DirTables {
    const T* coef;
    const DirItem* items;
    const DirStage* stages;
    const DirGroup* groups;
    DirList lists[2];   // long, short
};
// The short list is taken while it makes at most six work-groups per CU.  (us, long
// list / short: fp64 L = 4, 1 pair 18.7 / 7.7; L = 6, 1000 39.8 / 24.4 (800
// work-groups); L = 19, 16 103 / 46 (1229); L = 10, 300 49 / 32 (1560); above: L = 8,
// 1000 40 / 68 (2304).  fp32 L = 8, 16 19.6 / 7.9; L = 20, 1 24.4 / 9.1 (1060); real
// L = 13, 100 29 / 17 (1540); L = 8, 1000 23.3 / 24.4 (2205); L = 11, 300 20 / 25 (2223).)
constexpr int64_t kDirShortMax = 6 * 256;

// Elements from one pair's run in LDS to the next: room for its offset from a
// 16-byte boundary, and an odd number of 16-byte units, so that the pairs of a
// wave start on different banks.
template <typename T> __host__ __device__ inline int dir_run(int len) {
    const int v = 16 / (int)sizeof(T);
    return ((len + v - 1 + v - 1) / v | 1) * v;
}

// fp32 coefficients of a chunk: element (lane, mi) at 4 lane + mi with
// lane = ((group of orders) kc + k) 4 + row; fp64: (k, mi, row) at 16 k + 4 mi + row.
template <typename T> __host__ __device__ inline int dir_coef_index(int k, int order, int row);
template <> __host__ __device__ inline int dir_coef_index<float>(int k, int order, int row) {
    return (((order >> 2) * dir_kc<float>() + k) * 4 + row) * 4 + (order & 3);
}
template <> __host__ __device__ inline int dir_coef_index<double>(int k, int order, int row) {
    return 16 * k + 4 * order + row;
}

// ---------------------------------------------------------------- gradients (fp32)
//
// T_M[k] = sum over l3 of A_M[l3][k] g[l3, M] (the same matrices transposed, the
// rows now k, the k steps l3 = lt, lt-1, ...), then
//   grad_a[ma] += T_M[k] x_b[M - ma],   grad_b[M - ma] += T_M[k] x_a[ma].
// One work-group takes the gradient runs of one stage (consecutive blocks, or
// one large block in parts of some degrees l3 each) for a tile of 32 / G pairs
// into LDS; a task is up to kDgRows groups of four rows k of one block, which
// one wave takes through all orders, so grad_a stays in its registers and
// grad_b in an LDS array of its own: every sum has a fixed order.  G = 2 or 4
// groups of four orders per wave, so that the runs of 16 or 8 pairs leave room
// for two or three work-groups per CU.  (Measured at L = 16, N = 8192: 200
// outputs as the limit of G = 2 2420 us, 512 2692, 1100 4478; at L = 32,
// N = 1024: large blocks with 52 KiB of LDS 7994 us, 79 KiB 5143.)
constexpr int kDgThreads = 256;
constexpr int kDgWaves = kDgThreads / 64;
constexpr int kDgRows = 3;         // row groups per task
// Classes of blocks: up to 200 outputs with G = 2, the others with G = 4; those
// above 1100 outputs in parts, with two work-groups per CU (fewer parts: each
// costs another round of the two gradients) and a launch of their own.
constexpr int kDgClasses = 3;
__host__ __device__ constexpr int dg_class(int l1, int l2) {
    return (2 * l1 + 1) * (2 * l2 + 1) <= 200 ? 0 : (2 * l1 + 1) * (2 * l2 + 1) <= 1100 ? 1 : 2;
}
__host__ __device__ constexpr int dg_groups(int cls) { return cls == 0 ? 2 : 4; }
__host__ __device__ constexpr int dg_pairs(int G) { return 32 / G; }
__host__ __device__ constexpr int dg_kc(int G) { return 16 / G; }
__host__ __device__ constexpr int dg_orders(int G) { return 4 * G; }
__host__ __device__ constexpr int dg_row(int G) { return 2 * dg_pairs(G) + 1; }   // row of the tiles and the sums
constexpr int kDgMaxInputs = 192;  // inputs a stage may read per pair (both tiles)
// zero rows before each degree and after the last: a task's last row group
// reads up to three rows before its degree, and one row after a degree stands
// for all orders past it
constexpr int kDgPad = 3;
__host__ __device__ inline int dg_tile_row(int l, int l0) { return kDgPad + l * l - l0 * l0 + kDgPad * (l - l0); }
__host__ __device__ constexpr int dg_coef_index(int G, int k, int order, int row) {
    return (((order >> 2) * dg_kc(G) + k) * 4 + row) * 4 + (order & 3);
}

struct alignas(16) DgTask {
    int32_t chunk0;    // coefficients: [order group][chunk of k steps][row group]
    int32_t code;      // la | lb << 8 | first row k0 << 16 | row groups << 24 | (l1 > l2) << 28
    int32_t xa;        // tile element of (la, ma = la - k0); row k0 + i is i rows further down
    int32_t xb;        // tile element of (lb, mb = -lb)
    int32_t goff;      // g[l3, M] sits at goff + l3^2 + l3 + M of the stage's run
    int32_t acca;      // first element of the task's rows of grad_a, [k][column]
    int32_t accb;      // the task's grad_b, [lb + mb][column], one spare row at the end
    int32_t pad;
};

// One component of a block's two gradient rows: the sum over both order signs
// (and, for grad_b, the tasks) of elements plus + t stride, minus + t stride.
struct alignas(16) DgOut {
    int32_t plus, minus;
    int32_t code;      // tasks | stride << 4 | component << 20
    int32_t ws;        // the block's offset per pair in the workspace | its components << 20
};

// Some degrees of a stage: steps s0 .. s1-1 of its tasks.
struct alignas(16) DgPart {
    int32_t off, len;            // run of one pair's outputs
    int32_t s0, s1;
};

struct alignas(16) DgStage {
    int32_t off;                 // of the tasks' goff
    int32_t part0, nparts;
    int32_t task0, ntasks;       // heaviest first
    int32_t out0, nouts;
    int32_t l1a, l1b, l2a, l2b;
    int32_t x2tile, tile_len;    // elements; the run follows, then the sums
    int32_t acc0, acc_len;       // the sums' first element and length (multiples of 4)
    int32_t pad;
};

// One way to cut the blocks into stages (by class): the long list's stages fill
// the LDS of their class, the short list's hold one block, or small ones together.
// A block's tasks and parts are the same in both, and so are the gradients.
struct DgList {
    int32_t stage0;
    int32_t nstages[kDgClasses];
    int32_t lds_bytes[kDgClasses];
};

struct DgTables {
    const float* coef;
    const DgTask* tasks;
    const DgOut* outs;
    const DgPart* parts;
    const DgStage* stages;
    DgList lists[2];             // long, short
};
// The short list is taken while it makes at most two work-groups per CU.  (us, long
// list / short: L = 3, 16 pairs 16.8 / 14.1; L = 4, 300 20.3 / 16.9 (228
// work-groups); L = 5, 300 19.7 / 17.5 (380); above: L = 13, 48 24.3 / 26.8 (753);
// L = 3, 3000 18.6 / 22.8 (940).)
constexpr int64_t kDgShortMax = 2 * 256;

template <typename T> struct ChanArgs;

// HIP takes fewer than 2^32 work-items per launch, so a launch of many pairs at
// a low degree goes out in several: calls launch(first work-group, work-groups)
// until `total` work-groups, in rounds of `per`, are covered or a launch fails.
template <typename F>
int dir_launches(int64_t total, int64_t per, int threads, F&& launch) {
    const int64_t most = 0xffffffffLL / threads / per * per;
    for (int64_t first = 0; first < total; first += most) {
        const int64_t left = (total - first + per - 1) / per * per;
        const int err = launch(first, (unsigned)(left < most ? left : most));
        if (err) return err;
    }
    return 0;
}

int launch_direct_f32(const DirTables<float>& tb, const float* x1, const float* x2, float* out, int64_t N, int L,
                      const ChanArgs<float>* ch, bool real_basis, void* stream);
int launch_direct_f64(const DirTables<double>& tb, const double* x1, const double* x2, double* out, int64_t N, int L,
                      const ChanArgs<double>* ch, bool real_basis, void* stream);

int launch_direct_backward(const DgTables& tb, const float* x1, const float* x2, const float* g, float* gx1, float* gx2,
                           float* ws, int64_t N, int L, void* stream);
// The sums of the blocks' contributions (cgtp_backward.hip).
int launch_backward_sums(const float* ws, float* gx1, float* gx2, int64_t N, int L, void* stream);

}  // namespace cgtp
