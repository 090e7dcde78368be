// The packer of stb_pack on the GPU: Standardized Importance (Eq. 3), N:M mask (Sec. 3.1), residual binarisation of the
// kept salient weights (Eq. 4), break-point search and trisection of the kept non-salient ones (Alg. 2, Eq. 5-6), bit
// planes of STB1 in device memory.
//
// The result must agree with the host packer bit for bit.  Every value that is stored (scales, residuals) is computed by the same
// expression in the same order as there: float64, sums over a row's columns from left to right, no fused multiply-add
// (contraction is switched off for this file), and the three roundings of a scale (fp64 -> fp32 -> fp16) through the
// integer routine the host uses.  Choices (the mask of a layer, a block's break points) are made from sums in any order, in fp32
// where that suffices, with error bounds that prove them; what the bounds leave open is evaluated in the defined order, in
// which a sum over n rows is one lane's chain, fed by other wavefronts.  Importance per block takes the defined order throughout.
// Division and square root of float64 are correctly rounded on this hardware, as on the host.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <new>
#include <type_traits>
#include <vector>

#include "stb_f16.h"
#include "stb_internal.h"

#pragma clang fp contract(off)

namespace {

constexpr int CAND = 160;                  // break-point candidates of Alg. 2
constexpr int SH_COPIES = 16, LAYER_MASK_LDS = SH_COPIES * 257 * 4;      // copies of the tertile split's counts in LDS
constexpr int MK_ROWS = 256;               // rows of one block that a workgroup of the mask kernels takes
constexpr uint32_t ST_NONFINITE = 1u, ST_SALIENT = 2u, ST_GROUP = 4u, ST_UNDECIDED = 8u,
                   ST_CLOSE = 16u;         // a block's break points need the exact evaluation

struct PK {
    const float* W;
    const float* xnorm;
    const uint32_t* sal;
    int n, k, N, M, nb, nbS, per_block, region_mode, n_salient;
    uint8_t* mask;
    uint8_t* sign;
    uint8_t* region;
    uint32_t* res_sign;
    uint16_t* scales;
    uint16_t* res_scale;
    uint32_t* sal_out;
    uint32_t* prefix;
    int64_t mask_stride, sign_stride, region_stride, res_stride;
    uint32_t* status;       // [0] error bits, [1] [2] of k_layer_mean
    double* rs;             // [n][nbS] row sums of |W| (whole row, or per block)
    double2* cols;          // [k] column sums of |W| and their reciprocals
    double* rowacc;         // [n][nbS]
    double* stats;          // [nbS][2] mean, deviation (of the sums in the defined order)
    uint32_t* mxbits;       // [nb] largest kept non-salient magnitude of the block (fp32 bits)
    uint32_t* cnt;          // [nb] number of kept non-salient weights of the block
    double* p12;            // [nb][2] break points
    uint32_t* hist;         // [nb][2][256]
    uint32_t* sel;          // [nb][2][2] prefix, remaining rank of the two order statistics
};

// Whether an earlier kernel found what the host has to look at first: a wrong bitmap, numbers that are none, a mask or break points
// that the bounds leave open.
__device__ inline bool given_up(const PK& a) {
    return (__hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (ST_SALIENT | ST_NONFINITE | ST_UNDECIDED | ST_CLOSE)) != 0;
}

__device__ inline bool sal_bit(const uint32_t* bm, int j) { return (bm[j >> 5] >> (j & 31)) & 1u; }

// RN(x / d) for a divisor whose rounded reciprocal y = RN(1 / d) is at hand: after one correction the quotient is within an
// ulp, and then RN(q + r y) with the exact remainder r is the correctly rounded one (Markstein's theorem); 5 instructions
// instead of a division's 11.  d = 0 (with y = 0) only meets x = 0 and gives 0.  Magnitudes here are far from the ends of
// the float64 range: x is an fp32 or a difference of two quotients of fp32 sums.
__device__ inline double div_by(double x, double d, double y) {
    double q = x * y;
    q = __builtin_fma(__builtin_fma(-q, d, x), y, q);
    return __builtin_fma(__builtin_fma(-q, d, x), y, q);
}
__device__ inline double recip(double d) { return d > 0.0 ? 1.0 / d : 0.0; }

// ---- N:M mask from bounds (importance over the whole layer) -------------------------------------------------------------
// The mask needs the order of the scores s = (mu - mean) / sd * xnorm inside a group, not their values.  sd > 0 is common
// to all of them, the sums and the mean are within a few (n + k) roundings of their true values whatever the order of the
// additions, and the true mean of mu is (non-zero rows + non-zero columns) / (n k): every row's shares add up to 1, and
// every column's.  So sums in any order decide all groups in which no kept score is within the error bounds of a pruned one;
// a tie or a near-tie anywhere (ST_UNDECIDED) sends the layer through the sums in the defined order below.  Layers of
// continuous weights decide (of layers of normal weights the bounds left a group in 1 of 120 at 28672 x 8192 and at 8192 x 28672, in none of
// 200 at 8192 x 8192, in 1 of 300 at 11008 x 4096; the call then takes 2.96 ms instead of 1.26 at the first size); those of a single
// magnitude, whose scores are rounding errors, do not.
// 28672 x 8192: sums 0.19 ms and mask 0.20 (a pass over the weights takes 0.18 each), against 0.40 + 0.37 + 0.38 + 2 x 0.14 for
// the sums in order and 0.34 for the mask.
constexpr int FS_COLS = 1024, FS_BATCH = 8, FS_WGS = 768;        // (three workgroups a compute unit)

// Row and column sums of |w| in no defined order.  Workgroup = `rows` rows x 1024 columns, a thread 4 columns, the next 8 rows
// in flight; the rows are dealt so that the chip holds all workgroups at once (64 rows each, with nine times the
// additions in memory: 0.29 ms).
__global__ __launch_bounds__(256, 3) void k_layer_sums(PK a, int rows) {
    __shared__ double part[2][FS_BATCH * 256];
    if (__hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ST_UNDECIDED) return;       // (k_salient_tables')
    const int chunks = (a.k + FS_COLS - 1) / FS_COLS, tid = threadIdx.x;
    const int j = (int)(blockIdx.x % (unsigned)chunks) * FS_COLS + 4 * tid, i0 = (int)(blockIdx.x / (unsigned)chunks) * rows;
    const bool own = j < a.k;
    const float* w = a.W + (size_t)i0 * a.k + (own ? j : 0);
    double c0 = 0.0, c1 = 0.0, c2 = 0.0, c3 = 0.0;
    uint32_t top = 0;
    float4 v[FS_BATCH];
    auto load = [&](int b) {                               // the next FS_BATCH rows; b = the first, from i0
#pragma unroll
        for (int u = 0; u < FS_BATCH; u++) {
            v[u] = own && i0 + b + u < a.n ? *reinterpret_cast<const float4*>(w) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            w += a.k;
        }
    };
    load(0);
#pragma unroll 1
    for (int b = 0; b < rows && i0 + b < a.n; b += FS_BATCH) {
        double* const sums = part[(b / FS_BATCH) & 1];
#pragma unroll
        for (int u = 0; u < FS_BATCH; u++) {
            const float e[4] = {fabsf(v[u].x), fabsf(v[u].y), fabsf(v[u].z), fabsf(v[u].w)};
#pragma unroll
            for (int p = 0; p < 4; p++) top = __float_as_uint(e[p]) > top ? __float_as_uint(e[p]) : top;
            const double d0 = (double)e[0], d1 = (double)e[1], d2 = (double)e[2], d3 = (double)e[3];
            c0 += d0; c1 += d1; c2 += d2; c3 += d3;
            sums[u * 256 + tid] = (d0 + d1) + (d2 + d3);
        }
        if (b + FS_BATCH < rows) load(b + FS_BATCH);
        __syncthreads();                                   // (the sums before the last are read by then: two buffers)
        const int r = tid >> 5;
        double s = 0.0;
#pragma unroll
        for (int m = 0; m < 8; m++) s += sums[r * 256 + 32 * m + (tid & 31)];
#pragma unroll
        for (int d = 16; d > 0; d >>= 1) s += __shfl_xor(s, d);
        if ((tid & 31) == 0 && i0 + b + r < a.n) unsafeAtomicAdd(a.rs + i0 + b + r, s);
    }
    if (own) {
        unsafeAtomicAdd(&a.cols[j].x, c0); unsafeAtomicAdd(&a.cols[j + 1].x, c1);
        unsafeAtomicAdd(&a.cols[j + 2].x, c2); unsafeAtomicAdd(&a.cols[j + 3].x, c3);
    }
    if (top >= 0x7F800000u) atomicOr(a.status, ST_NONFINITE);              // an infinity or a NaN
}

// The numbers of non-zero rows and columns, from which the mean of mu follows (status[1]), the check of xnorm, and whether any sum or
// norm is of a size that fp32 scores could leave the fp32 range with (status[2]).  A thread a row or column (one workgroup: 21 us).
__global__ __launch_bounds__(256) void k_layer_mean(PK a) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    auto odd = [](double v) { return v != 0.0 && !(v >= 0x1p-40 && v <= 0x1p40); };
    bool nonzero = false, far = false, bad = false;
    if (i < a.n) {
        const double v = a.rs[i];
        nonzero = v != 0.0;
        far = odd(v);
    } else if (i < (int64_t)a.n + a.k) {
        const double v = a.cols[i - a.n].x;
        const float x = a.xnorm[i - a.n];
        nonzero = v != 0.0;
        far = odd(v) || odd((double)x);
        bad = !(x >= 0.0f) || !__builtin_isfinite(x);
    }
    const uint32_t count = (uint32_t)__popcll(__ballot(nonzero));
    const bool any_far = __any(far), any_bad = __any(bad);
    if ((threadIdx.x & 63) != 0) return;
    if (count) atomicAdd(a.status + 1, count);
    if (any_far) atomicOr(a.status + 2, 1u);
    if (any_bad) atomicOr(a.status, ST_NONFINITE);
}

// Which N of every M scores are kept (bit p of the result), the left one of equals first.
template <int M, typename T>
__device__ inline uint32_t rank_keep(const T (&s)[8], int N) {
    int better[8] = {0, 0, 0, 0, 0, 0, 0, 0};      // entries that rank before p: a higher score, or an equal one further left
#pragma unroll
    for (int p = 1; p < 8; p++)
#pragma unroll
        for (int o = p / M * M; o < p; o++) {
            const bool left = s[o] >= s[p];
            better[p] += left;
            better[o] += !left;
        }
    uint32_t byte = 0;
#pragma unroll
    for (int p = 0; p < 8; p++) byte |= better[p] < N ? 1u << p : 0u;
    return byte;
}

// The mask byte of 8 weights in float64, with the bounds: kept and pruned scores must differ by more than both errors, which
// are below (n + k + 16) 2^-50 x (mu + mean) each: sums of n or k terms and their mean are off by less than 2 (n + k) + 16
// roundings of 2^-53 in the defined order, and here.  Scores that are equal by definition (xnorm 0 for both, or weight 0 and
// the same norm) are ties in either order.
template <int M>
__device__ __forceinline__ uint32_t mask_byte_f64(const PK& a, const float (&e)[8], int i, int j0, double mean, bool& undecided) {
    double s[8], err[8];
    float x[8];
    const double rinv = recip(a.rs[i]), eta = (double)(a.n + a.k + 16) * 0x1p-50;
#pragma unroll
    for (int p = 0; p < 8; p++) {
        x[p] = a.xnorm[j0 + p];
        const double mu = (double)e[p] * (rinv + recip(a.cols[j0 + p].x));
        s[p] = (mu - mean) * (double)x[p];
        err[p] = (mu + mean) * (double)x[p] * eta;
    }
    const uint32_t byte = rank_keep<M>(s, a.N);
#pragma unroll
    for (int p = 0; p < 8; p++)
#pragma unroll
        for (int o = p / M * M; o < p / M * M + M; o++) {
            if (o == p) continue;
            const bool tie = x[o] == x[p] && (x[p] == 0.0f || (e[o] == 0.0f && e[p] == 0.0f));
            if ((byte >> p) & ~(byte >> o) & 1u) undecided |= !(s[p] - s[o] > err[p] + err[o]) && !tie;
        }
    return byte;
}

// The N-th and (N+1)-th largest of each M scores: Batcher's network, of which the compiler keeps what those two need.
template <int M, int N>
__device__ inline void around_cut(const float (&s)[8], int h, float& low, float& high) {
    float v[M];
#pragma unroll
    for (int p = 0; p < M; p++) v[p] = s[h + p];
    auto order = [&](int i, int j) { const float a = fmaxf(v[i], v[j]), b = fminf(v[i], v[j]); v[i] = a; v[j] = b; };
    if constexpr (M == 8) {
        order(0, 1); order(2, 3); order(4, 5); order(6, 7);
        order(0, 2); order(1, 3); order(4, 6); order(5, 7);
        order(1, 2); order(5, 6); order(0, 4); order(1, 5); order(2, 6); order(3, 7);
        order(2, 4); order(3, 5); order(1, 2); order(3, 4); order(5, 6);
    } else {
        order(0, 1); order(2, 3); order(0, 2); order(1, 3); order(1, 2);
    }
    low = v[N - 1];
    high = N < M ? v[N < M ? N : 0] : -__builtin_inff();
}

// A workgroup takes 256 rows of one block: 16 rows at a time, a thread 8 columns, whose column sums and norms stay in
// registers.  Scores in fp32, whose error is below 2^-20 xnorm (mu + mean): where the N-th largest of a group is further than
// both errors above the next, the scores not below it are kept; the few groups in a million where it is not are taken again
// in float64.  Also the largest kept non-salient magnitude and their number per block, and for the tertile split
// the counts of their leading bytes (k_select_hist's first pass, in LAYER_MASK_LDS bytes of dynamic LDS: 28672 x 8192 6:8 198 us without, 200 with them, against 219 for a pass of its own).
template <int M, int N>
__global__ __launch_bounds__(256) void k_layer_mask(PK a) {
    extern __shared__ uint32_t digits[];           // [SH_COPIES][257]
    const bool tertiles = a.region_mode != 0;
    // (the layer goes the other way: a wavefront by itself, or all of a workgroup that shares counts)
    if (tertiles ? __syncthreads_or(given_up(a)) != 0 : given_up(a)) return;
    uint32_t* const own = digits + (threadIdx.x & (SH_COPIES - 1)) * 257;
    if (tertiles) {
        for (int e = threadIdx.x; e < SH_COPIES * 257; e += 256) digits[e] = 0;
        __syncthreads();
    }
    const int q = (int)(blockIdx.x % (unsigned)a.nb), g = threadIdx.x & 15, r = threadIdx.x >> 4;
    const int ibeg = (int)(blockIdx.x / (unsigned)a.nb) * MK_ROWS + r, j0 = q * STB_BLOCK + 8 * g;
    const int iend = (int)(blockIdx.x / (unsigned)a.nb + 1) * MK_ROWS < a.n ? (int)(blockIdx.x / (unsigned)a.nb + 1) * MK_ROWS : a.n;
    const double mean = (double)a.status[1] / ((double)a.n * (double)a.k);
    const bool narrow = a.status[2] == 0;
    float x[8], cx[8], mx8[8], mxtop = 0.0f;       // xnorm, xnorm / column sum, mean * xnorm
    uint32_t normal[8];                            // all ones where the column is not salient
#pragma unroll
    for (int p = 0; p < 8; p++) {
        const float c = (float)a.cols[j0 + p].x;
        x[p] = a.xnorm[j0 + p];
        cx[p] = c > 0.0f ? x[p] * __builtin_amdgcn_rcpf(c) : 0.0f;
        mx8[p] = (float)mean * x[p];
        mxtop = fmaxf(mxtop, mx8[p]);
        normal[p] = sal_bit(a.sal, j0 + p) ? 0u : ~0u;
    }
    const uint32_t normal8 = ~(a.sal[j0 >> 5] >> (8 * (g & 3))) & 0xFFu;
    uint32_t mx = 0, members = 0, again = 0;       // again: rows (of the thread's 16) to take in float64
    float4 n0[2], n1[2];
    double nrs[2] = {0.0, 0.0};
    auto load = [&](int u, int i) {
        if (i >= iend) return;
        const float4* w = reinterpret_cast<const float4*>(a.W + (size_t)i * a.k + j0);
        n0[u] = w[0];
        n1[u] = w[1];
        nrs[u] = a.rs[i];
    };
    auto row = [&](int u, int i) {
        if (i >= iend) return;
        const float e[8] = {fabsf(n0[u].x), fabsf(n0[u].y), fabsf(n0[u].z), fabsf(n0[u].w), fabsf(n1[u].x), fabsf(n1[u].y), fabsf(n1[u].z), fabsf(n1[u].w)};
        const float rsum = (float)nrs[u], rinv = rsum > 0.0f ? __builtin_amdgcn_rcpf(rsum) : 0.0f;
        load(u, i + 32);
        float s[8], top = 0.0f, low[2], high[2];
#pragma unroll
        for (int p = 0; p < 8; p++) {
            s[p] = __builtin_fmaf(e[p], __builtin_fmaf(rinv, x[p], cx[p]), -mx8[p]);
            top = fmaxf(top, s[p]);
        }
        around_cut<M, N>(s, 0, low[0], high[0]);
        if constexpr (M == 4) around_cut<M, N>(s, 4, low[1], high[1]);
        else { low[1] = low[0]; high[1] = high[0]; }
        const float gap = fminf(low[0] - high[0], low[1] - high[1]);
        const bool sure = narrow && gap > 0x1p-19f * (top + 2.0f * mxtop);
        if (!sure) again |= 1u << ((i - ibeg) >> 4);
        uint32_t byte = 0;
#pragma unroll
        for (int p = 0; p < 8; p++) {
            const bool kept = s[p] >= (sure ? low[p / 4] : __builtin_nanf(""));       // (not sure: none, an infinite score neither)
            byte |= kept ? 1u << p : 0u;
            const uint32_t bits = kept ? __float_as_uint(e[p]) & normal[p] : 0u;      // magnitudes order like their bit patterns
            mx = bits > mx ? bits : mx;
        }
        if (tertiles) {
#pragma unroll
            for (int p = 0; p < 8; p++)
                if ((byte & normal8) >> p & 1u) atomicAdd(own + (__float_as_uint(e[p]) >> 24), 1u);
        }
        a.mask[(size_t)i * a.mask_stride + (j0 >> 3)] = (uint8_t)byte;
        members += (uint32_t)__popc(byte & normal8);
    };
    load(0, ibeg);
    load(1, ibeg + 16);
#pragma unroll 1
    for (int i = ibeg; i < iend; i += 32) {
        row(0, i);
        row(1, i + 16);
    }
    bool undecided = false;
    for (; again && !undecided; again &= again - 1) {      // (one group left open, and all of this is thrown away)
        const int i = ibeg + 16 * (__ffs(again) - 1);
        const float* w = a.W + (size_t)i * a.k + j0;
        float e[8];
#pragma unroll
        for (int p = 0; p < 8; p++) e[p] = fabsf(w[p]);
        const uint32_t byte = mask_byte_f64<M>(a, e, i, j0, mean, undecided);
#pragma unroll
        for (int p = 0; p < 8; p++) {
            const uint32_t bits = (byte >> p) & 1u ? __float_as_uint(e[p]) & normal[p] : 0u;
            mx = bits > mx ? bits : mx;
            if (tertiles && ((byte & normal8) >> p & 1u)) atomicAdd(own + (__float_as_uint(e[p]) >> 24), 1u);
        }
        a.mask[(size_t)i * a.mask_stride + (j0 >> 3)] = (uint8_t)byte;
        members += (uint32_t)__popc(byte & normal8);
    }
    if (undecided) atomicOr(a.status, ST_UNDECIDED);
    if (tertiles) {                                // both statistics start from the same counts
        __syncthreads();
        uint32_t sum = 0;
#pragma unroll
        for (int c = 0; c < SH_COPIES; c++) sum += digits[c * 257 + threadIdx.x];
        if (sum) {
            atomicAdd(a.hist + (size_t)q * 512 + threadIdx.x, sum);
            atomicAdd(a.hist + (size_t)q * 512 + 256 + threadIdx.x, sum);
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const uint32_t om = __shfl_xor(mx, d);
        mx = om > mx ? om : mx;
        members += __shfl_xor(members, d);
    }
    if ((threadIdx.x & 63) == 0) {
        if (mx) atomicMax(a.mxbits + q, mx);
        if (members) atomicAdd(a.cnt + q, members);
    }
}

// ---- Standardized Importance: sums in the defined order (importance per block, and layers that the bounds do not decide) ------------------------------------------------------------------------------
// A sum over a row (or column, or the rows' accumulators) is sequential by definition: one lane's chain.  So that nothing
// else is on that chain, four wavefronts of a workgroup load, convert and (for the sums of mu) divide into an LDS tile,
// and a fifth adds the tile before, a lane a row.  One barrier a tile.
constexpr int RC_ROWS = 32, RC_COLS = 64, RC_STRIDE = RC_COLS + 1;     // an odd row stride: the lanes of the chain meet different banks
constexpr int CC_COLS = 32, CC_ROWS = 64;                              // column sums: tile of 64 rows x 32 columns
constexpr int CHAIN_THREADS = 320;
constexpr int CHAIN_LDS0 = 2 * RC_ROWS * RC_STRIDE * 4;                // two tiles of fp32: the chain converts
constexpr int CHAIN_LDS = 2 * RC_ROWS * RC_STRIDE * 8;                 // two tiles of float64: four workgroups a compute unit
static_assert(2 * CC_ROWS * CC_COLS * 4 <= CHAIN_LDS0, "the column sums' tiles fit as well");

// MODE 0: sums of |w| (and the finiteness check); 1: of mu; 2: of (mu - mean)^2; over the row or, with per_block, over each
// block.  Workgroup = 32 rows; weights are loaded three tiles ahead, column sums one.  28672 x 8192: sums of |w| over rows and
// columns 0.40 ms, of mu 0.37, of (mu - mean)^2 0.38, against 0.95, 0.98 and 0.99 with a lane that loads and divides for its own
// chain (448 wavefronts on the chip, each waiting for its own loads and divisions).  Column c of a tile sits at position
// 16 (c % 4) + c / 4 of its LDS row: a producer has 4 columns in a row, and its lanes then write next to each other.
template <int MODE>
__device__ inline void row_chain(const PK& a, int wg, char* lds) {
    typedef typename std::conditional<MODE == 0, float, double>::type elem;
    elem* const buf = reinterpret_cast<elem*>(lds);
    const int tid = threadIdx.x, i0 = wg * RC_ROWS, tiles = a.k / RC_COLS;
    const bool chain = tid >= 256;
    const int lane = tid & 63, c = 4 * (tid & 15), r = tid >> 4;           // producers: 4 columns of rows r and r + 16
    const int ia = i0 + r < a.n ? i0 + r : a.n - 1, ib = i0 + r + 16 < a.n ? i0 + r + 16 : a.n - 1;
    const float* wa = a.W + (size_t)ia * a.k + c;
    const float* wb = a.W + (size_t)ib * a.k + c;
    float4 v[3][2];
    double2 col[4];                                                        // column sums and their reciprocals of the next tile
    double ra = 0.0, rb = 0.0, ya = 0.0, yb = 0.0, mean = 0.0, s = 0.0;
    bool bad = false;
    auto load_cols = [&](int t) {
        if (MODE == 0) return;
#pragma unroll
        for (int u = 0; u < 4; u++) col[u] = a.cols[t * RC_COLS + c + u];
    };
    auto load = [&](float4 (&d)[2], int t) {
        if (t >= tiles) return;
        d[0] = *reinterpret_cast<const float4*>(wa + t * RC_COLS);
        d[1] = *reinterpret_cast<const float4*>(wb + t * RC_COLS);
    };
    auto step = [&](float4 (&d)[2], int t) {
        if (!chain) {
            if (t < tiles) {
                const float fa[4] = {d[0].x, d[0].y, d[0].z, d[0].w}, fb[4] = {d[1].x, d[1].y, d[1].z, d[1].w};
                elem* da = buf + (t & 1) * (RC_ROWS * RC_STRIDE) + r * RC_STRIDE + (tid & 15);
                elem* db = da + 16 * RC_STRIDE;
                if (MODE == 0) {
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        bad |= !__builtin_isfinite(fa[u]) || !__builtin_isfinite(fb[u]);
                        da[16 * u] = (elem)fabsf(fa[u]);
                        db[16 * u] = (elem)fabsf(fb[u]);
                    }
                    load(d, t + 3);
                } else {
                    double2 cc[4];
#pragma unroll
                    for (int u = 0; u < 4; u++) cc[u] = col[u];
                    if (a.per_block && (t & 1) == 0) {
                        ra = a.rs[(size_t)ia * a.nbS + (t >> 1)]; rb = a.rs[(size_t)ib * a.nbS + (t >> 1)];
                        ya = recip(ra); yb = recip(rb);
                        if (MODE == 2) mean = a.stats[2 * (t >> 1)];
                    }
                    load_cols(t + 1 < tiles ? t + 1 : t);
                    load(d, t + 3);
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        double xa = fabs((double)fa[u]), xb = fabs((double)fb[u]);
                        xa = div_by(xa, ra, ya) + div_by(xa, cc[u].x, cc[u].y);
                        xb = div_by(xb, rb, yb) + div_by(xb, cc[u].x, cc[u].y);
                        if (MODE == 2) {
                            xa -= mean; xb -= mean;
                            xa *= xa; xb *= xb;
                        }
                        da[16 * u] = xa;
                        db[16 * u] = xb;
                    }
                }
            }
        } else if (t > 0 && t <= tiles && lane < RC_ROWS) {
            const elem* x = buf + ((t - 1) & 1) * (RC_ROWS * RC_STRIDE) + lane * RC_STRIDE;
#pragma unroll
            for (int u = 0; u < RC_COLS; u++) s += (double)x[16 * (u & 3) + (u >> 2)];
            if (i0 + lane < a.n) {
                double* out = MODE == 0 ? a.rs : a.rowacc;
                if (a.per_block) {
                    if ((t & 1) == 0) { out[(size_t)(i0 + lane) * a.nbS + (t >> 1) - 1] = s; s = 0.0; }
                } else if (t == tiles) out[i0 + lane] = s;
            }
        }
        __syncthreads();
    };
    if (!chain) {
        load_cols(0);
        load(v[0], 0);
        load(v[1], 1);
        load(v[2], 2);
        if (MODE >= 1 && !a.per_block) {
            ra = a.rs[ia]; rb = a.rs[ib];
            ya = recip(ra); yb = recip(rb);
        }
        if (MODE == 2 && !a.per_block) mean = a.stats[0];
    }
    for (int t = 0; t <= tiles; t += 3) {
        step(v[0], t);
        step(v[1], t + 1);
        step(v[2], t + 2);
    }
    if (MODE == 0 && bad) atomicOr(a.status, ST_NONFINITE);
}

// Sums of |w| over 32 columns, from the top row down; also their reciprocals, and the check of xnorm.  Six tiles of 8 KB
// are in flight per workgroup: with about one such workgroup a compute unit the loads need that much.
__device__ inline void col_chain(const PK& a, int wg, char* lds) {
    constexpr int AHEAD = 6;
    float* const buf = reinterpret_cast<float*>(lds);
    const int tid = threadIdx.x, j0 = wg * CC_COLS, tiles = (a.n + CC_ROWS - 1) / CC_ROWS;
    const bool chain = tid >= 256;
    const int lane = tid & 63, c = 4 * (tid & 7), r = tid >> 3;            // producers: 4 columns of rows r and r + 32
    const float* w = a.W + j0 + c;
    float4 v[AHEAD][2];
    auto load = [&](float4 (&d)[2], int t) {
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int i = t * CC_ROWS + r + 32 * u;
            d[u] = i < a.n ? *reinterpret_cast<const float4*>(w + (size_t)i * a.k) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    };
    double s = 0.0;
    auto step = [&](float4 (&d)[2], int t) {
        if (!chain) {
            if (t < tiles) {
                float* x = buf + (t & 1) * (CC_ROWS * CC_COLS) + r * CC_COLS + c;
                *reinterpret_cast<float4*>(x) = d[0];
                *reinterpret_cast<float4*>(x + 32 * CC_COLS) = d[1];
                load(d, t + AHEAD);                                        // (rows past the end are not touched)
            }
        } else if (t > 0 && t <= tiles && lane < CC_COLS) {
            const float* x = buf + ((t - 1) & 1) * (CC_ROWS * CC_COLS) + lane;
            // (rows past the last are zeros, and adding a zero to a sum that is not negative changes nothing)
#pragma unroll
            for (int u = 0; u < CC_ROWS; u++) s += fabs((double)x[u * CC_COLS]);
        }
        __syncthreads();
    };
    if (!chain) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) load(v[u], u);
    }
    for (int t = 0; t <= tiles; t += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) step(v[u], t + u);
    }
    if (chain && lane < CC_COLS) {
        const int j = j0 + lane;
        a.cols[j] = make_double2(s, recip(s));
        const float x = a.xnorm[j];
        if (!(x >= 0.0f) || !__builtin_isfinite(x)) atomicOr(a.status, ST_NONFINITE);
    }
}

// Column sums and row sums in one launch: the few long column chains (n additions each) start first and run beside the rows.
__global__ __launch_bounds__(CHAIN_THREADS) void k_abs_sums(PK a) {
    __shared__ __attribute__((aligned(16))) char lds[CHAIN_LDS0];
    const int cols = a.k / CC_COLS;
    if ((int)blockIdx.x < cols) col_chain(a, blockIdx.x, lds);
    else row_chain<0>(a, (int)blockIdx.x - cols, lds);
}

template <int MODE>
__global__ __launch_bounds__(CHAIN_THREADS) void k_mu_sums(PK a) {
    __shared__ __attribute__((aligned(16))) char lds[CHAIN_LDS];
    row_chain<MODE>(a, blockIdx.x, lds);
}

// One wavefront per scope (the layer, or a block): the row accumulators from the top row down.  MODE 0 -> mean, 1 -> deviation.
// The next 512 values load while the lanes (all alike) add the 512 in LDS: with one lane that loaded for itself the layer's
// 28672 additions took 395 us (now 137).
constexpr int TOT_CHUNK = 512;
template <int MODE>
__global__ __launch_bounds__(64) void k_total(PK a) {
    __shared__ double buf[TOT_CHUNK];
    const int sc = blockIdx.x, lane = threadIdx.x;
    const double* x = a.rowacc + sc;
    double v[TOT_CHUNK / 64], tot = 0.0;
    auto load = [&](int i0) {
#pragma unroll
        for (int u = 0; u < TOT_CHUNK / 64; u++) {
            const int i = i0 + 64 * u + lane;
            v[u] = i < a.n ? x[(size_t)i * a.nbS] : 0.0;                   // (zeros past the end change no sum)
        }
    };
    load(0);
    for (int i0 = 0; i0 < a.n; i0 += TOT_CHUNK) {
#pragma unroll
        for (int u = 0; u < TOT_CHUNK / 64; u++) buf[64 * u + lane] = v[u];
        __syncthreads();
        if (i0 + TOT_CHUNK < a.n) load(i0 + TOT_CHUNK);
#pragma unroll 64
        for (int u = 0; u < TOT_CHUNK; u++) tot += buf[u];
        __syncthreads();
    }
    if (lane != 0) return;
    const double cnt = (double)a.n * (double)(a.per_block ? STB_BLOCK : a.k);
    if (MODE == 0) a.stats[2 * sc] = tot / cnt;
    else {
        double sd = sqrt(tot / cnt);
        if (sd == 0.0) sd = 1.0;
        a.stats[2 * sc + 1] = sd;
    }
}

// ---- N:M mask, largest kept non-salient magnitude and their number per block -------------------------------------------
// A workgroup takes 256 rows of one block: 16 rows at a time, a thread 8 columns, whose column sums and norms stay in
// registers.  Of each pair the entry with the higher score, or the left one of equals, counts against the other; the N
// entries of a group with the fewest counts are kept.  28672 x 8192: 0.34 ms (0.96 with a thread that
// fetches everything for its 8 columns), with the maxima and counts that a second
// pass over the weights took 990 us for (one thread a row and block, each walking its own 512 bytes).
template <int M>
__global__ __launch_bounds__(256) void k_mask(PK a) {
    const int q = (int)(blockIdx.x % (unsigned)a.nb), g = threadIdx.x & 15, r = threadIdx.x >> 4;
    const int ibeg = (int)(blockIdx.x / (unsigned)a.nb) * MK_ROWS + r, j0 = q * STB_BLOCK + 8 * g, sc = a.per_block ? q : 0;
    const int iend = (int)(blockIdx.x / (unsigned)a.nb + 1) * MK_ROWS < a.n ? (int)(blockIdx.x / (unsigned)a.nb + 1) * MK_ROWS : a.n;
    const double mean = a.stats[2 * sc], sd = a.stats[2 * sc + 1], sinv = 1.0 / sd;
    double2 col[8];
    float xn[8];
#pragma unroll
    for (int p = 0; p < 8; p++) { col[p] = a.cols[j0 + p]; xn[p] = a.xnorm[j0 + p]; }
    const uint32_t normal = ~(a.sal[j0 >> 5] >> (8 * (g & 3))) & 0xFFu;
    uint32_t mx = 0, members = 0;
    float4 n0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), n1 = n0;
    double nrs = 0.0;
    auto load = [&](int i) {
        if (i >= iend) return;
        const float4* w = reinterpret_cast<const float4*>(a.W + (size_t)i * a.k + j0);
        n0 = w[0];
        n1 = w[1];
        nrs = a.rs[(size_t)i * a.nbS + sc];
    };
    load(ibeg);
    for (int i = ibeg; i < iend; i += 16) {
        const float e[8] = {fabsf(n0.x), fabsf(n0.y), fabsf(n0.z), fabsf(n0.w), fabsf(n1.x), fabsf(n1.y), fabsf(n1.z), fabsf(n1.w)};
        const double rsv = nrs, rinv = recip(rsv);
        load(i + 16);
        double s[8];
#pragma unroll
        for (int p = 0; p < 8; p++) {
            const double av = (double)e[p];
            const double mu = div_by(av, rsv, rinv) + div_by(av, col[p].x, col[p].y);
            s[p] = div_by(mu - mean, sd, sinv) * (double)xn[p];
        }
        const uint32_t byte = rank_keep<M>(s, a.N);
        a.mask[(size_t)i * a.mask_stride + (j0 >> 3)] = (uint8_t)byte;
        const uint32_t kept = byte & normal;
        members += (uint32_t)__popc(kept);
#pragma unroll
        for (int p = 0; p < 8; p++) {
            const uint32_t bits = (kept >> p) & 1u ? __float_as_uint(e[p]) : 0u;     // magnitudes order like their bit patterns
            mx = bits > mx ? bits : mx;
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const uint32_t om = __shfl_xor(mx, d);
        mx = om > mx ? om : mx;
        members += __shfl_xor(members, d);
    }
    if ((threadIdx.x & 63) == 0) {
        if (mx) atomicMax(a.mxbits + q, mx);
        if (members) atomicAdd(a.cnt + q, members);
    }
}

// ---- break-point search (Alg. 2 NonSalientAwareQuant) --------------------------------------------------------------
__device__ inline void candidate(int t, double mx, double& q1, double& q2, bool& skip) {
    const double step = (0.9 - 0.1) / 159.0;
    const double c = (t == CAND - 1) ? 0.9 : (double)t * step + 0.1;
    q1 = c * mx;
    q2 = 2.0 * q1;
    skip = q2 > 0.9 * mx;
}

// The chosen candidate is the first strict minimum of D_t = the sequential float64 sum, over the rows, of the squared errors
// of binarising the row's three regions separately (Eq. 5-6).  Evaluating D_t in that order for all candidates costs 2
// passes over 128 values per (row, block, candidate): 18.8 ms of errors and 2.9 ms of sums on a 28672 x 8192 layer.  But
// sum (a - mean)^2 = sum a^2 - (sum a)^2 / count, so the candidate with the smallest error is the one with the largest
//     G_t = sum over rows and regions of (sum a)^2 / count,
// and all G_t of a (row, block) follow from the suffix sums of one histogram over the 140 sorted break points p1(t) and
// p2(t) = 2 p1(t).  k_search_gain computes G_t with a proven error bound; k_search_narrow keeps the candidates that
// could still be the minimum of D_t: almost always one, and then it is the answer.  Of candidates that part the block's values
// alike, which have the same D_t bit for bit, the first is kept: the numbers of values above p1(t) and p2(t) fall with t, so two
// candidates are alike where their sums are equal.  (Without that a layer of few distinct magnitudes evaluates all that tie:
// 11008 x 4096 4:8 of one magnitude 7.6 ms, now 1.0; of two 7.7 and 1.8; 28672 x 8192 of 15 9.3 and 3.2.)  Where several are left
// k_exact_errors / k_exact_pick evaluate D_t for those alone, in the defined order.
constexpr int SC_NV = 70;                  // candidates that are not skipped when the block has a non-zero weight: 2 c_t <= 0.9
constexpr int SC_ROWS = 64;                // rows of a workgroup whose histograms are in LDS at a time, 8 a wavefront
constexpr int SC_WAVES = 8;
constexpr int SC_STEPS = 8;                // ... and how often at most: rows per workgroup = SC_ROWS * steps
constexpr int SC_SEG = 19;                 // bins per lane of the suffix sums (8 lanes a row; odd: their 8 x 8 first bins lie in all banks)
constexpr int SC_BINS = 8 * SC_SEG;        // bin b: the value exceeds b of the 2 SC_NV break points (141 bins)
constexpr int SC_MASKW = 8;                // words of a block's candidate mask (CAND bits)

// LDS keeps a wavefront's accesses in order; the compiler has to as well where lanes read what others wrote.
__device__ inline void wave_order() {
    asm volatile("" : : : "memory");
    __builtin_amdgcn_wave_barrier();
}

// The largest fp32 not above p >= 0: for an fp32 value a, a > p iff a > that.
__device__ inline float round_down_f32(double p) {
    const float f = (float)p;
    return (double)f > p ? __uint_as_float(__float_as_uint(f) - 1u) : f;
}

// The break points in ascending order.  In steps of the candidates' grid p1(t) lies at 19.875 + t and p2(t) at 39.75 + 2 t, an
// eighth of a step apart at least, and rounding keeps an order (it can only make neighbours equal): their ranks among all
// 2 SC_NV are known.
__device__ constexpr int rank_p1(int t) { return t + (t < 20 ? 0 : (t - 18) >> 1); }
__device__ constexpr int rank_p2(int t) { return t + (2 * t + 20 < SC_NV ? 2 * t + 20 : SC_NV); }

// Number of the ascending break points that a exceeds; tau[0] = -1, tau[b + 1] = break point b, tau[2 SC_NV + 1] = inf.
// The guess comes from the spacing of the break points, in fp32: its error is below 160 * 2^-22 steps; `go` is 2^-10 steps too
// high, so it is the number itself or one more.  TINY: the block's magnitudes are so
// small that the spacing itself may be lost; then the loops walk as far as it takes and end at the ends of the table.
template <bool TINY>
__device__ inline int search_bin(float a, float gs, float go, const float* tau) {
    const float g1 = __builtin_amdgcn_fmed3f(__builtin_fmaf(a, gs, go), 0.0f, (float)SC_NV);
    const float g2 = __builtin_amdgcn_fmed3f(__builtin_fmaf(a, 0.5f * gs, go), 0.0f, (float)SC_NV);
    int g = (int)g1 + (int)g2;
    if (TINY) {
        while (g > 0 && !(a > tau[g])) g--;
        while (g < 2 * SC_NV && a > tau[g + 1]) g++;
        return g;
    }
    return g - (a <= tau[g]);              // (tau[0] is below everything)
}

// A workgroup takes SC_ROWS * steps rows of one block, a wavefront 8 of every 64: it bins them (magnitudes as 36-bit fractions of the block's
// largest, the count in bits 44 up: one 64-bit LDS atomic a value) into histograms of its own, [bin][row], takes 19 bins of a row a lane for
// the suffix sums, and every eighth candidate of a row a lane, whose G_t it keeps in a register.  Nothing in the loop waits for another
// wavefront, so that the vector instructions of some run beside the LDS accesses of others.  The next step's weights load meanwhile.
// Error bound, with K = count * mx^2 >= sum a^2 and u = 2^-53: the fractions move G_t by at most 2^-36 K, float64
// rounding of G_t and of D_t (sequential sums over n rows of sums over 128 values) by less than (4 n + 200) u K.
// A load instruction covers 8 rows x 128 bytes, so that few lanes of one atomic instruction share a row's bin (with 2 rows
// x 512 bytes and a histogram for either break point: 1281 us).  Bound by vector instructions and LDS accesses.
// 28672 x 8192 at 4:8: 0.40 ms; 0.44 with the histograms of 64 rows shared by eight wavefronts, five barriers a step (each pipe busy for about
// half of the time); 0.82 with 32 rows a step, suffix sums by 128 of 320 threads and a lane a candidate, which meet in
// banks; 1.14 with loops around every bin search; 21.7 for evaluating every candidate in the defined order.
__global__ __launch_bounds__(64 * SC_WAVES, 4) void k_search_gain(PK a, int steps, double* __restrict__ gain, unsigned long long* __restrict__ above) {
    __shared__ __attribute__((aligned(16))) unsigned long long hists[SC_WAVES][SC_BINS * 8];   // a wavefront's: [bin][row]
    __shared__ double inv[256];            // 1 / count (a count is at most 128; 8 bits are read)
    __shared__ float tau[2 * SC_NV + 2];
    constexpr int PER = (SC_NV + 7) / 8;
    __shared__ uint32_t where[8 * PER];    // where a candidate's suffix sums are: p1(t) below, p2(t) in bits 16 up (9 registers a lane otherwise)
    if (given_up(a)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = (int)(blockIdx.x % (unsigned)a.nb), chunk = (int)(blockIdx.x / (unsigned)a.nb);
    const float mxf = __uint_as_float(a.mxbits[q]);
    if (mxf == 0.0f) return;               // nothing kept and non-salient, or all zero: every candidate is the same
    const double mx = (double)mxf;
    const int r0 = tid >> 3;
    float4 v[4];
    uint32_t m[4];
    auto load = [&](int i) {
        if (i >= a.n) i = a.n - 1;         // (counted for rows of the matrix only)
        const uint4 m4 = *reinterpret_cast<const uint4*>(a.mask + (size_t)i * a.mask_stride + 16 * q);
        const float4* w4 = reinterpret_cast<const float4*>(a.W + (size_t)i * a.k + q * STB_BLOCK);
#pragma unroll
        for (int it = 0; it < 4; it++) v[it] = w4[8 * it + (tid & 7)];
        m[0] = m4.x; m[1] = m4.y; m[2] = m4.z; m[3] = m4.w;
    };
    const int first = chunk * steps * SC_ROWS;
    load(first + r0);
    if (tid < SC_NV) {
        double p1, p2;
        bool skip;
        candidate(tid, mx, p1, p2, skip);
        tau[rank_p1(tid) + 1] = round_down_f32(p1);
        tau[rank_p2(tid) + 1] = round_down_f32(p2);
    }
    if (tid < 8 * PER) {
        const int t = tid < SC_NV ? tid : SC_NV - 1;
        where[tid] = (uint32_t)((rank_p1(t) + 1) * 8 | (rank_p2(t) + 1) * 8 << 16);
    }
    if (tid == 0) { tau[0] = -1.0f; tau[2 * SC_NV + 1] = __builtin_inff(); }
    if (tid < 256) inv[tid] = tid > 0 ? 1.0 / (double)tid : 0.0;
    uint32_t sal[4];
#pragma unroll
    for (int it = 0; it < 4; it++) sal[it] = a.sal[4 * q + it];
    const double scale = 68719476736.0 / mx;                   // 2^36
    const double step = (0.9 - 0.1) / 159.0;
    const bool tiny = !(mxf > 1e-30f);     // (or not a number: the loops end all the same)
    const float gs = (float)(1.0 / (step * mx)), go = (float)(1.0 + 0.0009765625 - 0.1 / step);
    double g_t[PER];
    uint32_t n_t[PER];                     // 8 x the values above p1(t) and above p2(t)
#pragma unroll
    for (int j = 0; j < PER; j++) { g_t[j] = 0.0; n_t[j] = 0; }
    unsigned long long* const hist = hists[wave];
    unsigned long long* const bins = hist + (lane >> 3);       // of the row whose weights the lane holds
    // the row and the part of its bins and candidates that the lane takes (8 rows next to each other: in the
    // suffix sums no two lanes share a bank; the candidates' reads, whose bins repeat modulo 4, do)
    const int part = lane >> 3;
    unsigned long long* const row = hist + (lane & 7);
    __syncthreads();
    for (int st = 0; st < steps; st++) {
        const int i0 = first + st * SC_ROWS;
        if (i0 + 8 * wave >= a.n) break;                       // uniform
#pragma unroll
        for (int e = 0; e < SC_BINS * 4; e += 64)
            if (e + 64 <= SC_BINS * 4 || lane < SC_BINS * 4 - e) reinterpret_cast<uint4*>(hist)[e + lane] = make_uint4(0u, 0u, 0u, 0u);
        wave_order();
        const bool live = i0 + r0 < a.n;
        auto count = [&](auto any_size) {
#pragma unroll
            for (int it = 0; it < 4; it++) {
                const uint32_t keep = live ? (m[it] & ~sal[it]) >> (4 * (tid & 7)) : 0u;
                const float e[4] = {fabsf(v[it].x), fabsf(v[it].y), fabsf(v[it].z), fabsf(v[it].w)};
                int b[4];
                unsigned long long fx[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    b[u] = search_bin<decltype(any_size)::value>(e[u], gs, go, tau);
                    // 2^52 + the fraction, rounded to a whole number: its low words are that number below 2^52's exponent
                    fx[u] = (unsigned long long)__double_as_longlong(__builtin_fma((double)e[u], scale, 4503599627370496.0)) - (0x4330000000000000ull - (1ull << 44));
                }
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if ((keep >> u) & 1u) atomicAdd(&bins[b[u] * 8], fx[u]);
            }
        };
        if (tiny) count(std::true_type{});
        else count(std::false_type{});
        if (st + 1 < steps) load(i0 + SC_ROWS + r0);
        wave_order();
        {
            unsigned long long h[SC_SEG], run = 0;
#pragma unroll
            for (int b = 0; b < SC_SEG; b++) { h[b] = row[(part * SC_SEG + b) * 8]; run += h[b]; }
            // the sums of the parts behind the lane's
            unsigned long long all = run;
#pragma unroll
            for (int d = 8; d < 64; d <<= 1) {
                const unsigned long long next = __shfl_down(all, d);
                if (lane + d < 64) all += next;
            }
            run = all - run;
#pragma unroll
            for (int b = SC_SEG - 1; b >= 0; b--) { run += h[b]; row[(part * SC_SEG + b) * 8] = run; }
        }
        wave_order();
        // the low 44 bits as a double (whole numbers: their differences are exact) and 8 x the count
        auto sum_of = [](unsigned long long s) {
            return __longlong_as_double((long long)((s & 0xFFFFFFFFFFFull) | 0x4330000000000000ull)) - 4503599627370496.0;
        };
        auto count_of = [](unsigned long long s) { return ((uint32_t)(s >> 32) >> 9) & (255u << 3); };
        auto inv_of = [&](uint32_t c8) { return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(inv) + c8); };
        const unsigned long long all = row[0];
        const double all_sum = sum_of(all);
        const uint32_t all_n = count_of(all);
#pragma unroll
        for (int j = 0; j < PER; j++) {                        // (lanes past the last candidate take that one once more)
            const uint32_t at = where[part + 8 * j];
            const unsigned long long above1 = row[at & 0xFFFFu], above2 = row[at >> 16];
            const double s1 = sum_of(above1), s2 = sum_of(above2), low = all_sum - s1, mid = s1 - s2;
            const uint32_t n1 = count_of(above1), n2 = count_of(above2);
            n_t[j] += n1 + n2;
            g_t[j] = __builtin_fma(s2 * s2, inv_of(n2), __builtin_fma(mid * mid, inv_of(n1 - n2), __builtin_fma(low * low, inv_of(all_n - n1), g_t[j])));
        }
        wave_order();
    }
#pragma unroll
    for (int j = 0; j < PER; j++) {
        const int t = part + 8 * j;
        double g = g_t[j];
        uint32_t cnt = n_t[j] >> 3;
#pragma unroll
        for (int d = 4; d > 0; d >>= 1) { g += __shfl_xor(g, d); cnt += __shfl_xor(cnt, d); }
        if ((lane & 7) == 0 && t < SC_NV) {                    // in units of (mx / 2^36)^2
            unsafeAtomicAdd(gain + (size_t)q * SC_NV + t, g);
            atomicAdd(above + (size_t)q * SC_NV + t, (unsigned long long)cnt);
        }
    }
}

// A wavefront per block, two candidates a lane: those whose G_t is within the error bounds (taken four times over) of the largest, the first of
// those that part the values alike.  One left: it is the answer.  Several: their bits go to the block's mask for the exact
// evaluation.
__global__ __launch_bounds__(64) void k_search_narrow(PK a, const double* __restrict__ gain, const unsigned long long* __restrict__ above, uint32_t* __restrict__ left) {
    const int q = blockIdx.x, lane = threadIdx.x;
    uint32_t* mask = left + (size_t)q * SC_MASKW;
    const double mx = (double)__uint_as_float(a.mxbits[q]);
    if (mx == 0.0 && lane < SC_MASKW) mask[lane] = 0;
    if (lane == 0) a.p12[2 * q] = a.p12[2 * q + 1] = 0.0;      // candidate 0 of a block without a non-zero weight
    if (mx == 0.0) return;
    const bool two = lane + 64 < SC_NV;
    const double g0 = gain[(size_t)q * SC_NV + lane], g1 = two ? gain[(size_t)q * SC_NV + 64 + lane] : 0.0;
    double best = g0 > g1 ? g0 : g1;
    best = best > 0.0 ? best : 0.0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const double o = __shfl_xor(best, d);
        best = o > best ? o : best;
    }
    const double K = (double)a.cnt[q] * 4722366482869645213696.0;                                  // 2^72
    const double slack = 4.0 * (1.0 / 68719476736.0 + (4.0 * (double)a.n + 200.0) / 9007199254740992.0) * K;
    unsigned long long close0 = __ballot(g0 >= best - slack), close1 = __ballot(two && g1 >= best - slack);
    int many = 0, first = 0;
    unsigned long long kept = 0;
    uint32_t bits[3] = {0u, 0u, 0u};
    while (close0 | close1) {                                  // (almost always once)
        const int t = close0 ? __ffsll(close0) - 1 : 63 + __ffsll(close1);
        if (close0) close0 &= close0 - 1; else close1 &= close1 - 1;
        const unsigned long long n = above[(size_t)q * SC_NV + t];
        if (many > 0 && n == kept) continue;
        if (many++ == 0) first = t;
        kept = n;
#pragma unroll
        for (int u = 0; u < 3; u++) bits[u] |= t >> 5 == u ? 1u << (t & 31) : 0u;
    }
    if (lane < SC_MASKW) mask[lane] = many == 1 ? 0u : lane == 0 ? bits[0] : lane == 1 ? bits[1] : lane == 2 ? bits[2] : 0u;
    if (lane == 0 && many > 1) atomicOr(a.status, ST_CLOSE);
    if (lane == 0 && many == 1) {
        bool skip;
        candidate(first, mx, a.p12[2 * q], a.p12[2 * q + 1], skip);
    }
}

// The exact errors of the remaining candidates.  list[e] = block << 8 | candidate, the entries of a block next to each other;
// first[b] .. first[b + 1] = the entries of the b-th block of the launch.  A workgroup stages 64 rows of the block
// (magnitudes of the kept non-salient weights, -1 elsewhere) and its wavefronts take one candidate after another, a lane
// a row: the row's kept magnitudes from left to right, as the definition has it.  err[e][i] = the row's error.
__global__ __launch_bounds__(256) void k_exact_errors(PK a, const uint32_t* __restrict__ list, const uint32_t* __restrict__ first,
                                                      double* __restrict__ err) {
    __shared__ float tile[64][STB_BLOCK + 1];
    const uint32_t e0 = first[blockIdx.y], e1 = first[blockIdx.y + 1];
    const int q = (int)(list[e0] >> 8), i0 = (int)blockIdx.x * 64, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int v = threadIdx.x; v < 64 * STB_BLOCK; v += 256) {
        const int r = v / STB_BLOCK, c = v % STB_BLOCK, i = i0 + r;
        float m = -1.0f;
        if (i < a.n && ((a.mask[(size_t)i * a.mask_stride + 16 * q + (c >> 3)] >> (c & 7)) & 1u) && !sal_bit(a.sal, q * STB_BLOCK + c))
            m = fabsf(a.W[(size_t)i * a.k + q * STB_BLOCK + c]);
        tile[r][c] = m;
    }
    __syncthreads();
    const double mx = (double)__uint_as_float(a.mxbits[q]);
    for (uint32_t e = e0 + wave; e < e1; e += 4) {
        double p1, p2;
        bool skip;
        candidate((int)(list[e] & 255u), mx, p1, p2, skip);
        double sum0 = 0.0, sum1 = 0.0, sum2 = 0.0;
        int n0 = 0, n1 = 0, n2 = 0;
        for (int c = 0; c < STB_BLOCK; c++) {
            const double av = (double)tile[lane][c];
            if (av < 0.0) continue;
            if (av > p2) { sum2 += av; n2++; }
            else if (av > p1) { sum1 += av; n1++; }
            else { sum0 += av; n0++; }
        }
        const double al0 = n0 > 0 ? sum0 / (double)n0 : 0.0;
        const double al1 = n1 > 0 ? sum1 / (double)n1 : 0.0;
        const double al2 = n2 > 0 ? sum2 / (double)n2 : 0.0;
        double row = 0.0;
        for (int c = 0; c < STB_BLOCK; c++) {
            const double av = (double)tile[lane][c];
            if (av < 0.0) continue;
            const double d = av - (av > p2 ? al2 : (av > p1 ? al1 : al0));
            row += d * d;
        }
        if (i0 + lane < a.n) err[(size_t)e * a.n + i0 + lane] = row;
    }
}

// One workgroup per block: a wavefront per entry adds the rows' errors from the top row down (64 loaded together, added in
// order by every lane alike), then the first strict minimum over the candidates in their order.
__global__ __launch_bounds__(1024) void k_exact_pick(PK a, const uint32_t* __restrict__ list, const uint32_t* __restrict__ first,
                                                     const double* __restrict__ err) {
    __shared__ double tot[CAND];
    const uint32_t e0 = first[blockIdx.x], e1 = first[blockIdx.x + 1];
    const int q = (int)(list[e0] >> 8), lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t e = e0 + wave; e < e1; e += 16) {
        const double* row = err + (size_t)e * a.n;
        double s = 0.0, next = lane < a.n ? row[lane] : 0.0;
        for (int i0 = 0; i0 < a.n; i0 += 64) {
            const double cur = next;
            next = i0 + 64 + lane < a.n ? row[i0 + 64 + lane] : 0.0;
            const int m = a.n - i0 < 64 ? a.n - i0 : 64;
            for (int l = 0; l < m; l++) s += __shfl(cur, l);
        }
        if (lane == 0) tot[e - e0] = s;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double mx = (double)__uint_as_float(a.mxbits[q]);
    double best = __builtin_inf(), b1 = 0.0, b2 = 0.0, p1, p2;
    bool skip;
    for (uint32_t e = e0; e < e1; e++)
        if (tot[e - e0] < best) {
            candidate((int)(list[e] & 255u), mx, p1, p2, skip);
            best = tot[e - e0]; b1 = p1; b2 = p2;
        }
    a.p12[2 * q] = b1;
    a.p12[2 * q + 1] = b2;
}

// ---- tertile split (region_mode 1): two order statistics per block by radix selection on the fp32 bit patterns ----
// sel[q][s] = {bits fixed so far, rank still to find among the values that share them}
__global__ void k_select_init(PK a) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= a.nb) return;
    const uint32_t m = a.cnt[q];
    a.sel[4 * q + 0] = 0; a.sel[4 * q + 1] = m ? (m + 2) / 3 - 1 : 0;
    a.sel[4 * q + 2] = 0; a.sel[4 * q + 3] = m ? (uint32_t)((2ull * m + 2) / 3 - 1) : 0;
}

// Counts, for both statistics, the next 8 bits of the values whose higher bits match.  A workgroup takes 256 rows of one
// block (a thread 8 columns of every 16th row) and counts in LDS, in 16 copies that lanes next to each other do not share
// (a block's magnitudes have few leading bytes); only its sums go to memory.  5120 x 8704: 0.21 ms for the four passes; 5120 x 13824 took
// 12.5 ms with an atomic in memory for every value.
constexpr int SH_STRIDE = 2 * 256 + 1;
__global__ __launch_bounds__(256) void k_select_hist(PK a, int pass) {
    __shared__ uint32_t h[SH_COPIES * SH_STRIDE];
    if (given_up(a)) return;
    const int q = (int)(blockIdx.x % (unsigned)a.nb), i0 = (int)(blockIdx.x / (unsigned)a.nb) * MK_ROWS, g = threadIdx.x & 15;
    const int iend = a.n - i0 < MK_ROWS ? a.n : i0 + MK_ROWS;
    for (int e = threadIdx.x; e < SH_COPIES * SH_STRIDE; e += 256) h[e] = 0;
    __syncthreads();
    uint32_t* const own = h + (threadIdx.x & (SH_COPIES - 1)) * SH_STRIDE;
    const int shift = 24 - 8 * pass, j0 = q * STB_BLOCK + 8 * g;
    const uint32_t pre0 = a.sel[4 * q + 0], pre1 = a.sel[4 * q + 2];
    const uint32_t normal = ~(a.sal[j0 >> 5] >> (8 * (g & 3))) & 0xFFu;
#pragma unroll 2
    for (int i = i0 + (threadIdx.x >> 4); i < iend; i += 16) {
        const float4* w4 = reinterpret_cast<const float4*>(a.W + (size_t)i * a.k + j0);
        const float4 v0 = w4[0], v1 = w4[1];
        const uint32_t keep = a.mask[(size_t)i * a.mask_stride + (j0 >> 3)] & normal;
        const float e[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
        for (int c = 0; c < 8; c++) {
            if (!((keep >> c) & 1u)) continue;
            const uint32_t bits = __float_as_uint(fabsf(e[c]));
            const uint32_t hi = pass == 0 ? 0u : bits >> (shift + 8), dig = (bits >> shift) & 255u;
            if (hi == pre0) atomicAdd(own + dig, 1u);
            if (hi == pre1) atomicAdd(own + 256 + dig, 1u);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 512; e += 256) {
        uint32_t sum = 0;
#pragma unroll
        for (int c = 0; c < SH_COPIES; c++) sum += h[c * SH_STRIDE + e];
        if (sum) atomicAdd(a.hist + (size_t)q * 512 + e, sum);
    }
}

// One wavefront per (block, statistic): the digit whose bucket holds the rank; clears the histogram for the next pass.
__global__ __launch_bounds__(64) void k_select_step(PK a, int pass) {
    const int id = blockIdx.x, lane = threadIdx.x;
    uint4* const h = reinterpret_cast<uint4*>(a.hist + (size_t)id * 256) + lane;
    const uint4 c = *h;
    *h = make_uint4(0u, 0u, 0u, 0u);
    const uint32_t rank = a.sel[2 * id + 1], own = c.x + c.y + c.z + c.w;
    uint32_t upto = own;                           // values in the buckets of this and the lower lanes
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(upto, d);
        if (lane >= d) upto += o;
    }
    const uint64_t past = __ballot(rank < upto);
    if (past == 0) {                               // an empty block
        if (lane == 0) { a.sel[2 * id] <<= 8; a.sel[2 * id + 1] = 0; }
    } else if (lane == __ffsll((unsigned long long)past) - 1) {
        uint32_t left = rank - (upto - own), dig = 4 * lane;
        if (left >= c.x) { left -= c.x; dig++;
            if (left >= c.y) { left -= c.y; dig++;
                if (left >= c.z) { left -= c.z; dig++; } } }
        a.sel[2 * id] = (a.sel[2 * id] << 8) | dig;
        a.sel[2 * id + 1] = left;
    }
    if (pass == 3) {
        __threadfence_block();
        __syncthreads();
        if (lane == 0) a.p12[2 * (id >> 1) + (id & 1)] = a.cnt[id >> 1] ? (double)__uint_as_float(a.sel[2 * id]) : 0.0;
    }
}

// ---- per (row, block): region ids, scales, sign and id bits of the block, the salient columns' residual -----------------
// A lane walks its (row, block) from left to right (the sums are sequential); a wavefront is 8 rows x 8 blocks, so that what
// it reads and writes of a row is contiguous (64 to 512 bytes).  The weights come through LDS 32 columns at a time, sign and
// id bits leave through it.  Only the kept columns are walked (all 128 with
// predicates: 0.81 ms), without a branch for a value's region (0.32 ms with them and the chunks unrolled: a wait for LDS a value, two
// wavefronts a SIMD).  Bound by vector instructions (about 30 a kept weight) beside a pass over the weights (0.18).  28672 x 8192 at 4:8:
// 0.27 ms, against 0.65 + 0.99 ms with one thread per (row, block) that reads and
// writes its own 512 and 24 bytes, once here and once for the salient columns.  Three workgroups a compute unit, two where all 8 are kept, which
// takes more registers than three leave (11008 x 4096 8:8: 79 us, 88 with 15 of them in scratch).
constexpr int AS_COLS = 32, AS_STRIDE = AS_COLS + 1, AS_SAL = 8;
template <int N8>                                              // kept weights of 8 columns
__global__ __launch_bounds__(256, N8 == 8 ? 2 : 3) void k_assign(PK a) {
    __shared__ float tile[4][64 * AS_STRIDE];
    __shared__ __attribute__((aligned(16))) uint8_t bits[4][8 * 8 * 48];          // per wavefront: 8 rows x 8 blocks x (16 + 32) bytes
    if (given_up(a)) return;               // (res_sign is indexed by the bitmap)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int qtiles = (a.nb + 7) / 8;
    const int i0 = ((int)(blockIdx.x / (unsigned)qtiles) * 4 + wave) * 8, q0 = (int)(blockIdx.x % (unsigned)qtiles) * 8;
    if (i0 >= a.n) return;                                     // (wavefronts are independent: no barrier below)
    float* const x = tile[wave];
    const int i = i0 + (lane >> 3), q = q0 + (lane & 7);
    const bool live = i < a.n && q < a.nb;
    const int ic = i < a.n ? i : a.n - 1, qc = q < a.nb ? q : a.nb - 1;
    constexpr int n8 = N8, sbytes = 2 * n8, rbytes = 4 * n8;
    uint8_t* const sout = bits[wave] + lane * sbytes;
    uint8_t* const rout = bits[wave] + 64 * sbytes + lane * rbytes;
    const uint4 m4 = *reinterpret_cast<const uint4*>(a.mask + (size_t)ic * a.mask_stride + 16 * qc);
    const uint4 s4 = make_uint4(a.sal[4 * qc], a.sal[4 * qc + 1], a.sal[4 * qc + 2], a.sal[4 * qc + 3]);
    const float p1 = round_down_f32(a.p12[2 * qc]), p2 = round_down_f32(a.p12[2 * qc + 1]);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, so = 0.0;
    int c1 = 0, c2 = 0;
    uint64_t sacc = 0;
    bool odd = false;
    // the wavefront's loads: row i0 + u, 8 lanes a block
    const int lq = q0 + (lane >> 3) < a.nb ? q0 + (lane >> 3) : a.nb - 1;
    float4 v[8];
    auto load = [&](int ch) {
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int row = i0 + u < a.n ? i0 + u : a.n - 1;
            v[u] = *reinterpret_cast<const float4*>(a.W + (size_t)row * a.k + lq * STB_BLOCK + ch * AS_COLS + 4 * (lane & 7));
        }
    };
    load(0);
#pragma unroll 1
    for (int ch = 0; ch < STB_BLOCK / AS_COLS; ch++) {
#pragma unroll
        for (int u = 0; u < 8; u++) {
            float* d = x + (8 * u + (lane >> 3)) * AS_STRIDE + 4 * (lane & 7);
            d[0] = v[u].x; d[1] = v[u].y; d[2] = v[u].z; d[3] = v[u].w;
        }
        wave_order();
        if (ch + 1 < STB_BLOCK / AS_COLS) load(ch + 1);
        const uint32_t m = ch == 0 ? m4.x : ch == 1 ? m4.y : ch == 2 ? m4.z : m4.w;
        const uint32_t sb = ch == 0 ? s4.x : ch == 1 ? s4.y : ch == 2 ? s4.z : s4.w;
        uint64_t racc = 0;
        uint32_t gsacc = 0;
#pragma unroll
        for (int g = 0; g < AS_COLS / 8; g++) {
            uint32_t left = (m >> (8 * g)) & 0xFFu, gid = 0;
            odd |= __popc(left) != n8;
            int c[n8];
            float w[n8];
#pragma unroll
            for (int r = 0; r < n8; r++) {                     // the group's kept columns, in slot order
                c[r] = 8 * g + (__ffs(left | 0x80u) - 1);
                left &= left - 1;
                w[r] = x[lane * AS_STRIDE + c[r]];
            }
#pragma unroll
            for (int r = 0; r < n8; r++) {
                // a sum takes 1 * |w| or 0 * |w| (exact products: the addition rounds as it would alone), without a branch.
                // one = the high word of 1.0; p1 <= p2
                constexpr uint32_t one = 0x3FF00000u;
                const float av = fabsf(w[r]);
                const bool is3 = ((sb >> c[r]) & 1u) != 0, over1 = av > p1, over2 = av > p2;
                const double d = (double)(is3 ? 0.0f : av);
                so += (double)(is3 ? av : 0.0f);
                const uint32_t h1 = over1 ? one : 0u, h2 = over2 ? one : 0u;
                s2 = __builtin_fma(__hiloint2double((int)h2, 0), d, s2);
                s1 = __builtin_fma(__hiloint2double((int)(h1 ^ h2), 0), d, s1);
                s0 = __builtin_fma(__hiloint2double((int)(h1 ^ one), 0), d, s0);
                const uint32_t id = is3 ? 3u : (uint32_t)over1 + (uint32_t)over2;
                gsacc |= w[r] >= 0.0f ? 1u << (g * n8 + r) : 0u;
                gid |= id << (2 * r);
            }
            racc |= (uint64_t)gid << (2 * g * n8);
        }
        const uint64_t lo = racc & 0x5555555555555555ull, hi = (racc >> 1) & 0x5555555555555555ull;
        c2 += __popcll(hi & ~lo);
        c1 += __popcll(lo & ~hi);
        sacc |= (uint64_t)gsacc << ((ch & 1) * 4 * n8);
        typedef std::conditional_t<n8 % 4 == 0, uint32_t, std::conditional_t<n8 % 2 == 0, uint16_t, uint8_t>> unit;
        constexpr int us = sizeof(unit);
#pragma unroll
        for (int u = 0; u < n8; u += us) *reinterpret_cast<unit*>(rout + ch * n8 + u) = (unit)(racc >> (8 * u));        // 8 n8 id bits
        if (ch & 1) {                                                                      // 8 n8 sign bits
#pragma unroll
            for (int u = 0; u < n8; u += us) *reinterpret_cast<unit*>(sout + (ch >> 1) * n8 + u) = (unit)(sacc >> (8 * u));
            sacc = 0;
        }
        wave_order();
    }
    const uint64_t sal[2] = {s4.x | (uint64_t)s4.y << 32, s4.z | (uint64_t)s4.w << 32}, kept[2] = {m4.x | (uint64_t)m4.y << 32, m4.z | (uint64_t)m4.w << 32};
    const int co = __popcll(sal[0] & kept[0]) + __popcll(sal[1] & kept[1]), c0 = STB_BLOCK / 8 * n8 - c1 - c2 - co;
    if (live && odd) atomicOr(a.status, ST_GROUP);                 // a group that does not keep N: scores that do not order (NaN)
    // residual binarisation of the kept salient weights (Eq. 4), from left to right; AS_SAL of them are loaded together and put
    // into LDS (one after the other each waits for memory)
    const uint16_t ao16 = stb_f64_to_f16_bits(co > 0 ? so / (double)co : 0.0);
    double sr = 0.0;
    if (live && co > 0) {
        const double ao = (double)stb_f16_bits_to_f32(ao16);
        const float* w = a.W + (size_t)i * a.k + q * STB_BLOCK;
        uint32_t* trow = a.res_sign + (size_t)i * (a.res_stride / 4);
        const uint32_t u0 = a.prefix[q];                           // index of the block's first salient column among all of them
        uint32_t word = 0, at = u0 >> 5;
        uint64_t l0 = sal[0] & kept[0], l1 = sal[1] & kept[1];     // still to be looked at
        for (int left = co; left > 0; left -= AS_SAL) {
            uint64_t f0 = l0, f1 = l1;
            float wv[AS_SAL];
#pragma unroll
            for (int e = 0; e < AS_SAL; e++) {                     // (past the last: a column that is not looked at)
                wv[e] = w[f0 ? __ffsll((unsigned long long)f0) - 1 : f1 ? 63 + __ffsll((unsigned long long)f1) : 0];
                f1 = f0 ? f1 : f1 & (f1 - 1);
                f0 &= f0 - 1;
            }
#pragma unroll
            for (int e = 0; e < AS_SAL; e++) x[lane * AS_STRIDE + e] = wv[e];
            const int count = left < AS_SAL ? left : AS_SAL;
            for (int e = 0; e < count; e++) {
                const float wf = x[lane * AS_STRIDE + e];
                const double res = (double)wf - ao * (wf >= 0.0f ? 1.0 : -1.0);
                sr += fabs(res);
                // rank of the column among the block's salient ones, kept or not
                const bool second = l0 == 0;
                const uint64_t l = second ? l1 : l0, below = (l & (0ull - l)) - 1;
                const uint32_t u = u0 + (second ? __popcll(sal[0]) + __popcll(sal[1] & below) : __popcll(sal[0] & below));
                l1 = second ? l1 & (l1 - 1) : l1;
                l0 &= l0 - 1;
                if ((u >> 5) != at) {                              // neighbouring blocks share words
                    if (word) atomicOr(trow + at, word);
                    word = 0;
                    at = u >> 5;
                }
                word |= res >= 0.0 ? 1u << (u & 31) : 0u;
            }
        }
        if (word) atomicOr(trow + at, word);
    }
    if (live) {
        const uint32_t h0 = stb_f64_to_f16_bits(c0 > 0 ? s0 / (double)c0 : 0.0), h1 = stb_f64_to_f16_bits(c1 > 0 ? s1 / (double)c1 : 0.0);
        const uint32_t h2 = stb_f64_to_f16_bits(c2 > 0 ? s2 / (double)c2 : 0.0);
        *reinterpret_cast<uint2*>(a.scales + ((size_t)i * a.nb + q) * 4) = make_uint2(h0 | h1 << 16, h2 | (uint32_t)ao16 << 16);
        a.res_scale[(size_t)i * a.nb + q] = stb_f64_to_f16_bits(co > 0 ? sr / (double)co : 0.0);
    }
    // what follows a row's last block up to its stride is zero
    if (q0 + 8 >= a.nb) {
        const int spad = (int)(a.sign_stride - (int64_t)a.nb * sbytes), rpad = (int)(a.region_stride - (int64_t)a.nb * rbytes);    // < 16 bytes
        if (i < a.n)
            for (int v = lane & 7; v < 16; v += 8) {
                if (v < spad) a.sign[(size_t)i * a.sign_stride + (size_t)a.nb * sbytes + v] = 0;
                if (v < rpad) a.region[(size_t)i * a.region_stride + (size_t)a.nb * rbytes + v] = 0;
            }
    }
    // sign and id bytes of the 8 rows: 8 blocks are 16 n8 and 32 n8 bytes, at multiples of that in the row
    const int blocks = a.nb - q0 < 8 ? a.nb - q0 : 8, rows = a.n - i0 < 8 ? a.n - i0 : 8;
    if (blocks == 8) {
        for (int v = lane; v < rows * n8; v += 64)
            *reinterpret_cast<uint4*>(a.sign + (size_t)(i0 + v / n8) * a.sign_stride + (size_t)q0 * sbytes + 16 * (v % n8)) =
                *reinterpret_cast<const uint4*>(bits[wave] + 16 * v);
        for (int v = lane; v < rows * 2 * n8; v += 64)
            *reinterpret_cast<uint4*>(a.region + (size_t)(i0 + v / (2 * n8)) * a.region_stride + (size_t)q0 * rbytes + 16 * (v % (2 * n8))) =
                *reinterpret_cast<const uint4*>(bits[wave] + 64 * sbytes + 16 * v);
    } else {
        for (int r = 0; r < rows; r++) {
            for (int v = lane; v < blocks * sbytes; v += 64) a.sign[(size_t)(i0 + r) * a.sign_stride + (size_t)q0 * sbytes + v] = bits[wave][r * 8 * sbytes + v];
            for (int v = lane; v < blocks * rbytes; v += 64)
                a.region[(size_t)(i0 + r) * a.region_stride + (size_t)q0 * rbytes + v] = bits[wave][64 * sbytes + r * 8 * rbytes + v];
        }
    }
}

// ---- the salient bitmap and its per-block prefix; one wavefront, a lane a block --------------------------------------
// With importance over the whole layer also a look at 64 weights: where all have one magnitude the mask by bounds would find nearly
// every group open after two passes over the weights, so the call goes to the sums in the defined order at once (11008 x 4096 4:8 of
// one magnitude: 947 us without the look and with every row taken again in float64, 768 with it; tertiles 1037 and 869, of which about 100 are
// launches that return at once and the second wait).
__global__ __launch_bounds__(64) void k_salient_tables(PK a) {
    const int lane = threadIdx.x;
    const float sample = fabsf(a.W[(size_t)((int64_t)lane * a.n / 64) * a.k + (size_t)lane * 2654435761u % (size_t)a.k]);
    uint32_t run = 0;
    for (int q0 = 0; q0 < a.nb; q0 += 64) {
        const int q = q0 + lane;
        uint32_t own = 0;
        if (q < a.nb)
            for (int u = 0; u < 4; u++) {
                const uint32_t wv = a.sal[4 * q + u];
                a.sal_out[4 * q + u] = wv;
                own += (uint32_t)__popc(wv);
            }
        uint32_t upto = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(upto, d);
            if (lane >= d) upto += o;
        }
        if (q < a.nb) a.prefix[q] = run + upto - own;
        run += __shfl(upto, 63);
    }
    const float first = __shfl(sample, 0);
    const bool one_magnitude = first > 0.0f && __all(sample == first);
    if (lane != 0) return;
    if (one_magnitude && !a.per_block) atomicOr(a.status, ST_UNDECIDED);
    a.prefix[a.nb] = run;
    if (run != (uint32_t)a.n_salient) atomicOr(a.status, ST_SALIENT);
}

inline int64_t up256(int64_t v) { return (v + 255) / 256 * 256; }

struct WsPlan {
    int64_t status, rs, cols, rowacc, stats, mxbits, cnt, p12, hist, sel, err, total;
    int64_t err_bytes;          // gains and counts of all blocks (k_search_gain), then errors of the remaining candidates
};

WsPlan plan_workspace(const stb_cfg_t& c, int per_block) {
    const int64_t n = c.n_out, k = c.k_in, nb = k / STB_BLOCK, nbS = per_block ? nb : 1;
    WsPlan p;
    int64_t o = 0;
    p.status = o; o += 256;
    p.rs = o; o += up256(n * nbS * 8);
    p.cols = o; o += up256(k * 16);
    p.rowacc = o; o += up256(n * nbS * 8);
    p.stats = o; o += up256(nbS * 16);
    p.mxbits = o; o += up256(nb * 4);
    p.cnt = o; o += up256(nb * 4);
    p.p12 = o; o += up256(nb * 16);
    p.hist = o; o += up256(nb * 2 * 256 * 4);
    p.sel = o; o += up256(nb * 16);
    // the gains and counts of all blocks, then candidate errors: as many blocks at once as fit into 1 GiB, at least one
    const int64_t per_block_bytes = n * CAND * 8;
    int64_t batch = (1ll << 30) / per_block_bytes;
    batch = batch < 1 ? 1 : (batch > nb ? nb : batch);
    p.err_bytes = c.region_mode != 0 ? 0 : batch * per_block_bytes > nb * SC_NV * 16 ? batch * per_block_bytes : nb * SC_NV * 16;
    p.err = o; o += up256(p.err_bytes);
    p.total = o;
    return p;
}

}  // namespace

extern "C" int64_t stb_pack_gpu_workspace(const stb_cfg_t* cfg, int per_block) {
    return plan_workspace(*cfg, per_block).total;
}

// ------------------------------------------------------------------------------------------------
// The compensation step of Alg. 1 on the GPU: the float64 working copy of W and the factor H^c stay in HBM, the host
// quantises block after block (stb_pack_obc_with) and sends each block's error matrix E.
//   W[i][j] -= sum_c E[i][c] * Hc[c0 + c][j]   for the columns j right of the block,
// the 128 terms in ascending c, one multiplication and one addition per term (no fused multiply-add: see the pragma
// at the top), the sum subtracted once -- the host loop's arithmetic, so the bytes that come out are the same.
// A workgroup takes OBC_TI rows x 256 columns: E's rows from LDS (every lane reads the same word), H^c coalesced.
// ------------------------------------------------------------------------------------------------
namespace {

constexpr int OBC_TI = 8;

__global__ __launch_bounds__(256) void k_obc_update(double* __restrict__ Wd, const double* __restrict__ E,
                                                    const double* __restrict__ Hc, int n, int k, int c0) {
    __shared__ double e[OBC_TI][STB_BLOCK];
    const int c1 = c0 + STB_BLOCK;
    const int i0 = (int)blockIdx.y * OBC_TI;
    for (int t = threadIdx.x; t < OBC_TI * STB_BLOCK; t += 256) {
        const int r = t / STB_BLOCK, c = t % STB_BLOCK;
        e[r][c] = i0 + r < n ? E[(size_t)(i0 + r) * STB_BLOCK + c] : 0.0;
    }
    __syncthreads();
    const int j = c1 + (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (j >= k) return;
    double acc[OBC_TI];
#pragma unroll
    for (int r = 0; r < OBC_TI; r++) acc[r] = 0.0;
    const double* h = Hc + (size_t)c0 * k + j;
    for (int c = 0; c < STB_BLOCK; c++) {
        const double hv = h[(size_t)c * k];
#pragma unroll
        for (int r = 0; r < OBC_TI; r++) acc[r] += e[r][c] * hv;
    }
#pragma unroll
    for (int r = 0; r < OBC_TI; r++)
        if (i0 + r < n) Wd[(size_t)(i0 + r) * k + j] -= acc[r];
}

struct ObcGpu {
    int n, k;
    double* Wd;
    double* Hc;
    double* E;
    hipStream_t st;
    int hip_err;
};

int obc_fail(ObcGpu* g, hipError_t e) { g->hip_err = (int)e; return STB_EHIP; }

int obc_start(void* ctx, const double* Wd_host) {
    ObcGpu* g = (ObcGpu*)ctx;
    hipError_t e = hipMemcpyAsync(g->Wd, Wd_host, (size_t)g->n * g->k * 8, hipMemcpyHostToDevice, g->st);
    if (e == hipSuccess) e = hipStreamSynchronize(g->st);
    return e == hipSuccess ? STB_OK : obc_fail(g, e);
}

int obc_fetch(void* ctx, int q, double* Wd_host) {
    ObcGpu* g = (ObcGpu*)ctx;
    const size_t pitch = (size_t)g->k * 8, off = (size_t)q * STB_BLOCK;
    hipError_t e = hipMemcpy2DAsync(Wd_host + off, pitch, g->Wd + off, pitch, (size_t)STB_BLOCK * 8, (size_t)g->n,
                                    hipMemcpyDeviceToHost, g->st);
    if (e == hipSuccess) e = hipStreamSynchronize(g->st);      // the update kernels of the blocks before are done too
    return e == hipSuccess ? STB_OK : obc_fail(g, e);
}

int obc_update(void* ctx, int q, const double* E_host) {
    ObcGpu* g = (ObcGpu*)ctx;
    const int c1 = (q + 1) * STB_BLOCK;
    if (c1 >= g->k) return STB_OK;
    hipError_t e = hipMemcpyAsync(g->E, E_host, (size_t)g->n * STB_BLOCK * 8, hipMemcpyHostToDevice, g->st);
    if (e == hipSuccess) e = hipStreamSynchronize(g->st);      // the host reuses its E for the next block
    if (e != hipSuccess) return obc_fail(g, e);
    const dim3 grid((unsigned)((g->k - c1 + 255) / 256), (unsigned)((g->n + OBC_TI - 1) / OBC_TI));
    hipLaunchKernelGGL(k_obc_update, grid, dim3(256), 0, g->st, g->Wd, g->E, g->Hc, g->n, g->k, q * STB_BLOCK);
    e = hipGetLastError();
    return e == hipSuccess ? STB_OK : obc_fail(g, e);
}


}  // namespace

extern "C" int64_t stb_pack_obc_gpu_workspace(const stb_cfg_t* cfg) {
    const int64_t n = cfg->n_out, k = cfg->k_in;
    return up256(n * k * 8) + up256(k * k * 8) + up256(n * STB_BLOCK * 8);
}

// W, Hc (not NULL), xnorm, sal_bitmap, out: host, as stb_pack_obc takes them; workspace: device.
extern "C" int stb_pack_obc_gpu(const float* W, const double* Hc, const float* xnorm, const uint32_t* sal_bitmap,
                                stb_layout_t* out, int32_t n_threads, void* workspace, void* stream, int* hip_err) {
    const int64_t n = out->cfg.n_out, k = out->cfg.k_in;
    if ((n + OBC_TI - 1) / OBC_TI > 65535) return STB_EUNSUPPORTED;          // rows of the update grid
    ObcGpu g;
    g.n = (int)n; g.k = (int)k; g.st = (hipStream_t)stream; g.hip_err = 0;
    g.Wd = (double*)workspace;
    g.Hc = (double*)((char*)workspace + up256(n * k * 8));
    g.E = (double*)((char*)workspace + up256(n * k * 8) + up256(k * k * 8));
    hipError_t e = hipMemcpyAsync(g.Hc, Hc, (size_t)k * k * 8, hipMemcpyHostToDevice, g.st);
    if (e == hipSuccess) e = hipStreamSynchronize(g.st);
    if (e != hipSuccess) { *hip_err = (int)e; return STB_EHIP; }
    stb_obc_accel_t accel;
    accel.ctx = &g; accel.start = obc_start; accel.fetch = obc_fetch; accel.update = obc_update;
    const int rc = stb_pack_obc_with(W, Hc, xnorm, sal_bitmap, out, n_threads, &accel);
    e = hipStreamSynchronize(g.st);                    // nothing of this call is still running when it returns
    if (rc == STB_EHIP) *hip_err = g.hip_err;
    else if (rc == STB_OK && e != hipSuccess) { *hip_err = (int)e; return STB_EHIP; }
    return rc;
}

// Break points of every block (region_mode 0) by bounds; ST_CLOSE if some block needs exact_breakpoints.  The gains start at zero.
static void bound_breakpoints(const PK& a, const WsPlan& wp, char* ws, hipStream_t st) {
    double* const gain = (double*)(ws + wp.err);
    unsigned long long* const above = (unsigned long long*)(gain + (size_t)a.nb * SC_NV);      // behind the gains
    // two workgroups a compute unit: four rounds of them at least before a workgroup takes more rows for its set-up
    const int64_t tiles = (int64_t)((a.n + SC_ROWS - 1) / SC_ROWS) * a.nb;
    const int steps = tiles >= 2048 * SC_STEPS ? SC_STEPS : tiles < 2048 ? 1 : (int)(tiles / 2048), rows = SC_ROWS * steps;
    hipLaunchKernelGGL(k_search_gain, dim3((unsigned)((int64_t)((a.n + rows - 1) / rows) * a.nb)), dim3(64 * SC_WAVES), 0, st, a, steps, gain, above);
    // (the masks of candidates left: nb * 512 words, which the tertile split alone uses otherwise)
    hipLaunchKernelGGL(k_search_narrow, dim3(a.nb), dim3(64), 0, st, a, gain, above, a.hist);
}

// ... of the blocks in which several candidates are left: waits for the stream to read which.
static int exact_breakpoints(const PK& a, const WsPlan& wp, char* ws, hipStream_t st, int* hip_err) {
    hipError_t e = hipSuccess;
    auto ok = [&](hipError_t r) { if (e == hipSuccess && r != hipSuccess) e = r; return e == hipSuccess; };
    double* const err = (double*)(ws + wp.err);
    uint32_t* const left = a.hist;
    std::vector<uint32_t> mask((size_t)a.nb * SC_MASKW);
    ok(hipMemcpyAsync(mask.data(), left, mask.size() * 4, hipMemcpyDeviceToHost, st));
    ok(hipStreamSynchronize(st));
    // batches of whole blocks whose entries fit into the error area (a block has at most CAND, and those always fit) and
    // into the list (the words behind the masks, as many again: at least CAND + 2)
    const int64_t fit = wp.err_bytes / ((int64_t)a.n * 8), words = (int64_t)a.nb * (512 - SC_MASKW);
    for (int q = 0; q < a.nb && e == hipSuccess;) {
        std::vector<uint32_t> list, first(1, 0u);
        for (; q < a.nb; q++) {
            const uint32_t* m = mask.data() + (size_t)q * SC_MASKW;
            int many = 0;
            for (int u = 0; u < SC_MASKW; u++) many += __builtin_popcount(m[u]);
            if (!many) continue;
            const int64_t entries = (int64_t)list.size() + many;
            if (!list.empty() && (first.size() > 32768 || entries > fit || entries + (int64_t)first.size() + 1 > words)) break;
            for (int t = 0; t < CAND; t++)
                if ((m[t >> 5] >> (t & 31)) & 1u) list.push_back((uint32_t)q << 8 | (uint32_t)t);
            first.push_back((uint32_t)list.size());
        }
        if (list.empty()) break;
        uint32_t* const dlist = left + (size_t)a.nb * SC_MASKW;
        uint32_t* const dfirst = dlist + list.size();
        ok(hipMemcpyAsync(dlist, list.data(), list.size() * 4, hipMemcpyHostToDevice, st));
        ok(hipMemcpyAsync(dfirst, first.data(), first.size() * 4, hipMemcpyHostToDevice, st));
        const unsigned blocks = (unsigned)first.size() - 1;
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(k_exact_errors, dim3((a.n + 63) / 64, blocks), dim3(256), 0, st, a, dlist, dfirst, err);
        hipLaunchKernelGGL(k_exact_pick, dim3(blocks), dim3(1024), 0, st, a, dlist, dfirst, err);
        ok(hipGetLastError());
        ok(hipStreamSynchronize(st));                          // the host lists must outlive their copies
    }
    *hip_err = (int)e;
    return e == hipSuccess ? STB_OK : STB_EHIP;
}

// out: row-major layout bound to device memory (checked by the caller).  Runs on `stream` and waits for it: the status
// word comes back before the call returns.
extern "C" int stb_pack_gpu(const float* W, const float* xnorm, const uint32_t* sal_bitmap, const stb_layout_t* out,
                            int per_block, void* workspace, void* stream, int* hip_err) {
    const stb_cfg_t& c = out->cfg;
    const WsPlan wp = plan_workspace(c, per_block);
    char* ws = (char*)workspace;
    const hipStream_t st = (hipStream_t)stream;
    PK a;
    a.W = W; a.xnorm = xnorm; a.sal = sal_bitmap;
    a.n = c.n_out; a.k = c.k_in; a.N = c.N; a.M = c.M; a.nb = c.k_in / STB_BLOCK; a.per_block = per_block ? 1 : 0;
    a.nbS = a.per_block ? a.nb : 1; a.region_mode = c.region_mode; a.n_salient = c.n_salient;
    a.mask = (uint8_t*)out->mask; a.sign = (uint8_t*)out->sign; a.region = (uint8_t*)out->region;
    a.res_sign = (uint32_t*)out->res_sign; a.scales = out->scales; a.res_scale = out->res_scale;
    a.sal_out = out->sal_bitmap; a.prefix = out->sal_block_prefix;
    a.mask_stride = out->mask_stride; a.sign_stride = out->sign_stride; a.region_stride = out->region_stride;
    a.res_stride = out->res_stride;
    a.status = (uint32_t*)(ws + wp.status); a.rs = (double*)(ws + wp.rs); a.cols = (double2*)(ws + wp.cols);
    a.rowacc = (double*)(ws + wp.rowacc); a.stats = (double*)(ws + wp.stats); a.mxbits = (uint32_t*)(ws + wp.mxbits);
    a.cnt = (uint32_t*)(ws + wp.cnt); a.p12 = (double*)(ws + wp.p12); a.hist = (uint32_t*)(ws + wp.hist);
    a.sel = (uint32_t*)(ws + wp.sel);

    hipError_t e = hipSuccess;
    auto ok = [&](hipError_t r) { if (e == hipSuccess && r != hipSuccess) e = r; return e == hipSuccess; };
    // everything that is accumulated into starts at zero, the gains of the search (behind the rest) among it
    ok(hipMemsetAsync(ws, 0, (size_t)(wp.err + (a.region_mode == 0 ? (int64_t)a.nb * SC_NV * 16 : 0)), st));
    if (out->res_bytes) ok(hipMemsetAsync(out->res_sign, 0, (size_t)out->res_bytes, st));
    if (e != hipSuccess) { *hip_err = (int)e; return STB_EHIP; }

    const int T = 256;
    // the salient bitmap must hold exactly cfg.n_salient columns before anything indexes the res_sign rows by it (k_assign looks)
    hipLaunchKernelGGL(k_salient_tables, dim3(1), dim3(64), 0, st, a);
    const dim3 mask_grid((unsigned)((int64_t)((a.n + MK_ROWS - 1) / MK_ROWS) * a.nb));
    auto ordered_mask = [&]() {                                // importance from the sums in the defined order
        const unsigned row_wgs = (unsigned)((a.n + RC_ROWS - 1) / RC_ROWS);
        hipLaunchKernelGGL(k_abs_sums, dim3(a.k / CC_COLS + row_wgs), dim3(CHAIN_THREADS), 0, st, a);
        hipLaunchKernelGGL(k_mu_sums<1>, dim3(row_wgs), dim3(CHAIN_THREADS), 0, st, a);
        hipLaunchKernelGGL(k_total<0>, dim3(a.nbS), dim3(64), 0, st, a);
        hipLaunchKernelGGL(k_mu_sums<2>, dim3(row_wgs), dim3(CHAIN_THREADS), 0, st, a);
        hipLaunchKernelGGL(k_total<1>, dim3(a.nbS), dim3(64), 0, st, a);
        if (a.M == 4) hipLaunchKernelGGL(k_mask<4>, mask_grid, dim3(T), 0, st, a);
        else hipLaunchKernelGGL(k_mask<8>, mask_grid, dim3(T), 0, st, a);
    };
    auto break_points = [&](bool first_counts) {               // first_counts: the mask kernel left them
        if (a.region_mode == 0) { bound_breakpoints(a, wp, ws, st); return; }
        hipLaunchKernelGGL(k_select_init, dim3((a.nb + 63) / 64), dim3(64), 0, st, a);
        for (int pass = 0; pass < 4; pass++) {
            if (pass > 0 || !first_counts) hipLaunchKernelGGL(k_select_hist, mask_grid, dim3(T), 0, st, a, pass);
            hipLaunchKernelGGL(k_select_step, dim3(2 * a.nb), dim3(64), 0, st, a, pass);
        }
    };
    auto assign = [&]() {
        const dim3 grid((unsigned)((int64_t)((a.n + 31) / 32) * ((a.nb + 7) / 8)));
        switch (8 * a.N / a.M) {
            case 1: hipLaunchKernelGGL(k_assign<1>, grid, dim3(T), 0, st, a); break;
            case 2: hipLaunchKernelGGL(k_assign<2>, grid, dim3(T), 0, st, a); break;
            case 3: hipLaunchKernelGGL(k_assign<3>, grid, dim3(T), 0, st, a); break;
            case 4: hipLaunchKernelGGL(k_assign<4>, grid, dim3(T), 0, st, a); break;
            case 5: hipLaunchKernelGGL(k_assign<5>, grid, dim3(T), 0, st, a); break;
            case 6: hipLaunchKernelGGL(k_assign<6>, grid, dim3(T), 0, st, a); break;
            case 7: hipLaunchKernelGGL(k_assign<7>, grid, dim3(T), 0, st, a); break;
            default: hipLaunchKernelGGL(k_assign<8>, grid, dim3(T), 0, st, a); break;
        }
    };
    uint32_t status = 0;
    auto finish = [&]() {                                      // waits for the stream and reads the status
        ok(hipGetLastError());
        ok(hipMemcpyAsync(&status, a.status, 4, hipMemcpyDeviceToHost, st));
        ok(hipStreamSynchronize(st));
        return e == hipSuccess;
    };
    if (!a.per_block) {
        const int64_t chunks = (a.k + FS_COLS - 1) / FS_COLS, rows = (a.n * chunks + FS_WGS * FS_BATCH - 1) / (FS_WGS * FS_BATCH) * FS_BATCH;
        hipLaunchKernelGGL(k_layer_sums, dim3((unsigned)((a.n + rows - 1) / rows * chunks)), dim3(T), 0, st, a, (int)rows);
        hipLaunchKernelGGL(k_layer_mean, dim3((unsigned)(((int64_t)a.n + a.k + 255) / 256)), dim3(T), 0, st, a);
        switch (a.M * 16 + a.N) {
#define STB_MASK(M, N) case M * 16 + N: hipLaunchKernelGGL((k_layer_mask<M, N>), mask_grid, dim3(T), a.region_mode ? LAYER_MASK_LDS : 0, st, a); break;
            STB_MASK(4, 1) STB_MASK(4, 2) STB_MASK(4, 3) STB_MASK(4, 4)
            STB_MASK(8, 1) STB_MASK(8, 2) STB_MASK(8, 3) STB_MASK(8, 4) STB_MASK(8, 5) STB_MASK(8, 6) STB_MASK(8, 7) STB_MASK(8, 8)
#undef STB_MASK
            default: return STB_EINVAL;
        }
    } else ordered_mask();
    // Almost always the whole call: what a later kernel must not work on (an unchecked bitmap, a mask or break points that the bounds
    // leave open) makes it return at once, and the host sees why.  (28672 x 8192 4:8, packing and tiling: 1390 us with a look after the mask,
    // one after the search and the small tables of the tiled order made on the host, 1262 like this.)
    break_points(!a.per_block);
    assign();
    if (!finish()) { *hip_err = (int)e; return STB_EHIP; }
    if (status & ST_SALIENT) return STB_EINVAL;
    if (status & ST_NONFINITE) return STB_ENONFINITE;
    if (status & ST_UNDECIDED) {
        ok(hipMemsetAsync(ws, 0, (size_t)wp.p12, st));         // status, sums, maxima and counts of the mask by bounds
        ordered_mask();
        break_points(false);                                   // (k_select_step has cleared the counts)
        assign();
        if (!finish()) { *hip_err = (int)e; return STB_EHIP; }
        if (status & ST_NONFINITE) return STB_ENONFINITE;
    }
    if (status & ST_CLOSE) {
        try {
            const int rc = exact_breakpoints(a, wp, ws, st, hip_err);
            if (rc != STB_OK) return rc;
        } catch (const std::bad_alloc&) { *hip_err = (int)hipErrorOutOfMemory; return STB_EHIP; }
        ok(hipMemsetAsync(a.status, 0, 4, st));
        assign();
        if (!finish()) { *hip_err = (int)e; return STB_EHIP; }
    }
    *hip_err = (int)e;
    return status ? STB_EINVAL : STB_OK;
}

// ------------------------------------------------------------------------------------------------
// stb_tile in device memory: the record permutation of the host routine, a wavefront a tile of 64 records
// ------------------------------------------------------------------------------------------------
namespace {

struct TK {
    const uint8_t* rmask; const uint8_t* rsign; const uint8_t* rreg; const uint16_t* rscales; const uint16_t* rres_scale;
    const uint32_t* rres_sign;
    uint8_t* tmask; uint8_t* tsign; uint8_t* treg; uint16_t* tscales; uint16_t* tres_scale; uint32_t* tres_sign;
    int64_t rmask_stride, rsign_stride, rreg_stride, rres_stride;
    int n, nb, nrt, nsb, res_words;
    uint32_t* finding;      // a mask byte that a padded layout cannot hold makes it non-zero; see stb_tile_gpu
};

// the WORDS words of a record: whole, or cut in two halves stored [tile][half][lane] when they are an even number
template <int WORDS>
__device__ inline void put_record(uint8_t* plane, int64_t tile, int lane, const uint32_t (&w)[WORDS]) {
    constexpr int HALVES = WORDS % 2 == 0 ? 2 : 1, HW = WORDS / HALVES;
#pragma unroll
    for (int h = 0; h < HALVES; h++) {
        uint32_t* const dst = reinterpret_cast<uint32_t*>(plane) + tile * 64 * WORDS + (int64_t)h * 64 * HW + (int64_t)lane * HW;
#pragma unroll
        for (int u = 0; u < HW; u++) dst[u] = w[h * HW + u];
    }
}

// bits [at, at + count) of a little-endian word string, count < 32
template <int WORDS>
__device__ inline uint32_t bits_at(const uint32_t (&w)[WORDS], int at, int count) {
    uint32_t v = w[at >> 5] >> (at & 31);
    if ((at & 31) + count > 32) v |= w[(at >> 5) + 1] << (32 - (at & 31));
    return v & ((1u << count) - 1u);
}
template <int WORDS>
__device__ inline void put_bits(uint32_t (&w)[WORDS], int at, int count, uint32_t v) {
    w[at >> 5] |= v << (at & 31);
    if ((at & 31) + count > 32) w[(at >> 5) + 1] |= v >> (32 - (at & 31));
}

// One thread per record, in the order in which the records lie (a wavefront = one tile: its stores are contiguous, its loads 64
// to 96 bytes of 16 rows); padding rows and blocks get zeros.  N8 kept of 8 columns, T8 slots stored for them.
// 28672 x 8192 at 4:8: 37 us (0.19 GB moved), against 460 us byte by byte.
template <int N8, int T8>
__global__ __launch_bounds__(256) void k_tile_records(TK a) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)a.nrt * a.nsb * 64) return;
    const int64_t tile = idx >> 6;
    const int lane = (int)(idx & 63), r = (int)(tile / a.nsb) * 16 + (lane & 15), q = (int)(tile % a.nsb) * 4 + (lane >> 4);
    const bool live = r < a.n && q < a.nb;
    uint32_t m[4] = {0, 0, 0, 0}, sg[(T8 + 1) / 2] = {}, id[T8] = {};
    uint2 sc = make_uint2(0u, 0u);
    uint16_t rs = 0;
    if (live) {
        const uint4 m4 = *reinterpret_cast<const uint4*>(a.rmask + (int64_t)r * a.rmask_stride + 16 * q);
        m[0] = m4.x; m[1] = m4.y; m[2] = m4.z; m[3] = m4.w;
        // (a row's block starts at a multiple of 2 N8 and 4 N8 bytes: words, but for the signs of an odd N8)
        const uint8_t* srow = a.rsign + (int64_t)r * a.rsign_stride + (int64_t)(2 * N8) * q;
        const uint32_t* grow = reinterpret_cast<const uint32_t*>(a.rreg + (int64_t)r * a.rreg_stride + (int64_t)(4 * N8) * q);
        sc = *reinterpret_cast<const uint2*>(a.rscales + ((int64_t)r * a.nb + q) * 4);
        rs = a.rres_scale[(int64_t)r * a.nb + q];
        uint32_t ss[(N8 + 1) / 2], gg[N8];
#pragma unroll
        for (int u = 0; u < N8; u++) gg[u] = grow[u];
        if (N8 % 2 == 0) {
#pragma unroll
            for (int u = 0; u < N8 / 2; u++) ss[u] = reinterpret_cast<const uint32_t*>(srow)[u];
        } else {
            const uint16_t* s2 = reinterpret_cast<const uint16_t*>(srow);
#pragma unroll
            for (int u = 0; u < (N8 + 1) / 2; u++) ss[u] = (uint32_t)s2[2 * u] | (2 * u + 1 < N8 ? (uint32_t)s2[2 * u + 1] << 16 : 0u);
        }
        if constexpr (N8 == T8) {
#pragma unroll
            for (int u = 0; u < (T8 + 1) / 2; u++) sg[u] = ss[u];
#pragma unroll
            for (int u = 0; u < T8; u++) id[u] = gg[u];
        } else {
            // 3 or 5 kept of 8: a free slot goes where the group's lowest pruned column would rank: all columns below
            // it are kept, so its rank is its position
            bool bad = false;
#pragma unroll
            for (int g = 0; g < 16; g++) {
                const uint32_t mb = (m[g >> 2] >> (8 * (g & 3))) & 0xFFu;
                bad |= __popc(mb) != N8;
                const int free = __ffs((int)~mb) - 1;
                const uint32_t s = bits_at(ss, N8 * g, N8), v = bits_at(gg, 2 * N8 * g, 2 * N8);
                const uint32_t slow = (1u << free) - 1u, vlow = (1u << (2 * free)) - 1u;
                put_bits(sg, T8 * g, T8, (s & slow) | ((s & ~slow) << 1));
                put_bits(id, 2 * T8 * g, 2 * T8, (v & vlow) | ((v & ~vlow) << 2));
            }
            if (bad) { atomicOr(a.finding, 1u); return; }
        }
    }
    put_record(a.tmask, tile, lane, m);
    if constexpr (T8 % 2 == 0) put_record(a.tsign, tile, lane, sg);
    else {
        uint16_t* const dst = reinterpret_cast<uint16_t*>(a.tsign) + idx * T8;
#pragma unroll
        for (int u = 0; u < T8; u++) dst[u] = (uint16_t)(sg[u >> 1] >> (16 * (u & 1)));
    }
    put_record(a.treg, tile, lane, id);
    reinterpret_cast<uint2*>(a.tscales)[idx] = sc;
    a.tres_scale[idx] = rs;
}

// The tables that depend on the salient bitmap alone.  Workgroup 0: bitmap and prefix padded to whole superblocks; the others: a
// thread per record of sal_tab, 8 salient columns of a half block, as the host routine fills it.
__global__ __launch_bounds__(256) void k_tile_tables(TK a, const uint32_t* __restrict__ bitmap, const uint32_t* __restrict__ prefix, int chunks,
                                                     uint32_t* __restrict__ bitmap_out, uint32_t* __restrict__ prefix_out, uint32_t* __restrict__ tab) {
    const int tid = threadIdx.x;
    if (blockIdx.x == 0) {
        for (int u = tid; u < a.nsb * 16; u += 256) bitmap_out[u] = u < a.nb * 4 ? bitmap[u] : 0u;
        for (int q = tid; q <= a.nsb * 4; q += 256) prefix_out[q] = prefix[q < a.nb ? q : a.nb];
        return;
    }
    const int rec = ((int)blockIdx.x - 1) * 256 + tid;
    if (rec >= a.nsb * 8 * chunks) return;
    const int c = rec % chunks, q = rec / chunks >> 1, h = rec / chunks & 1;
    auto half = [&](int b, int u) { return b < a.nb ? bitmap[4 * b + 2 * u] | (uint64_t)bitmap[4 * b + 2 * u + 1] << 32 : 0ull; };
    int need = 0;                                              // records of the fullest of the superblock's four halves
    for (int g = 0; g < 4; g++) {
        const int r = (__popcll(half((q & ~3) + g, h)) + 7) / 8;
        need = r > need ? r : need;
    }
    uint64_t left = half(q, h);
    for (int u = 0; u < 8 * c; u++) left &= left - 1;
    uint32_t sel[2] = {0u, 0u}, bit[2] = {0u, 0u}, pos[4] = {0u, 0u, 0u, 0u}, cnt = 0;
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const bool valid = left != 0;
        const uint32_t col = valid ? (uint32_t)(64 * h + __ffsll((unsigned long long)left) - 1) : 0xFFFFu;
        left &= left - 1;
        sel[e >> 2] |= (valid ? (col >> 3) & 7u : 0x0Cu) << (8 * (e & 3));
        bit[e >> 2] |= valid ? (1u << (col & 7u)) << (8 * (e & 3)) : 0u;
        pos[e >> 1] |= col << (16 * (e & 1));
        cnt += valid;
    }
    const uint32_t ord = prefix[q < a.nb ? q : a.nb] + (h ? (uint32_t)__popcll(half(q, 0)) : 0u) + 8u * (uint32_t)c;
    uint32_t* const out = tab + (int64_t)rec * 12;             // [block][half][chunk]
    out[0] = sel[0]; out[1] = sel[1]; out[2] = bit[0]; out[3] = bit[1];
    out[4] = ord; out[5] = (uint32_t)need; out[6] = cnt; out[7] = 0u;
#pragma unroll
    for (int e = 0; e < 4; e++) out[8 + e] = pos[e];
}

// res_sign: the row strings cut into 32-bit words and transposed inside each 16-row tile; one thread per word, padding rows
// included
__global__ void k_tile_res(TK a) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)a.nrt * 16 * a.res_words) return;
    const int r = (int)(idx / a.res_words), w = (int)(idx % a.res_words);
    a.tres_sign[((int64_t)(r / 16) * a.res_words + w) * 16 + r % 16] = r < a.n ? a.rres_sign[(int64_t)r * (a.rres_stride / 4) + w] : 0u;
}

// res_t: per (row, block) the res_sign bits of the first 16 salient columns of each half block; one thread per record
// (ord < n_salient wherever bitmap and prefix are right, which the host sees after the call's one wait)
__global__ void k_tile_res_t(TK a, const uint32_t* __restrict__ bitmap, const uint32_t* __restrict__ prefix, int n_salient,
                             uint32_t* __restrict__ res_t) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)a.nrt * a.nsb * 64) return;
    const int64_t tile = idx >> 6;
    const int lane = (int)(idx & 63), r = (int)(tile / a.nsb) * 16 + (lane & 15), q = (int)(tile % a.nsb) * 4 + (lane >> 4);
    if (r >= a.n || q >= a.nb) { res_t[idx] = 0u; return; }
    const uint32_t* row = a.rres_sign + (int64_t)r * (a.rres_stride / 4);
    uint32_t ord = prefix[q], word = 0;
    for (int h = 0; h < 2; h++) {
        int e = 0;
        for (int u = 0; u < 2; u++) {
            uint32_t bits = bitmap[4 * q + 2 * h + u];
            while (bits) {
                bits &= bits - 1;
                if (e < 16 && ord < (uint32_t)n_salient && ((row[ord >> 5] >> (ord & 31)) & 1u)) word |= 1u << (16 * h + e);
                e++;
                ord++;
            }
        }
    }
    res_t[idx] = word;
}

}  // namespace

// src: checked row-major layout, dst: checked tiled layout of the same cfg, both bound to device memory.
extern "C" int stb_tile_gpu(const stb_layout_t* src, stb_layout_t* dst, void* stream, int* hip_err) {
    const hipStream_t st = (hipStream_t)stream;
    hipError_t e = hipSuccess;
    auto ok = [&](hipError_t r) { if (e == hipSuccess && r != hipSuccess) e = r; return e == hipSuccess; };
    const int k = src->cfg.k_in, nb = src->n_blocks;
    TK a;
    a.rmask = (const uint8_t*)src->mask; a.rsign = (const uint8_t*)src->sign; a.rreg = (const uint8_t*)src->region;
    a.rscales = src->scales; a.rres_scale = src->res_scale; a.rres_sign = (const uint32_t*)src->res_sign;
    a.tmask = (uint8_t*)dst->mask; a.tsign = (uint8_t*)dst->sign; a.treg = (uint8_t*)dst->region;
    a.tscales = dst->scales; a.tres_scale = dst->res_scale; a.tres_sign = (uint32_t*)dst->res_sign;
    a.rmask_stride = src->mask_stride; a.rsign_stride = src->sign_stride; a.rreg_stride = src->region_stride;
    a.rres_stride = src->res_stride;
    a.n = src->cfg.n_out; a.nb = nb; a.nrt = dst->n_row_tiles; a.nsb = dst->n_super;
    a.res_words = (int)(src->res_stride / 4);
    // What the record kernel finds (a mask byte with the wrong number of bits in a padded layout) goes into the first word of the prefix that the
    // table kernel has written before it: 0 in every valid image, and the call's own, so calls on other streams do not meet it.
    a.finding = dst->sal_block_prefix;
    const int recs_tab = a.nsb * 8 * dst->sal_chunks;
    hipLaunchKernelGGL(k_tile_tables, dim3((unsigned)(1 + (recs_tab + 255) / 256)), dim3(256), 0, st, a, src->sal_bitmap, src->sal_block_prefix,
                       dst->sal_chunks, dst->sal_bitmap, dst->sal_block_prefix, dst->sal_tab);
    const int64_t recs = (int64_t)a.nrt * a.nsb * 64;
    const dim3 rec_grid((unsigned)((recs + 255) / 256));
    switch (8 * src->cfg.N / src->cfg.M) {
        case 1: hipLaunchKernelGGL((k_tile_records<1, 1>), rec_grid, dim3(256), 0, st, a); break;
        case 2: hipLaunchKernelGGL((k_tile_records<2, 2>), rec_grid, dim3(256), 0, st, a); break;
        case 3: hipLaunchKernelGGL((k_tile_records<3, 4>), rec_grid, dim3(256), 0, st, a); break;
        case 4: hipLaunchKernelGGL((k_tile_records<4, 4>), rec_grid, dim3(256), 0, st, a); break;
        case 5: hipLaunchKernelGGL((k_tile_records<5, 6>), rec_grid, dim3(256), 0, st, a); break;
        case 6: hipLaunchKernelGGL((k_tile_records<6, 6>), rec_grid, dim3(256), 0, st, a); break;
        case 7: hipLaunchKernelGGL((k_tile_records<7, 7>), rec_grid, dim3(256), 0, st, a); break;
        default: hipLaunchKernelGGL((k_tile_records<8, 8>), rec_grid, dim3(256), 0, st, a); break;
    }
    if (a.res_words > 0) {
        const int64_t words = (int64_t)a.nrt * 16 * a.res_words;
        hipLaunchKernelGGL(k_tile_res, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, a);
        hipLaunchKernelGGL(k_tile_res_t, rec_grid, dim3(256), 0, st, a, src->sal_bitmap, src->sal_block_prefix, src->cfg.n_salient, dst->res_t);
    }
    ok(hipGetLastError());
    // the two maxima follow from the bitmap; bitmap and prefix must describe cfg.n_salient columns
    std::vector<uint32_t> words;
    try { words.resize((size_t)k / 32 + (size_t)nb + 1); } catch (const std::bad_alloc&) { e = hipErrorOutOfMemory; }
    uint32_t *const bitmap = words.data(), *const prefix = bitmap + (size_t)k / 32;
    if (e == hipSuccess) {
        ok(hipMemcpyAsync(bitmap, src->sal_bitmap, (size_t)k / 8, hipMemcpyDeviceToHost, st));
        ok(hipMemcpyAsync(prefix, dst->sal_block_prefix, 4 * ((size_t)nb + 1), hipMemcpyDeviceToHost, st));
    }
    ok(hipStreamSynchronize(st));
    *hip_err = (int)e;
    if (e != hipSuccess) return STB_EHIP;
    int mx = 0, mh = 0;
    uint32_t run = 0;
    for (int q = 0; q < nb; q++) {
        int of[2];
        for (int h = 0; h < 2; h++) of[h] = __builtin_popcount(bitmap[4 * q + 2 * h]) + __builtin_popcount(bitmap[4 * q + 2 * h + 1]);
        mh = std::max(mh, std::max(of[0], of[1]));
        mx = std::max(mx, of[0] + of[1]);
        if (prefix[q] != run) return STB_EINVAL;
        run += (uint32_t)(of[0] + of[1]);
    }
    if (prefix[nb] != run || run != (uint32_t)src->cfg.n_salient) return STB_EINVAL;
    dst->max_sal_block = mx;
    dst->max_sal_half = mh;
    return STB_OK;
}
