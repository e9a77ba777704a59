// O(n d) kernels around the streaming passes: derived copies of the point
// clouds and their squared norms (Prop. 1: alpha, beta), the per-point bias
// (Alg. 1, "precompute bias"), and the merge of the per-split LSE statistics into
// the new shifted potential.
#include <string.h>

#include <atomic>
#include <chrono>

#include "fs_finalize.h"
#include "fs_internal.h"

namespace fs {
namespace {

__device__ inline float bf16_to_float(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// round-to-nearest-even float -> bfloat16 bits (NaN kept quiet)
__device__ inline uint16_t float_to_bf16(float v)
{
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ inline float load_pt(const void *pts, int dtype, int64_t idx)
{
    return dtype == FS_BF16 ? bf16_to_float(((const uint16_t *)pts)[idx]) : ((const float *)pts)[idx];
}

__global__ void k_fill_f64(double *dst, double v, int64_t cnt)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cnt) dst[i] = v;
}

// ---- squared row norms, float64 accumulation --------------------------------------------
__global__ void k_row_norms(const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld, float *out)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows) return;
    double s = 0.0;
    for (int64_t k = 0; k < d; ++k) {
        double v = (double)load_pt(pts, dtype, i * ld + k);
        s += v * v;
    }
    out[i] = (float)s;
}

__device__ inline float max_or_nan(float a, float b) { return a >= b || a != a ? a : b; }

// ---- common mean of both clouds (low-d path), deterministic two-stage reduction ---------
// stage 1: block b writes the coordinate sums of its slice to part[b][0..15]
// (blockIdx.y: 0 = the x cloud, 1 = the y cloud)
struct CloudIn {
    const void *pts;
    int64_t rows, ld;
    double *part;
};
__global__ __launch_bounds__(256) void k_coord_sums(CloudIn c0, CloudIn c1, int dtype, int d, bool bounds)
{
    const CloudIn &cl = blockIdx.y ? c1 : c0;
    const void *pts = cl.pts;
    const int64_t rows = cl.rows, ld = cl.ld;
    double *part = cl.part;
    // (all sixteen accumulators in registers, and one reduction over the wave per coordinate in use: sixteen block-wide
    // reductions through LDS took 13.7 us whatever the size)
    __shared__ double sh[4][kLowdMaxD];
    double acc[kLowdMaxD];
#pragma unroll
    for (int k = 0; k < kLowdMaxD; ++k) acc[k] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < rows; i += (int64_t)gridDim.x * 256)
#pragma unroll
        for (int k = 0; k < kLowdMaxD; ++k)
            if (k < d) acc[k] += (double)load_pt(pts, dtype, i * ld + k);
#pragma unroll
    for (int k = 0; k < kLowdMaxD; ++k)
        if (k < d) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc[k] += __shfl_xor(acc[k], off);
        }
    // bounds (d <= 3): columns 4 + k and 8 + k hold the largest -v and v of coordinate k
    float down[3] = {-INFINITY, -INFINITY, -INFINITY}, up[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (bounds) {
        for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < rows; i += (int64_t)gridDim.x * 256)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (k < d) {
                    const float v = load_pt(pts, dtype, i * ld + k);
                    down[k] = max_or_nan(down[k], -v);
                    up[k] = max_or_nan(up[k], v);
                }
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                down[k] = max_or_nan(down[k], __shfl_xor(down[k], off));
                up[k] = max_or_nan(up[k], __shfl_xor(up[k], off));
            }
    }
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < kLowdMaxD; ++k) sh[threadIdx.x >> 6][k] = acc[k];
        if (bounds) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                sh[threadIdx.x >> 6][4 + k] = (double)down[k];
                sh[threadIdx.x >> 6][8 + k] = (double)up[k];
            }
        }
    }
    __syncthreads();
    if (bounds && threadIdx.x >= 4 && threadIdx.x < kLowdMaxD) {
        float b = -INFINITY;
        for (int w = 0; w < 4; ++w) b = max_or_nan(b, (float)sh[w][threadIdx.x]);
        part[(int64_t)blockIdx.x * kLowdMaxD + threadIdx.x] = (double)b;
    } else if (threadIdx.x < kLowdMaxD)
        part[(int64_t)blockIdx.x * kLowdMaxD + threadIdx.x] = sh[0][threadIdx.x] + sh[1][threadIdx.x] + sh[2][threadIdx.x] + sh[3][threadIdx.x];
}

// stage 2: mean[k] = (sum of partX[.][k] + sum of partY[.][k]) / (n + m).  One block of 256: thread
// (group g, coordinate k) sums the blocks b = g mod 16, then coordinate k's 16 group sums are added
// in a fixed order.  Also clears zeroed[0..2] (the slots the next kernels take maxima into), and where `bounds` is given (d <= 3) leaves the bounds
// of the centred clouds in bounds[2 side + 0 (smallest) / 1 (largest)][coordinate] (a NaN where one is): the largest and the
// smallest of the centred coordinates to the last bit, since the same subtraction makes those (rounded to floats, a cloud narrower
// than the last place of its distance from the mean was one point).
__global__ __launch_bounds__(256) void k_mean_final(const double *partX, const double *partY, int blocks, double inv_cnt,
                                                    double *mean, double *zeroed, int d, double *bounds)
{
    static_assert(kLowdMaxD == 16, "thread mapping below");
    __shared__ double sh[16][kLowdMaxD];
    const int k = threadIdx.x & 15, g = threadIdx.x >> 4;
    const bool is_bound = bounds && k >= 4;   // (columns 4..6 and 8..10 of the partial sums, see k_coord_sums)
    __shared__ float shb[2][16][kLowdMaxD];
    if (is_bound) {
        float b[2] = {-INFINITY, -INFINITY};
        for (int q = g; q < blocks; q += 16) {
            b[0] = max_or_nan(b[0], (float)partX[(int64_t)q * kLowdMaxD + k]);
            b[1] = max_or_nan(b[1], (float)partY[(int64_t)q * kLowdMaxD + k]);
        }
        shb[0][g][k] = b[0];
        shb[1][g][k] = b[1];
    }
    double s = 0.0;
    if (!is_bound)
        for (int b = g; b < blocks; b += 16) s += partX[(int64_t)b * kLowdMaxD + k] + partY[(int64_t)b * kLowdMaxD + k];
    sh[g][k] = s;
    __syncthreads();
    if (threadIdx.x < kLowdMaxD) {
        double t = 0.0;
        for (int q = 0; q < 16; ++q) t += sh[q][threadIdx.x];
        mean[threadIdx.x] = t * inv_cnt;
    }
    __syncthreads();   // (mean is read below)
    if (bounds && threadIdx.x < 12) {
        const int side = threadIdx.x / 6, top = threadIdx.x / 3 % 2, c = threadIdx.x % 3;
        float b = -INFINITY;
        for (int q = 0; q < 16; ++q) b = max_or_nan(b, shb[side][q][top ? 8 + c : 4 + c]);
        // (column 4 + c holds the largest -v)
        bounds[(2 * side + top) * 3 + c] = c < d ? (top ? (double)b : -(double)b) - mean[c] : 0.0;
    }
    if (threadIdx.x < 3) zeroed[threadIdx.x] = 0.0;
}

// ---- low-d derived copies: coordinates centred at the common mean, packed with a bias slot;
//      float (rounded once) and double (exact difference), each with its own squared norms ----
// (blockIdx.y: 0 = the x cloud, 1 = the y cloud; a cloud's cnt_pad is a multiple of the block size, so a
// block is either entirely inside it or leaves as a whole)
struct PrepLowdSide {
    const void *pts;
    int64_t cnt, cnt_pad, ld;
    float *packed;
    double *packed_d, *norm_f, *norm;
    uint16_t *split;
    double *pts_d, *bias_d;   // d > 3: records of the fp64 matrix-core pass ([cnt_pad][kp] centred coordinates, bias), else null
};
// point i of a side (i < cnt_pad): its derived copies; returns its squared norm after centring
__device__ __forceinline__ double prep_lowd_point(const PrepLowdSide &sd, const int64_t i, const int dtype, const int d, const int dp, const int dpd,
                                                  const int kp, const double *mean, const int ks)
{
    const void *pts = sd.pts;
    const int64_t cnt = sd.cnt, ld = sd.ld;
    uint16_t *split = sd.split;
    float *o = sd.packed + i * dp;
    double *od = sd.packed_d + i * dpd;
    double nf = 0.0, nd = 0.0;
    for (int k = 0; k < dp; ++k) o[k] = 0.0f;
    for (int k = 0; k < dpd; ++k) od[k] = 0.0;
    if (i < cnt) {
        for (int k = 0; k < d; ++k) {
            double v = (double)load_pt(pts, dtype, i * ld + k) - mean[k];
            float vf = (float)v;
            o[k] = vf;
            od[k] = v;
            nf += (double)vf * (double)vf;
            nd += v * v;
        }
    }
    o[d] = -INFINITY;   // bias slots: padding rows never contribute; real rows are set per half-step
    od[d] = -INFINITY;
    if (sd.pts_d) {
        double *op = sd.pts_d + i * kp;
        for (int k = 0; k < kp; ++k) op[k] = k < d ? od[k] : 0.0;
        sd.bias_d[i] = -INFINITY;
    }
    sd.norm_f[i] = nf;
    sd.norm[i] = nd;
    if (split) {   // streamed-role split record of the float copy (see split_ksteps)
        auto put = [&](int t, uint32_t v) { reinterpret_cast<uint32_t *>(split)[4 * split_unit(ks, i, t >> 2) + (t & 3)] = v; };
        const uint32_t sign = split_negated(i) ? 0x80008000u : 0u;
        for (int q = 0; q < split_pairs(d); ++q) {
            __bf16 y[3], z[3];
            split3(o[2 * q], y);
            split3(2 * q + 1 < d ? o[2 * q + 1] : 0.0f, z);
            put(4 * q, bf16_pair(y[0], y[1]) ^ sign);
            put(4 * q + 1, bf16_pair(y[1], y[0]) ^ sign);
            if (2 * q + 1 < d) {
                put(4 * q + 2, bf16_pair(z[0], z[1]) ^ sign);
                put(4 * q + 3, bf16_pair(z[1], z[0]) ^ sign);
            }
            put(2 * d + q, bf16_pair(y[2], z[2]) ^ sign);
            put(split_lead(ks, d) + q, bf16_pair(y[0], z[0]) ^ sign);
        }
        for (int t = 2 * d + split_pairs(d); t < split_lead(ks, d); ++t) put(t, 0u);
        const uint2 none = split_bias_words(-INFINITY, split_negated(i));
        put(8 * ks - 2, none.x);
        put(8 * ks - 1, none.y);
    }
    return nd;
}
__global__ __launch_bounds__(256) void k_prep_lowd(PrepLowdSide s0, PrepLowdSide s1, int dtype, int d, int dp, int dpd, int kp,
                                                   const double *mean, int ks, unsigned long long *rho_max_bits)
{
    const PrepLowdSide &sd = blockIdx.y ? s1 : s0;
    if ((int64_t)blockIdx.x * 256 >= sd.cnt_pad) return;
    __shared__ double shmax[256];
    const double nd = prep_lowd_point(sd, (int64_t)blockIdx.x * 256 + threadIdx.x, dtype, d, dp, dpd, kp, mean, ks);
    // largest squared norm after centring, over both clouds: non-negative doubles order like their
    // bit patterns, and a maximum does not depend on the order of the atomics
    shmax[threadIdx.x] = nd;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) shmax[threadIdx.x] = fmax(shmax[threadIdx.x], shmax[threadIdx.x + st]);
        __syncthreads();
    }
    if (threadIdx.x == 0 && shmax[0] > 0.0) atomicMax(rho_max_bits, (unsigned long long)__double_as_longlong(shmax[0]));
}

// ---- "precise" split records (d <= 3) from the float64 copy; layout of the six 16-byte pieces
//      (resident counterparts in k_lse_lowd_split):
//   0: Y1_0 Y1_1 Y1_2 0 0 0 0 0          leading digits on the grid gy          x  X1_0 X1_1 X1_2
//   1: Ba Bb Bc 1 1 1 0 0                bias digits on the grid gx gy, ones    x  1 1 1 m1 m2 m3
//   2+k: ry1 ry2 ry3 Y1 Y1 Y1 ry1 ry2    residual pieces of coordinate k        x  X1 X1 X1 rx1 rx2 rx3 rx1 rx1
//   5: rb1 rb2 rb3 0 0 ry1_0 ry1_1 ry1_2 bias residual, second-order terms      x  1 1 1 0 0 rx2_0 rx2_1 rx2_2
// `rho_max`: device scalar (largest squared norm after centring): the grid comes from it
// (blockIdx.y: 0 = the x cloud, 1 = the y cloud)
__device__ __forceinline__ void prep_precise_point(const double *packed_d, uint16_t *out, const int64_t i, const int d, const int dpd,
                                                   const double rho_max)
{
    double gx_unused, gy;
    split_grids(rho_max, 1.0, &gx_unused, &gy);
    __bf16 Y1[3], ry[3][3];
    for (int k = 0; k < 3; ++k) {
        const double y = k < d ? packed_d[i * dpd + k] : 0.0;
        const double y1 = rint(y / gy) * gy;
        Y1[k] = (__bf16)(float)y1;
        split3d(y - y1, ry[k]);
    }
    const __bf16 z = (__bf16)0.0f;
    uint4 *rec = reinterpret_cast<uint4 *>(out) + split_unit(3, i, 0);   // (piece k: 32 k units on)
    rec[0] = make_uint4(bf16_pair(Y1[0], Y1[1]), bf16_pair(Y1[2], z), 0u, 0u);
    split_precise_bias(-INFINITY, 1.0, rec + 32, nullptr);
    for (int k = 0; k < 3; ++k)
        rec[64 + 32 * k] = make_uint4(bf16_pair(ry[k][0], ry[k][1]), bf16_pair(ry[k][2], Y1[k]), bf16_pair(Y1[k], Y1[k]),
                                bf16_pair(ry[k][0], ry[k][1]));
    rec[160] = make_uint4(0u, 0u, bf16_pair(z, ry[0][0]), bf16_pair(ry[1][0], ry[2][0]));
}
__global__ void k_prep_split_precise(const double *packed_d0, int64_t cnt_pad0, uint16_t *out0, const double *packed_d1,
                                     int64_t cnt_pad1, uint16_t *out1, int d, int dpd, const double *rho_max)
{
    const double *packed_d = blockIdx.y ? packed_d1 : packed_d0;
    const int64_t cnt_pad = blockIdx.y ? cnt_pad1 : cnt_pad0;
    uint16_t *out = blockIdx.y ? out1 : out0;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cnt_pad) prep_precise_point(packed_d, out, i, d, dpd, *rho_max);
}

constexpr double kSmallPrologue = 12288.0;   // coordinates of both clouds
// The whole prologue of a small problem in one launch: every workgroup forms the mean and the largest squared norm of both clouds
// for itself (in the same order, so all get the same bits), then 256 points of its side.  Bound by latency: the four launches
// (coordinate sums, mean, copies, precise records) take 19 us at n = 1000, m = 777, d = 3, this one 10.6; an f- and a g-half-step call
// there 93.4 us before, 81.6 now.  The line is where the loads that each workgroup repeats eat that up: both calls at n = 2500, m = 2600,
// d = 3 (15300 coordinates) 95 and 94 us, at n = m = 4000, d = 4 (32000) 111 and 129.
__global__ __launch_bounds__(1024) void k_prep_lowd_small(PrepLowdSide s0, PrepLowdSide s1, int dtype, int d, int dp, int dpd, int kp, int ks,
                                                          uint16_t *precise0, uint16_t *precise1, double *mean_out, double *scalars5)
{
    __shared__ double sh[16][kLowdMaxD], mean[kLowdMaxD], shr[16];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int64_t n = s0.cnt, all = n + s1.cnt;
    double acc[kLowdMaxD];
#pragma unroll
    for (int k = 0; k < kLowdMaxD; ++k) acc[k] = 0.0;
    for (int64_t i = tid; i < all; i += 1024) {
        const PrepLowdSide &c = i < n ? s0 : s1;
        const int64_t at = (i < n ? i : i - n) * c.ld;
#pragma unroll
        for (int k = 0; k < kLowdMaxD; ++k)
            if (k < d) acc[k] += (double)load_pt(c.pts, dtype, at + k);
    }
#pragma unroll
    for (int k = 0; k < kLowdMaxD; ++k)
        if (k < d) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc[k] += __shfl_xor(acc[k], off);
            if (l == 0) sh[w][k] = acc[k];
        }
    __syncthreads();
    if (tid < kLowdMaxD) {
        double t = 0.0;
        if (tid < d)
            for (int q = 0; q < 16; ++q) t += sh[q][tid];
        mean[tid] = t / (double)all;
    }
    __syncthreads();
    double rho = 0.0;
    for (int64_t i = tid; i < all; i += 1024) {
        const PrepLowdSide &c = i < n ? s0 : s1;
        const int64_t at = (i < n ? i : i - n) * c.ld;
        double nd = 0.0;
        for (int k = 0; k < d; ++k) {
            const double v = (double)load_pt(c.pts, dtype, at + k) - mean[k];
            nd += v * v;
        }
        rho = fmax(rho, nd);
    }
    for (int off = 32; off > 0; off >>= 1) rho = fmax(rho, __shfl_xor(rho, off));
    if (l == 0) shr[w] = rho;
    __syncthreads();
    for (int q = 0; q < 16; ++q) rho = fmax(rho, shr[q]);
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        if (tid < kLowdMaxD) mean_out[tid] = mean[tid];
        if (tid < 3) scalars5[tid] = tid == 2 ? rho : 0.0;
    }
    const PrepLowdSide &sd = blockIdx.y ? s1 : s0;
    const int64_t i = (int64_t)blockIdx.x * 256 + tid;
    if (tid >= 256 || i >= sd.cnt_pad) return;
    (void)prep_lowd_point(sd, i, dtype, d, dp, dpd, kp, mean, ks);
    if (d <= 3) prep_precise_point(sd.packed_d, blockIdx.y ? precise1 : precise0, i, d, dpd, rho);
}

// ---- float64 derived copy (fp64 matrix-core path) ----------------------------------------
__global__ void k_prep_f64(const void *pts, int dtype, int64_t cnt, int64_t cnt_pad, int64_t d, int64_t ld, int kp,
                           double *out, double *bias, double *norm)
{
    // one wave-sized group of 64 threads per row, strided over the coordinates
    int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    if (row >= cnt_pad) return;
    double nrm = 0.0;
    for (int k = lane; k < kp; k += 64) {
        double v = 0.0;
        if (row < cnt && k < d) v = (double)load_pt(pts, dtype, row * ld + k);
        out[row * kp + k] = v;
        nrm += v * v;
    }
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
    if (lane == 0) {
        norm[row] = nrm;
        bias[row] = -INFINITY;
    }
}

// ---- bfloat16 derived copy (bf16 matrix-core path); norms of the ROUNDED points ----------
// Layout: the copy is stored in 1 KB tiles of 16 rows x 32 coordinates; the sixteen tiles of a group
// of 256 rows at one chunk of 32 coordinates are contiguous (16 KB), and the groups of one row group
// follow each other chunk by chunk: tile (rb, ch) sits at (((rb / 16) * n_chunks + ch) * 16 + rb % 16) KB.
// Inside a tile row r occupies 64 bytes and its 16-byte piece p (coordinates 8p..8p+7 of the chunk)
// sits at position p ^ ((r >> 2) & 3).  A 16 KB group is exactly the image that half a pipeline stage
// needs in LDS, so the streaming kernel fills LDS with linear direct loads, each wave a contiguous run
// of it, and reads MFMA fragments without bank conflicts; the contraction loop of a tile walks through
// memory linearly.
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));       // four floats, sixteen bytes at an address that is only
typedef uint32_t u4_any __attribute__((ext_vector_type(4), aligned(2)));    // a multiple of the element's size (one load here)
// A workgroup of NW waves makes sixteen rows, a wave a whole 1 KB tile at a time (lane: row l / 4, piece l % 4), every NW-th chunk.  Bound by
// the memory, 330 MB at n = 40009, m = 30011, d = 784 in fp32: 158 us with a wave per row and a load per coordinate, 68 here (what is read
// last is still in the last-level cache).
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_prep_bf16(const void *pts, int dtype, int64_t cnt, int64_t d, int64_t ld, int kp, uint16_t *out, float *bias,
                                                   double *norm)
{
    __shared__ double shn[NW][16];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int64_t rb = blockIdx.x, row = rb * 16 + (l >> 2);
    const int n_chunks = kp >> 5, piece = l & 3;
    const int64_t base = row * ld;
    const bool real = row < cnt;
    unsigned char *dst = reinterpret_cast<unsigned char *>(out) + (((rb >> 4) * n_chunks * 16 + (rb & 15)) << 10) + (l >> 2) * 64 +
                         ((piece ^ ((l >> 4) & 3)) << 4);
    double nrm = 0.0;
#pragma unroll 4
    for (int ch = w; ch < n_chunks; ch += NW) {
        const int k0 = ch * 32 + piece * 8;
        uint16_t h[8];
        if (real && k0 + 8 <= d) {
            if (dtype == FS_BF16) {
                const u4_any v = *reinterpret_cast<const u4_any *>((const uint16_t *)pts + base + k0);
                const uint32_t q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) h[e] = (uint16_t)(q[e >> 1] >> (16 * (e & 1)));
            } else {
                const f4_any v0 = *reinterpret_cast<const f4_any *>((const float *)pts + base + k0);
                const f4_any v1 = *reinterpret_cast<const f4_any *>((const float *)pts + base + k0 + 4);
                const float q[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) h[e] = float_to_bf16(q[e]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                h[e] = 0;
                if (real && k0 + e < d)
                    h[e] = dtype == FS_BF16 ? ((const uint16_t *)pts)[base + k0 + e] : float_to_bf16(((const float *)pts)[base + k0 + e]);
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double v = (double)bf16_to_float(h[e]);
            nrm += v * v;
        }
        *reinterpret_cast<uint4 *>(dst + ((int64_t)ch << 14)) =
            make_uint4((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16), (uint32_t)h[4] | ((uint32_t)h[5] << 16),
                       (uint32_t)h[6] | ((uint32_t)h[7] << 16));
    }
    nrm += __shfl_xor(nrm, 1);
    nrm += __shfl_xor(nrm, 2);
    if (piece == 0) shn[w][l >> 2] = nrm;
    __syncthreads();
    if (tid < 16) {
        double sum = shn[0][tid];
#pragma unroll
        for (int k = 1; k < NW; ++k) sum += shn[k][tid];
        norm[rb * 16 + tid] = sum;
        bias[rb * 16 + tid] = -INFINITY;
    }
}

// ---- derived copies for 16 < d <= 128: the float64 records as above, and the digit images of the fixed-point
//      kernels (layout and digits: fs_fx.hip) ----------------------------------------------------------
// Floats as unsigned integers of the same order: -NaN < -inf < ... < inf < NaN
__device__ inline uint32_t order_key(float v)
{
    const uint32_t u = __float_as_uint(v);
    return u & 0x80000000u ? ~u : u | 0x80000000u;
}
__device__ inline float order_value(uint32_t k) { return __uint_as_float(k & 0x80000000u ? k & 0x7fffffffu : ~k); }

// smallest and largest of a workgroup of four waves, in every thread after the caller's barrier
__device__ inline void wave_range(uint32_t &mn, uint32_t &mx, uint2 *sh)
{
    for (int off = 32; off > 0; off >>= 1) {
        mn = min(mn, (uint32_t)__shfl_xor((int)mn, off, 64));
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
    }
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = make_uint2(mn, mx);
}

// stage 1: range of the coordinates of both clouds (as order keys), block b of side y writes part[y][b]
constexpr int kFxMaxBlocks = 128;
__global__ __launch_bounds__(256) void k_coord_range(CloudIn c0, CloudIn c1, int dtype, int d, uint2 *part)
{
    const CloudIn &cl = blockIdx.y ? c1 : c0;
    __shared__ uint2 sh[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t mn = 0xffffffffu, mx = 0;
    // eight rows in flight per wave: the loop is bound by the latency of its loads
    const int64_t step = (int64_t)gridDim.x * 4;
    for (int64_t i = (int64_t)blockIdx.x * 4 + wv; i < cl.rows; i += 8 * step)
        for (int k = lane; k < d; k += 64) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = load_pt(cl.pts, dtype, (i + q * step < cl.rows ? i + q * step : i) * cl.ld + k);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                mn = min(mn, order_key(v[q]));
                mx = max(mx, order_key(v[q]));
            }
        }
    wave_range(mn, mx, sh);
    __syncthreads();
    if (threadIdx.x == 0)
        part[blockIdx.y * kFxMaxBlocks + blockIdx.x] = make_uint2(min(min(sh[0].x, sh[1].x), min(sh[2].x, sh[3].x)),
                                                                  max(max(sh[0].y, sh[1].y), max(sh[2].y, sh[3].y)));
}

// stage 2: block = tile of 32 points.  Both clouds are shifted by the middle of the range of all their coordinates (the same
// shift for every coordinate; the cost does not change): coordinates of one sign, pixels for instance, get half the scale,
// which leaves a quarter of the error, and products of theirs have both signs, so that digits left out do not add up.  The
// shift is a multiple of 2^-7 r2, so a coordinate that is exact in fixed point stays exact; it is exact in the float64 records.
// The common scale r2 is the smallest power of two whose 127.49 / 128 covers the largest shifted coordinate, so the first
// digit stays within 127; a float's 24 bits are then kept exactly down to 2^-7 r2.
struct PrepFxSide {
    const void *pts;
    int64_t cnt, cnt_pad, ld;
    double *out, *bias, *norm;
    unsigned char *dig;
    int *brec;
};
// box, stamp: where the host learns r2 (see Prepared::box)
__global__ __launch_bounds__(256) void k_prep_fx(PrepFxSide s0, PrepFxSide s1, int dtype, int d, int kp, int ks, const uint2 *part,
                                                 double *r2_out, unsigned long long *box, uint32_t stamp)
{
    const PrepFxSide &sd = blockIdx.y ? s1 : s0;
    const int64_t row0 = (int64_t)blockIdx.x * 32;
    if (row0 >= sd.cnt_pad) return;
    __shared__ int pt[32][32 * kFxMaxKs + 1];
    __shared__ uint2 shm[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    static_assert(2 * kFxMaxBlocks == 256, "one partial range per thread");
    uint32_t mn = part[tid].x, mx = part[tid].y;
    wave_range(mn, mx, shm);
    // a wave takes eight rows, two coordinates per lane and row, all loads in flight
    float v[8][2];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const int64_t row = row0 + 8 * wv + q;
            const int k = lane + 64 * z;
            v[q][z] = (row < sd.cnt && k < d) ? load_pt(sd.pts, dtype, row * sd.ld + k) : 0.0f;
        }
    static_assert(32 * kFxMaxKs == 128, "two coordinates per lane");
    __syncthreads();
    const double lo = (double)order_value(min(min(shm[0].x, shm[1].x), min(shm[2].x, shm[3].x)));
    const double hi = (double)order_value(max(max(shm[0].y, shm[1].y), max(shm[2].y, shm[3].y)));
    int ex = 0;
    double r2 = 1.0, origin = 0.0, to_fixed = 0.0;
    if (!(lo > -INFINITY && hi < INFINITY))
        r2 = INFINITY;   // (the gate is off)
    else {
        // (126.99: the rounding of the shift is at most half a unit of the first digit)
        if (hi > lo) (void)frexp(0.5 * (hi - lo) * (128.0 / 126.99), &ex);
        r2 = ldexp(1.0, ex);
        origin = ldexp(rint(ldexp(0.5 * (hi + lo), 7 - ex)), ex - 7);
        to_fixed = ldexp(1.0, 31 - ex);
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
        r2_out[0] = r2;
        r2_out[1] = origin;
        if (box)
            __hip_atomic_store(box + kBoxFx, (unsigned long long)stamp << 32 | (unsigned)((r2 < INFINITY ? ex : kFxNoScale) & 0xffff),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t row = row0 + 8 * wv + q;
        double nrm = 0.0;
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const int k = lane + 64 * z;
            const double t = (row < sd.cnt && k < d) ? (double)v[q][z] - origin : 0.0;
            if (k < kp) {
                pt[8 * wv + q][k] = to_fixed > 0.0 ? (int)rint(t * to_fixed) : 0;
                sd.out[row * kp + k] = t;
            }
            nrm += t * t;
        }
        for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
        if (lane == 0) {
            sd.norm[row] = nrm;
            sd.bias[row] = -INFINITY;
        }
    }
    __syncthreads();
    for (int e = tid; e < ks * 64; e += 256) {
        const int q = e >> 6, l = e & 63;
        const int k0 = 32 * q + 16 * (l >> 5);
        uint4 o[4];
        fx_digits16(&pt[l & 31][k0], o);
#pragma unroll
        for (int dg = 0; dg < 4; ++dg)
            *reinterpret_cast<uint4 *>(sd.dig + ((((int64_t)blockIdx.x * ks + q) * 4 + dg) << 10) + l * 16) = o[dg];
    }
    if (tid < 128) sd.brec[(int64_t)blockIdx.x * 128 + tid] = tid >= 96 ? 1 : 0;   // flagged until biases come in
}

// ---- workspace potential (float64, unshifted) + bias from a user potential (float) -------
// `absmax` (optional) receives the largest finite |(pot - norm)/eps| log2e in absmax[1] and the
// largest finite |log w| log2e in absmax[0] (the two parts of a bias, which scale differently with
// eps), as bit patterns of non-negative doubles (for those, the order of the bit patterns is the
// order of the values)
// (FX here and below: the side has bias records of the fixed-point kernels, or two kernels may have written the statistics)
template <bool FX>
__global__ void k_bias_from_user(const float *pot_user, int64_t cnt, double inv_eps, const float *w,
                                 double log_uniform, double *pot, BiasSink sink, unsigned long long *absmax)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double mag_pot = 0.0, mag_w = 0.0, b = 0.0;
    if (i < cnt) {
        double pu = (double)pot_user[i];
        pot[i] = pu;
        double lw = w ? log((double)w[i]) : log_uniform;
        b = store_bias(sink, i, pu, inv_eps, lw);
        mag_pot = fabs((pu - sink.norm[i]) * inv_eps) * kLog2e;
        mag_w = fabs(lw) < INFINITY ? fabs(lw) * kLog2e : 0.0;   // zero-weight points never contribute
    }
    if constexpr (FX) store_fx_record(sink, i, cnt, b, inv_eps);
    if (absmax) {   // one pair of atomics per workgroup (256 threads)
        __shared__ double shm[2][4];
        for (int off = 32; off > 0; off >>= 1) {
            mag_pot = fmax(mag_pot, __shfl_xor(mag_pot, off));
            mag_w = fmax(mag_w, __shfl_xor(mag_w, off));
        }
        if ((threadIdx.x & 63) == 0) {
            shm[0][threadIdx.x >> 6] = mag_w;
            shm[1][threadIdx.x >> 6] = mag_pot;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            mag_w = fmax(fmax(shm[0][0], shm[0][1]), fmax(shm[0][2], shm[0][3]));
            mag_pot = fmax(fmax(shm[1][0], shm[1][1]), fmax(shm[1][2], shm[1][3]));
            if (mag_w > 0.0) atomicMax(absmax + 0, (unsigned long long)__double_as_longlong(mag_w));
            if (mag_pot > 0.0) atomicMax(absmax + 1, (unsigned long long)__double_as_longlong(mag_pot));
        }
    }
}

template <bool FX>
__device__ __forceinline__ void finalize_body(const FinalizeArgs &a, const int bx)
{
    // dev_part == nullptr: store the update.  dev_part != nullptr: measure the marginal deviation
    // only, unless save_old is given: then measure AND store, keeping the old potential in save_old.
    __shared__ double sh[256];
    if (bx == a.blocks) {   // (a workgroup of its own, launched where there is something to collect)
        if (a.gauge_prev_x)
            gauge_collect_pair(a.gauge_prev_x, a.gauge_prev_x_cnt, a.gauge_prev, a.gauge_prev_cnt, a.gauge_prev_eps,
                               a.gauge_scalars, sh);
        else
            gauge_collect(a.gauge_prev, a.gauge_prev_cnt, a.gauge_prev_eps, a.gauge_scalars, sh);
        return;
    }
    const int64_t i = (int64_t)bx * 256 + threadIdx.x;
    double dev = 0.0, mass = 0.0, bias = 0.0;
    const int splits = FX && !a.gate.on() ? a.splits_alt : a.splits;
    if (i < a.cnt) {
        constexpr int kOnce = 8;   // statistics read once into registers
        double2 ms[kOnce];
#pragma unroll
        for (int k = 0; k < kOnce; ++k)
            ms[k] = k < splits ? a.partial[(int64_t)k * a.stride + i] : make_double2(-INFINITY, 0.0);
        const PointIn p = load_point(a, i);
        double M = -INFINITY;
#pragma unroll
        for (int k = 0; k < kOnce; ++k) M = ms[k].x > M ? ms[k].x : M;
#pragma unroll 8
        for (int k = kOnce; k < splits; ++k) {
            double mk = a.partial[(int64_t)k * a.stride + i].x;
            M = mk > M ? mk : M;
        }
        double S = 0.0;
#pragma unroll
        for (int k = 0; k < kOnce; ++k)
            if (k < splits) S += rescale_split(ms[k].y, ms[k].x, M);
#pragma unroll 8
        for (int k = kOnce; k < splits; ++k) {
            double2 r = a.partial[(int64_t)k * a.stride + i];
            S += rescale_split(r.y, r.x, M);
        }
        finalize_point(a, i, p, M, S, &dev, &mass, &bias);
    }
    if (FX && a.inv_eps_next > 0.0 && (!a.dev_part || a.save_old)) store_fx_record(a.sink, i, a.cnt, bias, a.inv_eps_next);
    if (a.dev_part) {
        double t = block_sum_256(dev, sh);
        if (threadIdx.x == 0) a.dev_part[bx] = t;
    }
    if (a.gauge_out) {
        __syncthreads();
        double t = block_sum_256(mass, sh);
        if (threadIdx.x == 0) a.gauge_out[bx] = t;
    }
}

__global__ __launch_bounds__(256) void k_gauge_collect(const double *part, int64_t cnt, double eps, double *scalars)
{
    __shared__ double sh[256];
    gauge_collect(part, cnt, eps, scalars, sh);
}

__global__ __launch_bounds__(256) void k_gauge_collect_pair(const double *part_x, int64_t cnt_x, const double *part_y,
                                                            int64_t cnt_y, double eps, double *scalars)
{
    __shared__ double sh[256];
    gauge_collect_pair(part_x, cnt_x, part_y, cnt_y, eps, scalars, sh);
}

// f_user = (float)(x_pot - scalars[1]) for i < n, g_user = (float)(y_pot + scalars[0]) for the next m indices
__global__ void k_gauge_export(const double *x_pot, int64_t n, const double *y_pot, int64_t m, const double *scalars,
                               float *f_user, float *g_user)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        f_user[i] = (float)(x_pot[i] - scalars[1]);
    else if (i < n + m)
        g_user[i - n] = (float)(y_pot[i - n] + scalars[0]);
}

// (Bound by latency: loads, two logarithms in double, a sum over the workgroup.  6.1 us at 10000 rows and 6 splits with each load where
// it is used, the statistics read twice and the collection done by the first workgroup before its rows; 4.8 like this.)
template <bool FX>
__global__ __launch_bounds__(256) void k_finalize(FinalizeArgs a) { finalize_body<FX>(a, blockIdx.x); }

// the merges of the two passes of an averaged iteration (Eq. 4-5) in one launch
template <bool FX>
__global__ __launch_bounds__(256) void k_finalize_pair(FinalizeArgs a0, FinalizeArgs a1)
{
    const int b = (int)blockIdx.x, all = a0.blocks + a1.blocks;
    if (b < a0.blocks || b == all)   // (the last one collects, see finalize_body)
        finalize_body<FX>(a0, b == all ? a0.blocks : b);
    else
        finalize_body<FX>(a1, b - a0.blocks);
}

__global__ void k_export_f32(const double *src, int64_t cnt, float *dst)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cnt) dst[i] = (float)src[i];
}

// sum of `cnt` doubles by one block, fixed order
__global__ __launch_bounds__(256) void k_sum_to(const double *part, int64_t cnt, double *dst)
{
    __shared__ double sh[256];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < cnt; i += 256) acc += part[i];
    double t = block_sum_256(acc, sh);
    if (threadIdx.x == 0) *dst = t;
}

// the five sums of the dual objective's terms in one launch: block k < 3 sums pr[k][0..br), block 3 + k
// sums ps[k][0..bs), each in a fixed order
__global__ __launch_bounds__(256) void k_sum_value_terms(const double *pr, int64_t br, const double *ps, int64_t bs, double *dst)
{
    __shared__ double sh[256];
    const int k = blockIdx.x;
    const double *part = k < 3 ? pr + (int64_t)k * br : ps + (int64_t)(k - 3) * bs;
    const int64_t cnt = k < 3 ? br : bs;
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < cnt; i += 256) acc += part[i];
    const double t = block_sum_256(acc, sh);
    if (threadIdx.x == 0) dst[k] = t;
}

// ---- terms of the dual objective (App. B) -------------------------------------------------
// After an LSE pass over `res`: mass_i = w_i exp((pot_i - pot_i^+)/eps) is the row sum of the plan
// that the CURRENT potentials induce (Prop. 3).  Block sums of mass_i, w_i pot_i and w_i go to
// part[0][.], part[1][.], part[2][.] (part has 3 * gridDim.x doubles).
template <bool FX>
__global__ __launch_bounds__(256) void k_value_terms(const double2 *partial, int64_t stride, int splits_n, int splits_alt, FxGate gate, int64_t cnt,
                                                     double eps, const float *w, double log_uniform,
                                                     const double *res_norm, const double *pot, double *part)
{
    __shared__ double sh[256];
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double t[3] = {0.0, 0.0, 0.0};
    const int splits = FX && !gate.on() ? splits_alt : splits_n;
    if (i < cnt) {
        double M = -INFINITY;
#pragma unroll 8
        for (int k = 0; k < splits; ++k) {
            double mk = partial[(int64_t)k * stride + i].x;
            M = mk > M ? mk : M;
        }
        double S = 0.0;
#pragma unroll 8
        for (int k = 0; k < splits; ++k) {
            double2 ms = partial[(int64_t)k * stride + i];
            S += rescale_split(ms.y, ms.x, M);
        }
        const double pot_new = -eps * kLn2 * (M + log2(S)) + res_norm[i];
        const double wi = w ? (double)w[i] : exp(log_uniform);
        t[0] = wi > 0.0 ? wi * exp((pot[i] - pot_new) / eps) : 0.0;
        t[1] = wi * pot[i];
        t[2] = wi;
    }
    for (int k = 0; k < 3; ++k) {
        double v = block_sum_256(t[k], sh);
        if (threadIdx.x == 0) part[(int64_t)k * gridDim.x + blockIdx.x] = v;
        __syncthreads();
    }
}

// block counts of the entries that are NaN or infinite
__global__ __launch_bounds__(256) void k_count_nonfinite(const float *v, int64_t cnt, double *part)
{
    __shared__ double sh[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const double t = (i < cnt && !(fabsf(v[i]) < INFINITY)) ? 1.0 : 0.0;
    const double s = block_sum_256(t, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// block sums of the weights (part[0][.]) and of the indicator "not positive and finite" (part[1][.])
__global__ __launch_bounds__(256) void k_weight_stats(const float *w, int64_t cnt, double *part)
{
    __shared__ double sh[256];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double t[2] = {0.0, 0.0};
    if (i < cnt) {
        const float v = w[i];
        const bool ok = v > 0.0f && v < INFINITY;
        t[0] = ok ? (double)v : 0.0;
        t[1] = ok ? 0.0 : 1.0;
    }
    for (int k = 0; k < 2; ++k) {
        double s = block_sum_256(t[k], sh);
        if (threadIdx.x == 0) part[(int64_t)k * gridDim.x + blockIdx.x] = s;
        __syncthreads();
    }
}

// block sums of w_i pot_i and w_i: part[0][.], part[1][.]
__global__ __launch_bounds__(256) void k_weighted_sums(int64_t cnt, const float *w, double log_uniform, const double *pot,
                                                       double *part)
{
    __shared__ double sh[256];
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double t[2] = {0.0, 0.0};
    if (i < cnt) {
        const double wi = w ? (double)w[i] : exp(log_uniform);
        t[0] = wi * pot[i];
        t[1] = wi;
    }
    for (int k = 0; k < 2; ++k) {
        double v = block_sum_256(t[k], sh);
        if (threadIdx.x == 0) part[(int64_t)k * gridDim.x + blockIdx.x] = v;
        __syncthreads();
    }
}

// merge the splits of an application pass and apply the epilogue of Alg. 2:
//   out_i = a_i * exp(fhat_i/eps + m_i) * O_i   with everything in base 2;  mass_i = same with s.
// A block of 256 threads covers 256 / PC rows; thread (row, c) produces one output entry, so the
// reads of the [splits][rows][PC] accumulators are contiguous; the row's max and factor are
// computed once (by its thread c = 0) and shared.  (When PC does not divide 256 the last 256 % PC threads idle.)
struct ApplyFinalizeArgs {
    const double2 *partial;
    int64_t stride;
    const float *opart;
    int64_t opart_stride;
    int PC, splits, PC_alt, splits_alt;   // (alt: where the gate chose the float64 kernel of the pass)
    FxGate gate;
    int64_t cnt;
    double inv_eps;
    const float *w;
    double log_uniform;
    const double *pot, *res_norm;
    int p0, p;
    float *out;
    int64_t ldo;
    float *mass_out;
};
// ALT: one of two kernels wrote the accumulators, with rows of different length, so a block may take several groups of rows
// (see the launch)
template <bool ALT>
__global__ __launch_bounds__(256) void k_apply_finalize(ApplyFinalizeArgs a)
{
    __shared__ double shM[256], shFac[256];
    const bool alt = ALT && !a.gate.on();
    const int PC = alt ? a.PC_alt : a.PC, splits = alt ? a.splits_alt : a.splits;
    const int rows_per_block = 256 / PC;
    const int rl = threadIdx.x / PC, c = threadIdx.x - rl * PC;
    for (int64_t base = (int64_t)blockIdx.x * rows_per_block; base < a.cnt; base += (int64_t)gridDim.x * rows_per_block) {
        const int64_t i = rl < rows_per_block ? base + rl : a.cnt;   // (idle threads: no row)
        if (c == 0 && i < a.cnt) {
            double M = -INFINITY;
#pragma unroll 8
            for (int k = 0; k < splits; ++k) {
                double mk = a.partial[(int64_t)k * a.stride + i].x;
                M = mk > M ? mk : M;
            }
            double lw = a.w ? log((double)a.w[i]) : a.log_uniform;
            // row factor  a_i * exp(fhat_i/eps + m_i): add the exponents BEFORE exponentiating
            const double fac = exp2(((a.pot[i] - a.res_norm[i]) * a.inv_eps + lw) * kLog2e + M);
            shM[rl] = M;
            shFac[rl] = fac;
            if (a.mass_out && a.p0 == 0) {
                double S = 0.0;
#pragma unroll 8
                for (int k = 0; k < splits; ++k) {
                    double2 ms = a.partial[(int64_t)k * a.stride + i];
                    S += rescale_split(ms.y, ms.x, M);
                }
                a.mass_out[i] = (float)(fac * S);
            }
        }
        __syncthreads();
        if (i < a.cnt && a.p0 + c < a.p) {
            const double M = shM[rl];
            double acc = 0.0;
#pragma unroll 4
            for (int k = 0; k < splits; ++k) {
                const double mk = a.partial[(int64_t)k * a.stride + i].x;
                acc += rescale_split((double)a.opart[((int64_t)k * a.opart_stride + i) * PC + c], mk, M);
            }
            a.out[i * a.ldo + a.p0 + c] = (float)(shFac[rl] * acc);
        }
        if (!ALT) break;
        __syncthreads();
    }
}

// `eps`: the eps of the pass that will stream these biases
// `rho_on_device`: the host does not know rho_max yet (prologue of an entry call): the kernel
// derives the grid from the device scalar
BiasSink sink_of(const Prepared *P, const Side *s, double eps, bool rho_on_device = false)
{
    BiasSink k{};
    k.split_p = s->split_p;
    if (s->split_p && eps > 0.0) {
        if (rho_on_device) {
            k.q = 0.0;
            k.rho_dev = P->scalars + 7;
            k.q_eps = eps;
        } else {
            double gx, gy;
            split_grids(P->rho_max, eps, &gx, &gy);
            k.q = gx * gy;
        }
    } else {
        k.split_p = nullptr;
    }
    k.packed = s->packed;
    k.packed_d = s->packed_d;
    k.split = s->split;
    k.ks = P->ks;
    k.dp = P->dp;
    k.dpd = P->dpd;
    k.d = (int)P->d;
    k.bias_f = s->bias_f;
    k.bias_d = s->bias_d;
    k.brec = s->brec;
    k.r2 = P->scalars + 10;
    k.norm_f = s->norm_f;
    k.norm = s->norm;
    return k;
}

}  // namespace

fs_status launch_apply_finalize(Ctx *c, const Prepared *P, const Side *res, const double *res_norm, Splits splits,
                                double eps, const float *opart, int PC, int p0, int p, float *out, int64_t ldo,
                                float *mass_out, int PC_alt)
{
    if (PC < 1 || PC > 256 || (splits.alt && (PC_alt < 1 || PC_alt > 256))) return fail(c, FS_ERR_DEVICE, "internal: accumulator width of the application merge");
    const ApplyFinalizeArgs a{(const double2 *)P->partial, res->cnt_pad, opart,           res->cnt_pad, PC,       splits.n,  PC_alt, splits.alt, fx_gate(P, eps),
                              res->cnt,                    1.0 / eps,    res->w,          res->log_uniform,       res->pot,  res_norm, p0,       p,
                              out,                         ldo,          mass_out};
    int64_t blocks = ceil_div(res->cnt, 256 / PC);
    if (splits.alt) {
        // enough blocks for either kernel's rows, up to 2048 for the other's: with the main kernel's grid alone (one column:
        // 256 rows a block, eleven blocks at n = 2600) the 64-column rows of the fp64 kernel took 64 rounds, 240 us instead of 8
        const int64_t other = ceil_div(res->cnt, 256 / PC_alt);
        const int64_t enough = other < 2048 ? other : 2048;
        if (enough > blocks) blocks = enough;
        hipLaunchKernelGGL(k_apply_finalize<true>, dim3((unsigned)blocks), dim3(256), 0, c->stream, a);
    } else
        hipLaunchKernelGGL(k_apply_finalize<false>, dim3((unsigned)blocks), dim3(256), 0, c->stream, a);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

// float copy of a point matrix (bf16 storage) for use as the value matrix of a plan application
__global__ void k_pts_to_f32(const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld, float *dst)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * d) return;
    // (a 64-bit division costs more than the rest of an entry)
    const int64_t i = rows * d < (int64_t(1) << 32) ? (int64_t)((uint32_t)e / (uint32_t)d) : e / d, k = e - i * d;
    dst[e] = load_pt(pts, dtype, i * ld + k);
}

// Gradient assembly on top of T = (plan applied to the other cloud), in place in `g` (rows x d):
//   mode 0: 2 (w_i z_i - T_i)        Cor. 4, w the given weights (uniform 1/rows when NULL)
//   mode 1: 2 (mass_i z_i - T_i)     the same with the plan's own marginal (appendix on gradients)
//   mode 2: z_i - T_i / w_i          displacement to the barycentric image
__global__ void k_grad_assemble(float *g, int64_t ldg, const void *pts, int dtype, int64_t ld, int64_t rows, int64_t d,
                                const float *w, double uniform_w, const float *mass, int mode)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * d) return;
    // (a 64-bit division costs more than the rest of an entry)
    const int64_t i = rows * d < (int64_t(1) << 32) ? (int64_t)((uint32_t)e / (uint32_t)d) : e / d, k = e - i * d;
    const double z = (double)load_pt(pts, dtype, i * ld + k);
    const double t = (double)g[i * ldg + k];
    const double wi = w ? (double)w[i] : uniform_w;
    double r;
    if (mode == 0)
        r = 2.0 * (wi * z - t);
    else if (mode == 1)
        r = 2.0 * ((double)mass[i] * z - t);
    else
        r = z - t / wi;
    g[i * ldg + k] = (float)r;
}

// ---- label-augmented cost  l1 |x_i - y_j|^2 + l2 W[lx_i, ly_j]  (Section 3.1's remark on generalised costs; the
// appendix on the dataset-distance application).  The table lookup is itself a contraction,
// W[lx, ly] = <onehot(lx), W[:, ly]>, so V more coordinates carry it through the score contraction of every kernel:
//     xa_i = [x_i, onehot(lx_i)],   ya_j = [y_j, u_j],  u_j = -(l2 / 2 l1) W[:, ly_j]
//     l1 |xa_i - ya_j|^2 = l1 |x_i - y_j|^2 + l2 W[lx_i, ly_j] + l1 + v_j,   v_j = l1 |u_j|^2,
// a cost that differs from the wanted one by per-point constants only, which the potentials absorb exactly.
// In bf16 mode u is rounded to bfloat16 here, so that v_j is taken from the values the matrix cores will see.
// Labels outside [0, V) are counted in *bad (and read as class 0).
__global__ void k_label_augment(const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld, const int32_t *labels,
                                const float *W, int V, int target_side, double half_ratio, double l1, int round_bf16,
                                float *out, float *vconst, unsigned *bad)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows) return;
    int lab = labels[i];
    if (lab < 0 || lab >= V) {
        atomicAdd(bad, 1u);
        lab = 0;
    }
    float *o = out + i * (d + V);
    for (int64_t k = 0; k < d; ++k) o[k] = load_pt(pts, dtype, i * ld + k);
    double v = 0.0;
    for (int k = 0; k < V; ++k) {
        float u;
        if (target_side) {
            u = (float)(-half_ratio * (double)W[(int64_t)k * V + lab]);
            if (round_bf16) u = bf16_to_float(float_to_bf16(u));
            v += (double)u * (double)u;
        } else {
            u = k == lab ? 1.0f : 0.0f;
        }
        o[d + k] = u;
    }
    if (vconst) vconst[i] = (float)(l1 * v);
}

// potentials of the labelled problem <-> potentials of the augmented one:  p' = (p + shift) / l1  and back
__global__ void k_label_potential(const float *src, const float *vconst, double cshift, double l1, int to_augmented,
                                  int64_t cnt, float *dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cnt) return;
    const double sh = cshift + (vconst ? (double)vconst[i] : 0.0);
    dst[i] = to_augmented ? (float)(((double)src[i] + sh) / l1) : (float)((double)src[i] * l1 - sh);
}

fs_status launch_label_augment(Ctx *c, const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld,
                               const int32_t *labels, const float *W, int V, bool target_side, double l1, double l2,
                               bool round_bf16, float *out, float *vconst, unsigned *bad)
{
    hipLaunchKernelGGL(k_label_augment, dim3((unsigned)ceil_div(rows, 128)), dim3(128), 0, c->stream, pts, dtype, rows, d, ld,
                       labels, W, V, target_side ? 1 : 0, l2 / (2.0 * l1), l1, round_bf16 ? 1 : 0, out, vconst, bad);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

fs_status launch_label_potential(Ctx *c, const float *src, const float *vconst, double cshift, double l1, bool to_augmented,
                                 int64_t cnt, float *dst)
{
    hipLaunchKernelGGL(k_label_potential, dim3((unsigned)ceil_div(cnt, 256)), dim3(256), 0, c->stream, src, vconst, cshift, l1,
                       to_augmented ? 1 : 0, cnt, dst);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

fs_status launch_pts_to_f32(Ctx *c, const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld, float *dst)
{
    hipLaunchKernelGGL(k_pts_to_f32, dim3((unsigned)ceil_div(rows * d, 256)), dim3(256), 0, c->stream, pts, dtype, rows, d,
                       ld, dst);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

fs_status launch_grad_assemble(Ctx *c, float *g, int64_t ldg, const void *pts, int dtype, int64_t ld, int64_t rows,
                               int64_t d, const float *w, const float *mass, int mode)
{
    hipLaunchKernelGGL(k_grad_assemble, dim3((unsigned)ceil_div(rows * d, 256)), dim3(256), 0, c->stream, g, ldg, pts, dtype,
                       ld, rows, d, w, 1.0 / (double)rows, mass, mode);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

fs_status launch_export_f32(Ctx *c, const double *src, int64_t cnt, float *dst)
{
    hipLaunchKernelGGL(k_export_f32, dim3((unsigned)ceil_div(cnt, 256)), dim3(256), 0, c->stream, src, cnt, dst);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

fs_status launch_fill_f64(Ctx *c, double *dst, double v, int64_t cnt)
{
    hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)ceil_div(cnt, 256)), dim3(256), 0, c->stream, dst, v, cnt);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

fs_status launch_row_norms(Ctx *c, const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld, float *out)
{
    hipLaunchKernelGGL(k_row_norms, dim3((unsigned)ceil_div(rows, 256)), dim3(256), 0, c->stream, pts, dtype, rows, d,
                       ld, out);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

// (of the whole process: contexts share the box of the static scratch array)
static uint32_t next_stamp()
{
    static std::atomic<uint32_t> last{0};
    uint32_t s = ++last;
    if (s == 0) s = ++last;
    return s;
}

fs_status launch_prepare(Ctx *c, const fs_problem *p, Prepared *P)
{
    const int dtype = p->dtype;
    struct In { const void *pts; int64_t ld; Side *S; };
    In in[2] = {{p->x, p->ldx, &P->X}, {p->y, p->ldy, &P->Y}};
    if (P->path == Path::LowD) {
        // the reserved area holds 16 doubles (mean) + 2 x 128 x 16 doubles (per-block sums of x, of y)
        const int half = 128;
        double *partX = P->mean + kLowdMaxD;
        double *partY = partX + (size_t)half * kLowdMaxD;
        const CloudIn cx{p->x, p->n, p->ldx, partX}, cy{p->y, p->m, p->ldy, partY};
        const int64_t pad_max = P->X.cnt_pad > P->Y.cnt_pad ? P->X.cnt_pad : P->Y.cnt_pad;
        PrepLowdSide sd[2];
        for (int k = 0; k < 2; ++k) {
            const Side *S = in[k].S;
            sd[k] = PrepLowdSide{in[k].pts, S->cnt, S->cnt_pad, in[k].ld, S->packed, S->packed_d, S->norm_f, S->norm, S->split,
                                 S->pts_d,   S->bias_d};
        }
        if ((double)(p->n + p->m) * (double)p->d <= kSmallPrologue && !P->mom.base) {
            hipLaunchKernelGGL(k_prep_lowd_small, dim3((unsigned)ceil_div(pad_max, 256), 2), dim3(1024), 0, c->stream, sd[0], sd[1], dtype,
                               (int)p->d, P->dp, P->dpd, P->kp, P->ks, P->X.split_p, P->Y.split_p, P->mean, P->scalars + 5);
            P->rho_max = -1.0;
            FS_HIP(c, hipGetLastError());
            return FS_OK;
        }
        // (bounds of the clouds only where half-steps may run through cell moments)
        const bool bounds = P->mom.base != nullptr;
        hipLaunchKernelGGL(k_coord_sums, dim3(half, 2), dim3(256), 0, c->stream, cx, cy, dtype, (int)p->d, bounds);
        // (also clears scalars[5..7]: the sizes of the biases and the largest squared norm, all taken by atomic maxima)
        hipLaunchKernelGGL(k_mean_final, dim3(1), dim3(256), 0, c->stream, partX, partY, half,
                           1.0 / (double)(p->n + p->m), P->mean, P->scalars + 5, (int)p->d, bounds ? P->scalars + kScalarBounds : nullptr);
        hipLaunchKernelGGL(k_prep_lowd, dim3((unsigned)ceil_div(pad_max, 256), 2), dim3(256), 0, c->stream, sd[0], sd[1], dtype,
                           (int)p->d, P->dp, P->dpd, P->kp, P->mean, P->ks, reinterpret_cast<unsigned long long *>(P->scalars + 7));
        // (the host reads rho_max back together with the sizes of the biases, see launch_bias_from_user)
        P->rho_max = -1.0;
        if (p->d <= 3)   // the grid of the precise records' leading digits depends on rho_max
            hipLaunchKernelGGL(k_prep_split_precise, dim3((unsigned)ceil_div(pad_max, 256), 2), dim3(256), 0, c->stream,
                               P->X.packed_d, P->X.cnt_pad, P->X.split_p, P->Y.packed_d, P->Y.cnt_pad, P->Y.split_p, (int)p->d,
                               P->dpd, P->scalars + 7);
        FS_HIP(c, hipGetLastError());
    } else if (P->path == Path::F64 && P->fx_ks) {
        uint2 *part = reinterpret_cast<uint2 *>(P->mean);
        const CloudIn cx{p->x, p->n, p->ldx, nullptr}, cy{p->y, p->m, p->ldy, nullptr};
        hipLaunchKernelGGL(k_coord_range, dim3(kFxMaxBlocks, 2), dim3(256), 0, c->stream, cx, cy, dtype, (int)p->d, part);
        PrepFxSide sd[2];
        for (int k = 0; k < 2; ++k) {
            const Side *S = in[k].S;
            sd[k] = PrepFxSide{in[k].pts, S->cnt, S->cnt_pad, in[k].ld, S->pts_d, S->bias_d, S->norm, S->dig, S->brec};
        }
        const int64_t pad_max = P->X.cnt_pad > P->Y.cnt_pad ? P->X.cnt_pad : P->Y.cnt_pad;
        // (A graph does not write to the box: no launch of the call is decided by what its replays would leave there, and a replay may
        // come after fs_destroy, which frees the box, while a graph of fs_solve_noalloc holds no other memory of the context.)
        unsigned long long *const box = capturing(c) ? nullptr : P->box;
        if (box) P->fx_stamp = next_stamp();
        hipLaunchKernelGGL(k_prep_fx, dim3((unsigned)(pad_max / 32), 2), dim3(256), 0, c->stream, sd[0], sd[1], dtype, (int)p->d, P->kp,
                           P->fx_ks, part, P->scalars + 10, box, P->fx_stamp);
    } else if (P->path == Path::F64) {
        for (auto &s : in)
            hipLaunchKernelGGL(k_prep_f64, dim3((unsigned)ceil_div(s.S->cnt_pad, 4)), dim3(256), 0, c->stream, s.pts,
                               dtype, s.S->cnt, s.S->cnt_pad, p->d, s.ld, P->kp, s.S->pts_d, s.S->bias_d, s.S->norm);
    } else {
        // Few rows do not fill the chip, and four waves walk through many chunks each, one after the other: sixteen there.  A half-step in
        // fp32 storage, us, with a wave per row as it was before / four waves / sixteen: n = m = 100, d = 500: 28.3 / 30.5 / 27.9, d = 1024: 39.9 / 44.1 /
        // 37.6, d = 2048: 63.8 / 72.5 / 58.9; n = m = 2000, d = 1024: 47.7 / 48.6 / 43.9; d = 256, n = m = 1000: 25.1 / 24.1 / 23.7.  From
        // n = m = 3000 on the four are ahead of the wave per row (54.1 / 51.9 at d = 1024).
        for (auto &s : in) {
            const dim3 grid((unsigned)(s.S->cnt_pad / 16));
            if (s.S->cnt_pad <= 2048 && P->kp >= 256)
                hipLaunchKernelGGL(k_prep_bf16<16>, grid, dim3(1024), 0, c->stream, s.pts, dtype, s.S->cnt, p->d, s.ld, P->kp, s.S->pts_b,
                                   s.S->bias_f, s.S->norm);
            else
                hipLaunchKernelGGL(k_prep_bf16<4>, grid, dim3(256), 0, c->stream, s.pts, dtype, s.S->cnt, p->d, s.ld, P->kp, s.S->pts_b,
                                   s.S->bias_f, s.S->norm);
        }
    }
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

__global__ __launch_bounds__(64) void k_publish(const double *src, int cnt, unsigned long long *box, uint32_t stamp)
{
    const int t = threadIdx.x;
    if (t >= 2 * cnt) return;
    const unsigned long long v = (unsigned long long)__double_as_longlong(src[t >> 1]);
    __hip_atomic_store(box + t, (unsigned long long)stamp << 32 | (t & 1 ? v >> 32 : v & 0xffffffffull), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// cnt doubles of the device in dst, once everything before has run.  The GPU is idle from here until the host has them and the next
// launch arrives; with a copy to host memory and a wait for the stream, two half-step calls at n = 1000, m = 777, d = 3 took 82 us,
// with a kernel that writes to pinned memory and a host that looks there 59 (kernels 44).  Where the stream has long work
// ahead of it, the host stops looking after a fifth of a millisecond and waits for the stream.
// All reads of a call go this way: a copy behind kernels that the host has not waited for costs more than one behind a wait (dual
// value at n = 200, m = 150, d = 3: prologue and value by copies 71 us, prologue through the box and value by a copy 80, both through
// the box 46; a half-step and fs_check_finite at n = m = 3000, d = 3 73, 87 and 62).
fs_status read_back(Ctx *c, const double *src, int cnt, double *dst)
{
    static_assert(kBoxLowd + 2 * kMostReadBack <= kBoxWords && kMostReadBack <= 32, "scalars fit the box, and a wave of k_publish");
    unsigned long long *const box = c->ws_static ? c->static_box : c->box;
    if (!box) {
        FS_HIP(c, hipMemcpyAsync(dst, src, cnt * sizeof(double), hipMemcpyDeviceToHost, c->stream));
        FS_HIP(c, hipStreamSynchronize(c->stream));
        return FS_OK;
    }
    const uint32_t stamp = next_stamp();
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, c->stream, src, cnt, box + kBoxLowd, stamp);
    FS_HIP(c, hipGetLastError());
    const auto t0 = std::chrono::steady_clock::now();
    bool waited = false;
    for (int k = 0; k < 2 * cnt;) {
        const unsigned long long w = __atomic_load_n(box + kBoxLowd + k, __ATOMIC_RELAXED);
        if ((uint32_t)(w >> 32) == stamp) {
            uint32_t half = (uint32_t)w;
            memcpy(reinterpret_cast<char *>(dst) + 4 * k, &half, 4);
            ++k;
        } else if (waited)
            return fail(c, FS_ERR_DEVICE, "scalars of the prologue did not arrive");
        else if (std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(200)) {
            FS_HIP(c, hipStreamSynchronize(c->stream));
            waited = true;
        }
    }
    return FS_OK;
}

fs_status launch_bias_from_user(Ctx *c, Prepared *P, Side *side, const float *pot_user, double eps, bool first, bool last)
{
    // low-d problems: the size of the bias enters the choice of the score precision (lowd_precise),
    // so it is measured where a caller's potential comes in; it is read back together with the
    // largest squared norm, once per entry call (three doubles)
    unsigned long long *absmax = nullptr;
    if (P->path == Path::LowD) {
        absmax = reinterpret_cast<unsigned long long *>(P->scalars + 5);   // scalars[5], [6]
        if (first && !(P->rho_max < 0.0)) {   // (a fresh prologue has cleared them already)
            fs_status st = launch_fill_f64(c, P->scalars + 5, 0.0, 2);
            if (st != FS_OK) return st;
        }
    }
    hipLaunchKernelGGL(P->fx_ks ? k_bias_from_user<true> : k_bias_from_user<false>, dim3((unsigned)ceil_div(side->cnt, 256)), dim3(256), 0, c->stream, pot_user,
                       side->cnt, 1.0 / eps, side->w, side->log_uniform, side->pot, sink_of(P, side, eps, P->rho_max < 0.0),
                       absmax);
    FS_HIP(c, hipGetLastError());
    if (absmax && last) {
        double h[kScalarBounds - 5 + 12] = {};   // |log w| part, potential part, rho_max; at the end bounds of the clouds, see k_mean_final
        const fs_status st = read_back(c, P->scalars + 5, P->mom.base ? (int)(sizeof h / sizeof *h) : 3, h);
        if (st != FS_OK) return st;
        static_assert(sizeof h / sizeof *h <= kMostReadBack, "read back at once");
        if (h[0] > P->logw_mag) P->logw_mag = h[0];
        if (h[1] * eps > P->pot_mag_eps) P->pot_mag_eps = h[1] * eps;
        P->rho_max = h[2];
        const double *b = h + kScalarBounds - 5;
        for (int s = 0; s < 2 && P->mom.base; ++s)
            for (int k = 0; k < 3; ++k) {
                P->mom.lo[s][k] = b[6 * s + k];
                P->mom.hi[s][k] = b[6 * s + 3 + k];
            }
        if (c->kept_valid) c->kept_rho_max = h[2];   // belongs to the kept derived copies (no-op when they are another problem's)
    }
    return FS_OK;
}

static FinalizeArgs finalize_args(const Prepared *P, const void *partial, Side *res, const double *res_norm, Splits splits,
                                  double eps_cur, double eps_next_bias, float *user_out, double *dev_part, double mix,
                                  double *save_old)
{
    FinalizeArgs a{};
    a.partial = (const double2 *)partial;
    a.stride = res->cnt_pad;
    a.splits = splits.n;
    a.splits_alt = splits.alt;
    a.gate = fx_gate(P, eps_cur);
    a.cnt = res->cnt;
    a.eps = eps_cur;
    a.inv_eps_next = eps_next_bias > 0.0 ? 1.0 / eps_next_bias : 0.0;
    a.w = res->w;
    a.log_uniform = res->log_uniform;
    a.res_norm = res_norm;
    a.pot = res->pot;
    a.sink = sink_of(P, res, eps_next_bias);
    a.user_out = user_out;
    a.dev_part = dev_part;
    a.mix = mix;
    a.save_old = save_old;
    a.blocks = (int)ceil_div(res->cnt, 256);
    return a;
}

fs_status launch_gauge_export(Ctx *c, const Prepared *P, int64_t collect_last, double eps_last, const double *x_pot,
                              float *f_user, float *g_user)
{
    if (collect_last)
        hipLaunchKernelGGL(k_gauge_collect, dim3(1), dim3(256), 0, c->stream, P->gauge_part, collect_last, eps_last, P->scalars + 8);
    hipLaunchKernelGGL(k_gauge_export, dim3((unsigned)ceil_div(P->X.cnt + P->Y.cnt, 256)), dim3(256), 0, c->stream, x_pot,
                       P->X.cnt, P->Y.pot, P->Y.cnt, P->scalars + 8, f_user, g_user);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

static void set_gauge(FinalizeArgs *a, const Prepared *P, GaugeMode gauge, int64_t prev_cnt, double prev_eps)
{
    if (gauge == GaugeMode::Measure) a->gauge_out = P->gauge_part;
    if (gauge == GaugeMode::Collect && prev_cnt > 0) {
        a->gauge_prev = P->gauge_part;
        a->gauge_prev_cnt = prev_cnt;
        a->gauge_prev_eps = prev_eps;
        a->gauge_scalars = P->scalars + 8;
    }
}

FinalizeArgs make_finalize_args(const Prepared *P, Side *res, const double *res_norm, double eps_cur, double eps_next_bias,
                                float *user_out, GaugeMode gauge, int64_t gauge_prev_cnt, double gauge_prev_eps)
{
    FinalizeArgs a = finalize_args(P, nullptr, res, res_norm, Splits(), eps_cur, eps_next_bias, user_out, nullptr, 1.0, nullptr);
    set_gauge(&a, P, gauge, gauge_prev_cnt, gauge_prev_eps);
    return a;
}

fs_status launch_finalize(Ctx *c, const Prepared *P, Side *res, const double *res_norm, Splits splits, double eps_cur,
                          double eps_next_bias, float *user_out, double *abs_dev_sum, double mix, double *save_old,
                          GaugeMode gauge, int64_t gauge_prev_cnt, double gauge_prev_eps)
{
    double *dev_part = abs_dev_sum ? P->dev_part : nullptr;   // per-block sums of the marginal deviation
    FinalizeArgs a = finalize_args(P, P->partial, res, res_norm, splits, eps_cur, eps_next_bias, user_out, dev_part,
                                   mix, save_old);
    set_gauge(&a, P, gauge, gauge_prev_cnt, gauge_prev_eps);
    hipLaunchKernelGGL(P->fx_ks ? k_finalize<true> : k_finalize<false>, dim3((unsigned)(a.blocks + (a.gauge_prev ? 1 : 0))), dim3(256), 0, c->stream, a);
    if (abs_dev_sum)
        hipLaunchKernelGGL(k_sum_to, dim3(1), dim3(256), 0, c->stream, dev_part, (int64_t)a.blocks, abs_dev_sum);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

// merges of the f-pass (records in partial_x) and of the g-pass (partial_y) in one launch
fs_status launch_finalize_pair(Ctx *c, const Prepared *P, Side *X, const double *norm_x, const void *partial_x, Splits splits_x,
                               float *f_out, Side *Y, const double *norm_y, const void *partial_y, Splits splits_y,
                               float *g_out, double eps_cur, double eps_next_bias, double mix, int gauge_parity, bool collect_prev)
{
    FinalizeArgs ax = finalize_args(P, partial_x, X, norm_x, splits_x, eps_cur, eps_next_bias, f_out, nullptr, mix, nullptr);
    FinalizeArgs ay = finalize_args(P, partial_y, Y, norm_y, splits_y, eps_cur, eps_next_bias, g_out, nullptr, mix, nullptr);
    if (gauge_parity >= 0) {
        // the sums of this iteration go to one half of the two arrays while a workgroup of its own
        // collects the previous iteration's from the other half
        const int64_t nbx = ceil_div(X->cnt, 256), nby = ceil_div(Y->cnt, 256);
        const int64_t half = nbx > nby ? nbx : nby;
        ax.gauge_out = P->gauge_part_x + (gauge_parity & 1) * half;
        ay.gauge_out = P->gauge_part + (gauge_parity & 1) * half;
        if (collect_prev) {
            ax.gauge_prev = P->gauge_part + ((gauge_parity & 1) ^ 1) * half;
            ax.gauge_prev_cnt = nby;
            ax.gauge_prev_x = P->gauge_part_x + ((gauge_parity & 1) ^ 1) * half;
            ax.gauge_prev_x_cnt = nbx;
            ax.gauge_prev_eps = eps_cur;
            ax.gauge_scalars = P->scalars + 8;
        }
    }
    hipLaunchKernelGGL(P->fx_ks ? k_finalize_pair<true> : k_finalize_pair<false>,
                       dim3((unsigned)(ax.blocks + ay.blocks + (ax.gauge_prev ? 1 : 0))), dim3(256), 0, c->stream, ax, ay);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

// the term of the last averaged iteration (its sums sit in half `gauge_parity` of the two arrays)
fs_status launch_gauge_collect_pair(Ctx *c, const Prepared *P, double eps, int gauge_parity)
{
    const int64_t nbx = ceil_div(P->X.cnt, 256), nby = ceil_div(P->Y.cnt, 256);
    const int64_t half = nbx > nby ? nbx : nby;
    hipLaunchKernelGGL(k_gauge_collect_pair, dim3(1), dim3(256), 0, c->stream, P->gauge_part_x + (gauge_parity & 1) * half, nbx,
                       P->gauge_part + (gauge_parity & 1) * half, nby, eps, P->scalars + 8);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

// dst[0] <- how many of the cnt floats are NaN or infinite; `scratch` holds one double per 256 values
fs_status launch_count_nonfinite(Ctx *c, const float *v, int64_t cnt, double *scratch, double *dst)
{
    const unsigned nb = (unsigned)ceil_div(cnt, 256);
    hipLaunchKernelGGL(k_count_nonfinite, dim3(nb), dim3(256), 0, c->stream, v, cnt, scratch);
    hipLaunchKernelGGL(k_sum_to, dim3(1), dim3(256), 0, c->stream, scratch, (int64_t)nb, dst);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

// dst[0] <- sum of the weights, dst[1] <- how many of them are not positive and finite; `scratch` holds
// 2 * blocks doubles
fs_status launch_weight_stats(Ctx *c, const float *w, int64_t cnt, double *scratch, double *dst)
{
    const unsigned nb = (unsigned)ceil_div(cnt, 256);
    hipLaunchKernelGGL(k_weight_stats, dim3(nb), dim3(256), 0, c->stream, w, cnt, scratch);
    hipLaunchKernelGGL(k_sum_to, dim3(1), dim3(256), 0, c->stream, scratch, (int64_t)nb, dst);
    hipLaunchKernelGGL(k_sum_to, dim3(1), dim3(256), 0, c->stream, scratch + nb, (int64_t)nb, dst + 1);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

// dst[0..4] <- sum_i mass_i, <w_res, pot_res>, sum w_res, <w_str, pot_str>, sum w_str  (see k_value_terms);
// `scratch` holds 3 * blocks(res) + 2 * blocks(str) doubles
fs_status launch_value_terms(Ctx *c, const Prepared *P, const Side *res, const double *res_norm, const Side *str,
                             Splits splits, double eps, double *scratch, double *dst)
{
    const unsigned br = (unsigned)ceil_div(res->cnt, 256), bs = (unsigned)ceil_div(str->cnt, 256);
    double *pr = scratch, *ps = scratch + 3 * (size_t)br;
    hipLaunchKernelGGL(P->fx_ks ? k_value_terms<true> : k_value_terms<false>, dim3(br), dim3(256), 0, c->stream, (const double2 *)P->partial, res->cnt_pad, splits.n,
                       splits.alt, fx_gate(P, eps), res->cnt, eps, res->w, res->log_uniform, res_norm, res->pot, pr);
    hipLaunchKernelGGL(k_weighted_sums, dim3(bs), dim3(256), 0, c->stream, str->cnt, str->w, str->log_uniform, str->pot, ps);
    hipLaunchKernelGGL(k_sum_value_terms, dim3(5), dim3(256), 0, c->stream, pr, (int64_t)br, ps, (int64_t)bs, dst);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

}  // namespace fs
