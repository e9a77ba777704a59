// Half-steps at d <= 3 through cell moments: the row sums  S_i = sum_j 2^(cscale <x_i, y_j> + bias_j)  without an exponential
// per pair.
//
// Both clouds are dealt to a grid of cells.  With x in a cell of centre x0 and y in one of centre y0, dx = x - x0, dy = y - y0,
//     cscale <x, y> = cscale (<x0, y0> + <dx, y0> + <x0, dy>) + log2(e) t,      t = 2 <dx, dy> / eps,
// and only e^t couples a row to a streamed point of its own.  |t| <= tau by the choice of the cells, and there e^t is a polynomial
// of degree p to 3e-8 of itself (half an ulp of the float exponential that it takes the place of): with s_k = hx_k hy_k / (2 eps),
// xi and eta the coordinates of dx and dy in half cells,
//     e^t = sum over |alpha| <= p of  c_alpha xi^alpha eta^alpha,    c_alpha = a_|alpha| |alpha|! / alpha! prod s_k^alpha_k,
// a_n the coefficients of the truncated Chebyshev series of e^t on [-tau, tau].  So a cell of streamed points acts on a cell of
// rows through its moments  M_alpha = sum_j 2^(bias_j + cscale <x0, dy_j>) eta_j^alpha  (k_mom_gather), and
//     S_i = sum over cells of  2^(cscale (<x0, y0> + <dx_i, y0>)) sum_alpha c_alpha xi_i^alpha M_alpha   (k_mom_rows).
// The error is relative to every single term (the factors taken out are exact), so it holds for any potentials.  The
// expansion is the one of the fast Gauss transform (Greengard and Strain, SIAM J. Sci. Stat. Comput. 12 (1991); total degree as
// in Yang, Duraiswami, Gumerov and Davis, ICCV 2003) without its translation operators, which would not keep relative errors.
//
// Both steps are contractions, over the points of a cell and over the moments, and run on the fp16 matrix cores
// (v_mfma_f32_32x32x16_f16) from operands in two fp16 pieces, 22 bits: per 32 cells a point costs 32 .. 224 products instead of an
// exponential per pair.  Everything that a potential or a product of full coordinates enters is float64 up to a difference that is
// small where it counts: biases against the largest of a block, cell pairs against the largest of a row cell.
//
// What is held in fewer bits than over the pairs: weights, monomials and moments (22 bits there), and the series (3e-8).  Exponents are
// floats of at most 48 (points of a cell) and 96 (rows) in size, differences that are no larger than the scores of the pairs and round no
// more (2e-6 and 4e-6 of a term at most).  So
// moments stand for fp32 scores only; where float64-grade ones are asked for (lowd_precise, and every measurement) passes run over
// the pairs.  Errors of a half-step in units of eps (rms of f and of g against 64 bits; n = 20021, m = 18013) here, over the pairs with
// fp32 scores, and what rounding f to float costs:
//     d = 3, cube     eps 0.01 1.3e-7 7e-8   2.6e-6 2.6e-6   1.1e-7      d = 2, cube     eps 0.01 1.4e-7 1.0e-7  1.9e-6 1.9e-6   1.1e-7
//                     0.03     1.0e-7 5e-8   2.3e-7 2.1e-7   0.9e-7                      0.03     1.1e-7 0.9e-7  2.1e-7 1.9e-7   0.7e-7
//                     0.1      0.9e-7 6e-8   1.1e-7 0.8e-7   0.6e-7                      0.1      0.8e-7 0.6e-7  0.9e-7 0.6e-7   0.4e-7
//                     1        0.7e-7 8e-8   0.5e-7 0.3e-7   0.1e-7                      1        0.6e-7 1.0e-7  0.5e-7 0.3e-7   0.1e-7
//             mixture 0.01     3.1e-7 9e-8   2.2e-6 2.7e-6   2.9e-7              mixture 0.01     2.7e-7 1.0e-7  1.7e-6 1.7e-6   2.5e-7
//             normal  0.3      1.5e-7 7e-8   4.2e-7 4.1e-7   1.4e-7              normal  0.3      1.5e-7 1.3e-7  3.4e-7 3.8e-7   1.0e-7
// so they are nearer up to an eps of about a tenth of the squared extent, and beyond it (where a cloud is a few cells and nothing averages) off by
// 1e-7 to 2e-7 instead of 2e-8 to 5e-8.  A spare monomial with what two pieces leave of the moment of degree 0 did not change that.
// Sums are formed in a fixed order (the sort is stable), so a result does not depend on the run.
//
// Measured (half-step of a solve, us, over the pairs and here): n = m = 262144, d = 3, mixture / cube, eps = 0.01: 5900 -> 1290 / 1700, 0.046:
// 5900 -> 207 / 202, 1: 5900 -> 76 / 73; n = 50021, m = 40013, cube, eps = 0.05: 219 -> 48.
// Bound at large sizes: what a SIMD's two waves do not overlap of the vector, matrix and LDS instructions of k_mom_gather (a weight
// costs its exponential, three fma and the split, 110 instructions per 16 points and 32 cells beside 21 products at RT = 7; products
// alone would take a third of its time), products of k_mom_rows (three quarters of its loop); at small ones latency, the gather takes
// 8 us without its loops (as the rows did, 4 less now).
// What helps both is that the two waves of a SIMD (w and w + 4) do not do the same at a time, so that one's products run beside the
// other's vector instructions, that reads from LDS are on their way before they are waited for, where the compiler would place each
// at its use, and that a workgroup's constants and first tiles are asked for with its points.  At n = m = 262144 and RT = 7: gather of
// 763 blocks for 384 cells 350 -> 304 us, rows of 568 groups over 1331 cells 336 -> 259.
// Tried since: the exponents as fp32 products on the matrix cores, 295 us for 310, but 30 for 28.6 where a wave has every other
// k-step, and other roundings; four tiles of monomials at a time and two workgroups per CU, weights formed twice: 302, 31.8; powers
// of 512 points at a time, or monomials over four workgroups: no change.
// Tried, as the whole call of four stages of one iteration at n = m = 262144 (48 ms over the pairs, 4.8 here then): fp32 matrix
// instructions 9.4 ms; three bf16 pieces and six products 6.7 with every wave forming the monomials for itself (their LDS reads
// bound it), 6.9 with shared ones and moments as floats split by the rows' kernel.
#include <math.h>

#include <new>

#include "fs_internal.h"

namespace fs {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));

// Power tables in LDS: row = power (see pow_stride), then ones, biases, values; column = point
constexpr int kOne = 30, kBias = 31, kValue = 32;
constexpr int kTabRows = 33;
// Stored moments are below 2^8 and coefficients have a factor 2^10, so that what fp16 drops of small ones does not count; the
// moments' exponents take both out.
constexpr int kMomShift = 8, kCoefShift = 10;
constexpr int kSortBins = kMomMaxCells;

// ---- the monomials -----------------------------------------------------------------------------------------------
// kind: dimension, degree, number of monomials and how many tiles of 32 they take.  tau: where the truncated series is off by
// 3e-8 of e^t.
struct Kind {
    int d, p, cnt, rt;
    double tau;
};
constexpr int kKinds = 7;
constexpr Kind kKind[kKinds] = {{3, 5, 56, 2, 0.284}, {3, 7, 120, 4, 0.725}, {3, 9, 220, 7, 1.313}, {2, 6, 28, 1, 0.482},
                                {2, 9, 55, 2, 1.313}, {2, 14, 120, 4, 3.126}, {1, 9, 10, 1, 1.313}};
constexpr int kMaxTerms = kMomTerms;
// By falling degree, so that a row's sum meets its small terms first and the constant one, the largest, last.  An entry holds
// the rows of the three powers in a power table (power e of coordinate k at k stride + e) and the degree.
struct Basis {
    uint32_t e[kKinds][kMaxTerms];
};
constexpr int pow_stride(int d) { return d == 2 ? 15 : 10; }
constexpr Basis make_basis()
{
    Basis b{};
    for (int k = 0; k < kKinds; ++k) {
        const int d = kKind[k].d, p = kKind[k].p, st = pow_stride(d);
        int at = 0;
        for (int n = p; n >= 0; --n)
            for (int i = n; i >= 0; --i) {
                if (d == 1 && i != n) continue;
                for (int j = n - i; j >= 0; --j) {
                    const int l = n - i - j;
                    if (d < 3 && l != 0) continue;
                    b.e[k][at++] = (uint32_t)i | (uint32_t)(d > 1 ? st + j : kOne) << 8 | (uint32_t)(d > 2 ? 2 * st + l : kOne) << 16 |
                                   (uint32_t)n << 24;
                }
            }
        for (; at < kMaxTerms; ++at) b.e[k][at] = (uint32_t)kOne | (uint32_t)kOne << 8 | (uint32_t)kOne << 16 | 0xff000000u;
    }
    return b;
}
constexpr Basis kBasisHost = make_basis();
__device__ const Basis kBasis = make_basis();

// powers of a point's coordinates in half cells
template <int STRIDE> __device__ __forceinline__ void fill_powers(float *tab, const int pt, const float4 v, const int d, const float first = 1.0f)
{
    const int st = pow_stride(d);
    const float c[3] = {v.x, v.y, v.z};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (k >= d) break;
        float *o = tab + k * st * STRIDE + pt;
        float q = k ? 1.0f : first;
        for (int e = 0; e < st; ++e) {
            o[e * STRIDE] = q;
            q *= c[k];
        }
    }
    tab[kOne * STRIDE + pt] = 1.0f;
}

// Two fp16 pieces of eight floats (22 bits; what is below 2^-24 counts nothing here: monomials are at most 1, weights and moments
// are scaled to near the top of the range) and the three piece products that matter, small ones first
__device__ __forceinline__ void split8(const float (&v)[8], h8 (&o)[2])
{
#pragma unroll
    for (int z = 0; z < 8; z += 2) {
        float x = v[z], y = v[z + 1];
        // (opaque: the compiler folds the product that v comes from into one of the two conversions of it, and where that rounds
        // once instead of twice the pieces are a leading digit apart)
        asm("" : "+v"(x), "+v"(y));
        h2 hi{(_Float16)x, (_Float16)y};
        asm("" : "+v"(hi));   // (or it converts each a second time for the difference)
        // (x - hi in one instruction, which takes its fp16 operand from either half: 16 instructions for eight floats, not 32)
        float dx, dy;
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(dx) : "v"(hi), "v"(x));
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(dy) : "v"(hi), "v"(y));
        const h2 lo{(_Float16)dx, (_Float16)dy};
        o[0][z] = hi[0], o[0][z + 1] = hi[1];
        o[1][z] = lo[0], o[1][z + 1] = lo[1];
    }
}
__device__ __forceinline__ f16v mm2(const h8 (&a)[2], const h8 (&b)[2], f16v c)
{
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[1], c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[0], c, 0, 0, 0);
}

__device__ __forceinline__ void cell_centre(const MomGeom &g, int bin, double (&c)[3])
{
    const int i = bin % g.nc[0], j = bin / g.nc[0] % g.nc[1], l = bin / (g.nc[0] * g.nc[1]);
    c[0] = g.lo[0] + (i + 0.5) * g.h[0];
    c[1] = g.lo[1] + (j + 0.5) * g.h[1];
    c[2] = g.lo[2] + (l + 0.5) * g.h[2];
}

// ---- dealing the points to the cells: a stable counting sort ----------------------------------------------------
struct SortSide {
    const double *pts;   // centred coordinates [.][dpd]
    int64_t cnt, chunk;  // points, and how many of them a workgroup takes
    int ncell, chunks, block;
    MomGeom g;
    MomSide s;
};
__device__ __forceinline__ int cell_of(const SortSide &a, const double *p, const int d)
{
    int idx = 0;
#pragma unroll
    for (int k = 2; k >= 0; --k) {
        const double q = k < d && a.g.h[k] > 0.0 ? (p[k] - a.g.lo[k]) / a.g.h[k] : 0.0;
        const int i = q > 0.0 ? min(a.g.nc[k] - 1, (int)q) : 0;
        idx = idx * a.g.nc[k] + i;
    }
    return idx;
}
// (blockIdx.y here and in the next kernels: 0 = the x cloud, 1 = the y cloud)
__global__ __launch_bounds__(256) void k_mom_hist(SortSide s0, SortSide s1, int d, int dpd)
{
    const SortSide &a = blockIdx.y ? s1 : s0;
    if ((int)blockIdx.x >= a.chunks) return;
    __shared__ int bins[kSortBins];
    for (int b = threadIdx.x; b < a.ncell; b += 256) bins[b] = 0;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * a.chunk, i1 = min(a.cnt, i0 + a.chunk);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const int key = cell_of(a, a.pts + i * dpd, d);
        a.s.key[i] = (uint16_t)key;
        atomicAdd(&bins[key], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < a.ncell; b += 256) a.s.hist[(int64_t)blockIdx.x * a.ncell + b] = bins[b];
}
// per cell: what the chunks before a chunk hold of it, and its total
__global__ __launch_bounds__(256) void k_mom_scan(SortSide s0, SortSide s1)
{
    const SortSide &a = blockIdx.y ? s1 : s0;
    const int b = (int)blockIdx.x * 256 + threadIdx.x;
    if (b >= a.ncell) return;
    int acc = 0;
    for (int c0 = 0; c0 < a.chunks; c0 += 8) {
        int v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = c0 + q < a.chunks ? a.s.hist[(int64_t)(c0 + q) * a.ncell + b] : 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (c0 + q < a.chunks) a.s.hist[(int64_t)(c0 + q) * a.ncell + b] = acc;
            acc += v[q];
        }
    }
    a.s.total[b] = acc;
}
// one workgroup per side: where each cell's points start, the cells that hold points, their blocks of at most SortSide::block
// streamed points and their groups of at most kMomRows rows
__global__ __launch_bounds__(1024) void k_mom_lists(SortSide s0, SortSide s1)
{
    const SortSide &a = blockIdx.y ? s1 : s0;
    constexpr int Q = kSortBins / 1024;
    __shared__ int4 wsum[16];   // (.y: cells, and in the upper half those of several blocks)
    __shared__ int fb[kSortBins + 1], fr[kSortBins + 1];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int4 own = make_int4(0, 0, 0, 0);   // points, cells, blocks, groups of rows
    int cnt[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = tid * Q + q;
        cnt[q] = b < a.ncell ? a.s.total[b] : 0;
        own.x += cnt[q];
        own.y += (cnt[q] > 0) + (cnt[q] > a.block ? 1 << 16 : 0);
        own.z += (cnt[q] + a.block - 1) / a.block;
        own.w += (cnt[q] + kMomRows - 1) / kMomRows;
    }
    int4 inc = own;
    for (int off = 1; off < 64; off <<= 1) {
        const int4 o = make_int4(__shfl_up(inc.x, off), __shfl_up(inc.y, off), __shfl_up(inc.z, off), __shfl_up(inc.w, off));
        if (lane >= off) inc = make_int4(inc.x + o.x, inc.y + o.y, inc.z + o.z, inc.w + o.w);
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    int4 at = make_int4(inc.x - own.x, inc.y - own.y, inc.z - own.z, inc.w - own.w), all = make_int4(0, 0, 0, 0);
    for (int w = 0; w < 16; ++w) {
        const int4 o = wsum[w];
        if (w < wv) at = make_int4(at.x + o.x, at.y + o.y, at.z + o.z, at.w + o.w);
        all = make_int4(all.x + o.x, all.y + o.y, all.z + o.z, all.w + o.w);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = tid * Q + q;
        if (b < a.ncell) a.s.total[b] = at.x;   // (from here on: where the cell starts)
        if (cnt[q] > 0) {
            const int k = at.y & 65535, several = cnt[q] > a.block;
            a.s.cell[k] = make_int4(b, at.x, cnt[q], 0);
            fb[k] = at.z;
            fr[k] = at.w;
            if (several) a.s.several[at.y >> 16] = k;
            at = make_int4(at.x + cnt[q], at.y + 1 + (several << 16), at.z + (cnt[q] + a.block - 1) / a.block, at.w + (cnt[q] + kMomRows - 1) / kMomRows);
        }
    }
    const int nseveral = all.y >> 16;
    all.y &= 65535;
    if (tid == 0) {
        fb[all.y] = all.z;
        fr[all.y] = all.w;
    }
    __syncthreads();
    for (int k = tid; k <= all.y; k += 1024) {
        a.s.first_block[k] = fb[k];
        a.s.first_rows[k] = fr[k];
    }
    if (tid == 0) {
        a.s.counts[0] = all.y;
        a.s.counts[1] = all.z;
        a.s.counts[2] = all.w;
        a.s.counts[3] = nseveral;
    }
    // (cut at multiples of `unit`)
    auto fill = [&](const int *first, int total, int4 *out, int unit) {
        for (int b = tid; b < total; b += 1024) {
            int lo = 0, hi = all.y;   // first[lo] <= b < first[hi]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (first[mid] <= b)
                    lo = mid;
                else
                    hi = mid;
            }
            const int4 c = a.s.cell[lo];
            const int parts = first[lo + 1] - first[lo], k = b - first[lo];
            const int64_t units = (c.z + unit - 1) / unit;
            const int s = (int)(units * k / parts) * unit, e = min(c.z, (int)(units * (k + 1) / parts) * unit);
            out[b] = make_int4(lo, c.y + s, e - s, 0);
        }
    };
    fill(fb, all.z, a.s.block, 1);
    fill(fr, all.w, a.s.rows, 32);
    for (int k = tid; k < all.y; k += 1024) {
        double c[3];
        cell_centre(a.g, a.s.cell[k].x, c);
        a.s.centre[k] = make_double4(c[0], c[1], c[2], 0.0);
    }
}
// each wave takes a quarter of the workgroup's chunk, 64 points at a time, in order
__global__ __launch_bounds__(256) void k_mom_scatter(SortSide s0, SortSide s1, int d, int dpd)
{
    const SortSide &a = blockIdx.y ? s1 : s0;
    if ((int)blockIdx.x >= a.chunks) return;
    // [4][kSortBins] 16-bit places inside the chunk's share of a cell (a chunk has at most 2^15 points)
    __shared__ uint32_t place32[2 * kSortBins];
    uint16_t *place = reinterpret_cast<uint16_t *>(place32);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int w = 0; w < 4; ++w)
        for (int b = tid; b < (a.ncell + 1) / 2; b += 256) place32[w * (kSortBins / 2) + b] = 0;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * a.chunk, i1 = min(a.cnt, i0 + a.chunk);
    const int64_t quarter = (i1 - i0 + 255) / 256 * 64;
    const int64_t q0 = min(i1, i0 + wv * quarter), q1 = min(i1, q0 + quarter);
    for (int64_t i = q0 + lane; i < q1; i += 64) {
        const int key = a.s.key[i];
        atomicAdd(place32 + wv * (kSortBins / 2) + (key >> 1), key & 1 ? 65536u : 1u);
    }
    __syncthreads();
    for (int b = tid; b < a.ncell; b += 256) {
        int at = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int n = place[w * kSortBins + b];
            place[w * kSortBins + b] = (uint16_t)at;
            at += n;
        }
    }
    __syncthreads();
    volatile uint16_t *mine = place + wv * kSortBins;
    const int *before = a.s.hist + (int64_t)blockIdx.x * a.ncell;
    for (int64_t i = q0; i < q1; i += 64) {   // (uniform over the wave)
        const bool in = i + lane < q1;
        const int key = in ? (int)a.s.key[i + lane] : 0;
        unsigned long long same = __ballot(in);
#pragma unroll
        for (int bit = 0; bit < 13; ++bit) {
            const unsigned long long v = __ballot(key >> bit & 1);
            same &= key >> bit & 1 ? v : ~v;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1));
        int pos = 0;
        if (in) pos = mine[key] + rank;
        __builtin_amdgcn_wave_barrier();
        if (in && rank == 0) mine[key] = (uint16_t)(pos + (int)__popcll(same));
        __builtin_amdgcn_wave_barrier();
        if (in) pos += a.s.total[key] + before[key];
        if (in) {
            const double *p = a.pts + (i + lane) * dpd;
            double c[3];
            cell_centre(a.g, key, c);
            float v[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (k < d && a.g.h[k] > 0.0) v[k] = (float)((p[k] - c[k]) * 2.0 / a.g.h[k]);
            a.s.perm[pos] = (int)(i + lane);
            a.s.xi[pos] = make_float4(v[0], v[1], v[2], 0.0f);
        }
    }
}
static_assert(kMomMaxCells <= 1 << 13, "bits of a key in k_mom_scatter");

// ---- moments of the blocks ---------------------------------------------------------------------------------------
struct GatherArgs {
    const int4 *block;           // blocks of the streamed side
    const double4 *centre;       // of the row cells, from the launch's first one on
    const float4 *xi;
    const int *perm;
    const double *bias;          // bias of point i at bias[i bstride]
    int bstride, nblock, ncells; // cells of the launch
    MomGeom sg;
    double cscale;
    int d, kind;
    int rt, tsplit;              // tiles of monomials, and over how many workgroups they are spread
    int halves;                  // see k_mom_gather
    const float *V;              // applications: the values, of any size; moments of 1 and of each column
    int64_t ldv;
    float *ex;                   // [1 + columns][cells of the launch][nblock] power of two of the moments, -inf: all are zero
    unsigned char *M;            // [1 + columns][cells of the launch][nblock] moments: 32 RT leading pieces, then 32 RT trailing ones
};
// One workgroup of eight waves: TW tiles of 32 monomials (of the RT of an expansion) of one block, for 8 tiles of 32 row cells, or
// for 4 where `halves` is set; then waves w and w + 4 share their cells and take every other k-step of 16 points each.
// A stage is 32 points.  Their monomials (A operand: a lane holds those of eight points) are formed once for all waves, in two
// fp16 pieces in LDS, while the stage before is multiplied; a wave's own are the weights of the points for its 32 cells (B operand:
// eight exponentials per lane and k-step).  Waves 0 to 3 form their share of the next stage's monomials before this stage's products,
// waves 4 to 7 after them.
template <int TW>
__global__ __launch_bounds__(512, 2) void k_mom_gather(GatherArgs a)
{
    constexpr int ST = kMomBlock + 4, kStage = 2 * TW * 2 * 1024;
    __shared__ __attribute__((aligned(1024))) unsigned char frag[2][kStage];
    __shared__ __attribute__((aligned(16))) float tab[kTabRows * ST];
    __shared__ double wmax[8];
    __shared__ float vmax[8];
    const int tid = threadIdx.x, l = tid & 63, lh = l >> 5, lj = l & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int4 blk = a.block[blockIdx.x];
    const int col = blockIdx.z / a.tsplit, t0 = (blockIdx.z - col * a.tsplit) * TW, nt = min(TW, a.rt - t0);
    // this thread's points of the block, tid and tid + 512 (a block has at most 1024)
    double ub[2] = {-INFINITY, -INFINITY};   // (points beyond the block's end weigh nothing)
    float4 xb[2];
    float vb[2] = {1.0f, 1.0f};
    // the matrix cores truncate downwards where they align a product to an accumulator: every other sum runs over negated weights
    const float sign = blockIdx.x & 1 ? -1.0f : 1.0f;
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        xb[z] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (tid + 512 * z < blk.z) {
            const int64_t j = a.perm[blk.y + tid + 512 * z];
            xb[z] = a.xi[blk.y + tid + 512 * z];
            ub[z] = a.bias[j * a.bstride];
            if (col) vb[z] = a.V[j * a.ldv + col - 1];
        } else if (col)
            vb[z] = 0.0f;
    }
    const int xt = a.halves ? (int)blockIdx.y * 4 + (w & 3) : (int)blockIdx.y * 8 + w;
    const int cell = xt * 32 + lj;
    const bool busy = xt * 32 < a.ncells;
    const int ks0 = a.halves ? w >> 2 : 0, ks1 = !busy ? ks0 : a.halves ? ks0 + 1 : 2;
    const bool late = w >= 4;   // (the other wave of this SIMD is not)
    const double4 c0 = a.centre[min(cell, a.ncells - 1)];
    const float tilt[3] = {sign * (float)(a.cscale * c0.x * 0.5 * a.sg.h[0]), a.d > 1 ? (float)(a.cscale * c0.y * 0.5 * a.sg.h[1]) : 0.0f,
                           a.d > 2 ? (float)(a.cscale * c0.z * 0.5 * a.sg.h[2]) : 0.0f};
    const int st = pow_stride(a.d);
    const int p1 = (a.d > 1 ? st + 1 : kOne) * ST, p2 = (a.d > 2 ? 2 * st + 1 : kOne) * ST;
    // this thread's units of a stage: (k-step, tile, lane) = eight points of one monomial
    constexpr int NU = (2 * TW * 64 + 511) / 512;
    int uo[NU][3];
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const int u = tid + 512 * i, ul = u & 63, ut = (u >> 6) % TW, uk = (u >> 6) / TW;
        const uint32_t e = kBasis.e[a.kind][min(32 * (t0 + ut) + (ul & 31), kMaxTerms - 1)];
        const int pt = 16 * uk + 8 * (ul >> 5);
        uo[i][0] = (e & 255) * ST + pt;
        uo[i][1] = (e >> 8 & 255) * ST + pt;
        uo[i][2] = (e >> 16 & 255) * ST + pt;
    }
    // Values are of any size and weights close to the end of the fp16 range: a power of two that takes the block's largest value
    // below 1 comes out of them (vexp).
    double top = fmax(ub[0], ub[1]);
    float vtop = fmaxf(fabsf(vb[0]), fabsf(vb[1]));
    for (int off = 32; off > 0; off >>= 1) {
        top = fmax(top, __shfl_xor(top, off));
        vtop = fmaxf(vtop, __shfl_xor(vtop, off));
    }
    if (l == 0) {
        wmax[w] = top;
        vmax[w] = vtop;
    }
    __syncthreads();
    top = wmax[0];
    vtop = vmax[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) {
        top = fmax(top, wmax[k]);
        vtop = fmaxf(vtop, vmax[k]);
    }
    top = ceil(top);
    const int vexp = col && vtop > 0.0f ? ilogbf(vtop) + 1 : 0;
#pragma unroll
    for (int z = 0; z < 2; ++z) vb[z] = ldexpf(vb[z], -vexp);

    auto eight = [&](const float *p, float (&o)[8]) __attribute__((always_inline)) {
        const float4 x = *reinterpret_cast<const float4 *>(p), y = *reinterpret_cast<const float4 *>(p + 4);
        o[0] = x.x, o[1] = x.y, o[2] = x.z, o[3] = x.w, o[4] = y.x, o[5] = y.y, o[6] = y.z, o[7] = y.w;
    };
    auto monomials = [&](int pt, unsigned char *out) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const int u = tid + 512 * i;
            if (NU * 512 != 2 * TW * 64 && u >= 2 * TW * 64) break;
            float m[8], c[2][8];
            eight(tab + uo[i][0] + pt, m);
            eight(tab + uo[i][1] + pt, c[0]);
            eight(tab + uo[i][2] + pt, c[1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int z = 0; z < 8; ++z) m[z] = m[z] * c[0][z] * c[1][z];
            h8 o[2];
            split8(m, o);
#pragma unroll
            for (int k = 0; k < 2; ++k) *reinterpret_cast<h8 *>(out + ((u >> 6) * 2 + k) * 1024 + (u & 63) * 16) = o[k];
        }
    };
    // weights are 2^(exponent - off): off moves when one would leave the fp16 range
    float off = -1.0e30f, mass = 0.0f;
    f16v acc[TW];
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
    for (int base = 0; base < blk.z; base += kMomBlock) {
        const int cnt = min(kMomBlock, blk.z - base);
        if (base) __syncthreads();
        if ((tid >> 8) == (base >> 8 & 1)) {
            const int z = base >> 9, i = tid & 255;
            const double u = z ? ub[1] : ub[0];
            fill_powers<ST>(tab, i, z ? xb[1] : xb[0], a.d, sign);
            tab[kBias * ST + i] = u == -INFINITY ? -INFINITY : (float)(u - top);
            tab[kValue * ST + i] = z ? vb[1] : vb[0];
        }
        __syncthreads();
        monomials(0, frag[0]);
        int cur = 0;
        for (int pt = 0; pt < cnt; pt += 32, cur ^= 1) {
            __syncthreads();   // this stage's monomials are there, and the other buffer is read
            const bool more = pt + 32 < cnt;
            if (more && !late) monomials(pt + 32, frag[cur ^ 1]);
            for (int ks = ks0; ks < ks1; ++ks) {
                const float *q = tab + pt + 16 * ks + 8 * lh;
                float e[8], x[3][8];
                eight(q + kBias * ST, e);
                eight(q + ST, x[0]);
                eight(q + p1, x[1]);
                eight(q + p2, x[2]);
                __builtin_amdgcn_sched_barrier(0);   // (all reads on their way before the first wait)
                float big = -INFINITY;
#pragma unroll
                for (int z = 0; z < 8; ++z) {
                    e[z] = fmaf(tilt[2], x[2][z], fmaf(tilt[1], x[1][z], fmaf(tilt[0], x[0][z], e[z])));
                    big = fmaxf(big, e[z]);
                }
                if (__any(big > off + 14.0f)) {
                    big = fmaxf(big, __shfl_xor(big, 32));   // (the products run over both lane halves)
                    const float now = big > off + 14.0f ? ceilf(big) - 8.0f : off, f = __builtin_amdgcn_exp2f(off - now);
                    off = now;
                    mass *= f;
#pragma unroll
                    for (int t = 0; t < TW; ++t)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[t][r] *= f;
                }
#pragma unroll
                for (int z = 0; z < 8; ++z) e[z] = __builtin_amdgcn_exp2f(e[z] - off);
                if (col) {
                    eight(q + kValue * ST, x[0]);
#pragma unroll
                    for (int z = 0; z < 8; ++z) e[z] *= x[0][z];
                }
                mass += ((fabsf(e[0]) + fabsf(e[1])) + (fabsf(e[2]) + fabsf(e[3]))) + ((fabsf(e[4]) + fabsf(e[5])) + (fabsf(e[6]) + fabsf(e[7])));
                asm("" : "+v"(mass));   // (here: later, the weights would be copied for it)
                h8 eb[2];
                split8(e, eb);
                const unsigned char *f = frag[cur] + ks * (TW * 2 * 1024) + l * 16;
                // a tile's monomials are read two tiles before their products (the compiler would read them right there, and wait)
                h8 ma[3][2];
                auto operand = [&](int t) __attribute__((always_inline)) {
#pragma unroll
                    for (int k = 0; k < 2; ++k) ma[t % 3][k] = *reinterpret_cast<const h8 *>(f + (t * 2 + k) * 1024);
                };
                operand(0);
                if (TW > 1) operand(1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < TW; ++t) {
                    if (t + 2 < TW) operand(t + 2);
                    acc[t] = mm2(ma[t % 3], eb, acc[t]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (more && late) monomials(pt + 32, frag[cur ^ 1]);
        }
    }
    mass += __shfl_xor(mass, 32);
    // Sixteen floats of a lane and tile are four groups of four neighbouring monomials of one cell.
    if (a.halves) {
        __shared__ float4 other[4 * 4 * 64];
        __shared__ float2 scale[8][32];
        if (lh == 0) scale[w][lj] = make_float2(off, mass);
        __syncthreads();
        const float2 o2 = scale[w ^ 4][lj];
        const float now = fmaxf(off, o2.x), f = __builtin_amdgcn_exp2f(off - now), g2 = __builtin_amdgcn_exp2f(o2.x - now);
        off = now;
        mass = mass * f + o2.y * g2;
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            __syncthreads();
            if (w >= 4) {
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    other[((w & 3) * 4 + g) * 64 + l] =
                        make_float4(acc[t][4 * g] * f, acc[t][4 * g + 1] * f, acc[t][4 * g + 2] * f, acc[t][4 * g + 3] * f);
            }
            __syncthreads();
            if (w < 4) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 o = other[(w * 4 + g) * 64 + l];
                    acc[t][4 * g] = fmaf(acc[t][4 * g], f, o.x);
                    acc[t][4 * g + 1] = fmaf(acc[t][4 * g + 1], f, o.y);
                    acc[t][4 * g + 2] = fmaf(acc[t][4 * g + 2], f, o.z);
                    acc[t][4 * g + 3] = fmaf(acc[t][4 * g + 3], f, o.w);
                }
            }
        }
        if (w >= 4) return;
    }
    if (cell < a.ncells) {
        // the moments are at most the weights' sum: stored as 2^(power of two above it) times two fp16 pieces
        // (A mass of 1 has values of 2^-7 of the block's largest where the weights are.  From 2^-60 down what there is of it is
        // nothing beside the rounding of the others, and its scale would leave the range of a float.)
        float up = 0.0f, ex = -INFINITY;
        if (mass > 0x1p-60f) {
            const int sc = ilogbf(mass) + 1;
            up = ldexpf(sign, kMomShift - sc);
            ex = (float)top + off + (float)(sc - kMomShift - kCoefShift + vexp);
        }
        if (mass != mass) ex = up = NAN;
        const int64_t at = ((int64_t)col * a.ncells + cell) * a.nblock + blockIdx.x;
        if (t0 == 0 && lh == 0) a.ex[at] = ex;
        unsigned char *o = reinterpret_cast<unsigned char *>(a.M) + at * (128 * a.rt) + t0 * 64 + 8 * lh;
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            if (t >= nt) break;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                h4 hi, lo;
#pragma unroll
                for (int z = 0; z < 4; ++z) {
                    float v = acc[t][4 * g + z] * up;
                    asm("" : "+v"(v));   // (see split8)
                    hi[z] = (_Float16)v;
                    lo[z] = (_Float16)(v - (float)hi[z]);
                }
                *reinterpret_cast<h4 *>(o + t * 64 + g * 16) = hi;
                *reinterpret_cast<h4 *>(o + t * 64 + g * 16 + 64 * a.rt) = lo;
            }
        }
    }
}

// Cells of several blocks: their moments become those of the first block, whose place the rows read.  One workgroup: such a cell
// and one row cell; each of its groups of 256 threads sums its share of the blocks.
__global__ __launch_bounds__(1024) void k_mom_reduce(unsigned char *M, float *ex, const int *several, const int *first_block, int nblock,
                                                     int RP)
{
    __shared__ float sh[4][256];
    const int k = several[blockIdx.x], groups = blockDim.x >> 8, g = threadIdx.x >> 8, al = threadIdx.x & 255;
    const int b0 = first_block[k], b1 = first_block[k + 1];
    const int per = (b1 - b0 + groups - 1) / groups;
    const int g0 = min(b1, b0 + g * per), g1 = min(b1, g0 + per);
    float *e = ex + (int64_t)blockIdx.y * nblock;
    float t = -INFINITY;
    bool nan = false;
    for (int b = b0; b < b1; ++b) {
        t = fmaxf(t, e[b]);
        nan |= e[b] != e[b];
    }
    t += (float)(32 - __clz(b1 - b0 - 1));   // (a sum of so many)
    float s = 0.0f;
    _Float16 *m = reinterpret_cast<_Float16 *>(M + (int64_t)blockIdx.y * nblock * RP * 4) + al;
    if (al < RP && t > -INFINITY) {
#pragma unroll 8
        for (int b = g0; b < g1; ++b) {
            const _Float16 *v = m + (int64_t)b * RP * 2;
            s = fmaf((float)v[0] + (float)v[RP], __builtin_amdgcn_exp2f(e[b] - t), s);
        }
    }
    sh[g][al] = s;
    __syncthreads();   // (also: the exponents are read)
    if (g == 0 && al < RP) {
        float v = sh[0][al];
        for (int q = 1; q < groups; ++q) v += sh[q][al];
        asm("" : "+v"(v));   // (see split8)
        const _Float16 hi = (_Float16)v;
        m[(int64_t)b0 * RP * 2] = hi;
        m[(int64_t)b0 * RP * 2 + RP] = (_Float16)(v - (float)hi);
        if (al == 0) e[b0] = nan ? NAN : t;
    }
}

// ---- the rows ----------------------------------------------------------------------------------------------------
struct RowArgs {
    const int4 *rows;                   // groups of rows (of the launch)
    const double4 *tcentre, *scentre;   // of the cells of both sides
    int first_cell;                     // of the launch
    int ncell;                          // streamed cells
    const float4 *xi;
    const int *perm;
    MomGeom tg;
    double cscale;
    float coef[kMaxTerms];              // c_alpha
    const int *first_block;             // where a streamed cell's moments are
    int nblock, cells, groups;          // blocks of the streamed side, row cells and groups of rows of the launch
    const float *ex;                    // as k_mom_gather leaves them
    const unsigned char *M;
    double2 *partial;
    float *opart;                       // applications: [rows][p]
    int p;
};
// One workgroup of eight waves: up to 256 rows of one cell, 32 per wave, against all streamed cells, 32 at a time.  Their moments
// (A operand) arrive in a ring of three tiles in LDS; the rows' monomials with their coefficients stay in registers in two pieces (B
// operand).  What comes out is, in lane j, sixteen cells' sums for row j, which get the factor 2^(...) that is left of the pair of
// cells and the row: right away in waves 0 to 3, after the next tile's barrier, before its products, in waves 4 to 7.
// A cell's 8 RT units of 16 bytes are rotated by a number of units that depends on its place in the tile, so that the reads of
// sixteen cells at one unit fall on different banks.
__device__ __forceinline__ int round_up_32(int v) { return (v + 31) & ~31; }
template <int RT> __device__ __forceinline__ int unit_rot(int c) { return (RT % 2 ? c >> 1 : c) & (RT == 1 ? 7 : 15); }
// power of coordinate k in a monomial of the basis
constexpr int row_power(uint32_t e, int k, int stride)
{
    const int at = (int)(e >> 8 * k & 255);
    return at == kOne ? 0 : at - k * stride;
}
template <int KIND>
__global__ __launch_bounds__(512, kKind[KIND].rt <= 2 ? 4 : 2) void k_mom_rows(RowArgs a)
{
    constexpr int RT = kKind[KIND].rt, DIM = kKind[KIND].d, TOP = kKind[KIND].p;
    constexpr int RP = 32 * RT, KS = 2 * RT, UN = 8 * RT;   // units of a cell
    constexpr int kTile = 32 * RP * 4;
    __shared__ __attribute__((aligned(1024))) unsigned char ring[3 * kTile];
    // of the streamed cells of a segment: what is left of the pair of cells, and where the moments are
    constexpr int kSeg = 1024;
    __shared__ float4 pair[kSeg];
    __shared__ int fb[kSeg];
    __shared__ __attribute__((aligned(16))) float cf[RP];
    __shared__ double wbest[8], wcol[8];
    __shared__ int warg[8], wnan[8];
    const int tid = threadIdx.x, l = tid & 63, lh = l >> 5, lj = l & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups are dealt to the eight XCDs in turn: an XCD takes neighbouring groups, which share their moments in its L2.
    const int per_xcd = (int)(gridDim.x + 7) / 8, gi = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (gi >= a.groups) return;
    const int4 grp = a.rows[gi];
    const int64_t at0 = (int64_t)(grp.x - a.first_cell) * a.nblock, at = at0 + (int64_t)blockIdx.z * a.cells * a.nblock;
    const unsigned char *M = a.M + at * (RP * 4);
    const float *ex0 = a.ex + at0, *ex = a.ex + at;
    const unsigned ring_off = (unsigned)(size_t)ring;
    // a tile's moments, 4 RT KB (cells beyond the last: a repeated one, which counts nothing)
    constexpr int NF = (RT + 1) / 2;
    int fc[NF], fo[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        const int u = (w * NF + i) * 64 + l, c = u / UN, p = u - c * UN - unit_rot<RT>(c) % UN;
        fc[i] = min(c, 31);   // (units beyond the tile are not fetched)
        fo[i] = (p < 0 ? p + UN : p) * 16;
    }
    // (k0: within the segment; no global load but the copies themselves, or a wait for it would be one for them)
    auto fetch = [&](int k0, int buf) __attribute__((always_inline)) {
        int b[NF];
#pragma unroll
        for (int i = 0; i < NF; ++i) b[i] = fb[k0 + fc[i]];
        __builtin_amdgcn_sched_barrier(0);   // (one wait for all of them)
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            if (RT % 2 && w * NF + i >= 4 * RT) break;
            dma16(M + (int64_t)b[i] * (RP * 4) + fo[i], ring_off + buf * kTile + (w * NF + i) * 1024);
        }
    };
    const double4 x0 = a.tcentre[grp.x];
    auto centre_dot = [&](const double4 &y) __attribute__((always_inline)) { return a.cscale * (x0.x * y.x + x0.y * y.y + x0.z * y.z); };

    if (tid < RP) cf[tid] = a.coef[tid];
    float4 row = 32 * w + lj < grp.z ? a.xi[grp.y + 32 * w + lj] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    // the streamed cell that counts most for this cell of rows: its size is the sums' scale, its centre their origin.  The sums of a
    // column of values have a scale of their own, that of their largest cell (col).
    double best = -INFINITY, col = -INFINITY;
    int arg = 0, nan = 0;
    for (int k = tid; k < a.ncell; k += 512) {
        const double cd = centre_dot(a.scentre[k]), t = cd + (double)ex0[a.first_block[k]];
        nan |= t != t;
        if (blockIdx.z) col = fmax(col, cd + (double)ex[a.first_block[k]]);
        if (t > best) {
            best = t;
            arg = k;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const double ob = __shfl_xor(best, off);
        const int oa = __shfl_xor(arg, off);
        nan |= __shfl_xor(nan, off);
        col = fmax(col, __shfl_xor(col, off));
        if (ob > best || (ob == best && oa < arg)) {
            best = ob;
            arg = oa;
        }
    }
    if (l == 0) {
        wbest[w] = best;
        warg[w] = arg;
        wnan[w] = nan;
        wcol[w] = col;
    }
    __syncthreads();
    nan = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        nan |= wnan[k];
        col = fmax(col, wcol[k]);
        if (wbest[k] > best || (wbest[k] == best && warg[k] < arg)) {
            best = wbest[k];
            arg = warg[k];
        }
    }
    const bool has_row = 32 * w + lj < grp.z && lh == 0;
    if (nan || !(best > -INFINITY)) {   // (uniform over the workgroup)
        if (has_row) {
            const int64_t i = a.perm[grp.y + 32 * w + lj];
            if (blockIdx.z)
                a.opart[i * a.p + blockIdx.z - 1] = nan ? NAN : 0.0f;
            else
                a.partial[i] = make_double2(nan ? 0.0 : (double)kNegInit, nan ? (double)NAN : 0.0);
        }
        return;
    }
    const double m = ceil(best), mc = blockIdx.z ? (col > -INFINITY ? ceil(col) : 0.0) : m;
    const double4 yr = a.scentre[arg];
    auto segment = [&](int s0) __attribute__((always_inline)) {
        for (int i = tid; i < min(kSeg, round_up_32(a.ncell - s0)); i += 512) {
            const int k = min(s0 + i, a.ncell - 1);   // (cells beyond the last: a repeated one, which counts nothing)
            const double4 y = a.scentre[k];
            const int b = a.first_block[k];
            fb[i] = b;
            pair[i] = make_float4((float)(y.x - yr.x), (float)(y.y - yr.y), (float)(y.z - yr.z),
                                  s0 + i < a.ncell ? (float)(centre_dot(y) + (double)ex[b] - mc) : -INFINITY);
        }
    };
    segment(0);
    asm volatile("" : "+v"(row.x), "+v"(row.y), "+v"(row.z));   // (here: a wait for it further down would be one for the copies)
    __syncthreads();
    // (nothing below waits for memory before the first tile is needed)
    fetch(0, 0);
    if (a.ncell > 32) fetch(32, 1);

    // The rows' monomials, eight neighbouring ones of a k-step's sixteen from either lane half, from powers in registers (out of
    // tables in LDS, 48 reads a k-step with an address each, and with the first tiles asked for after them, 256 groups over 125 cells
    // at RT = 7 took 21.5 us, 17.2 now).
    h8 psi[KS][2];
    const float sign = lj & 1 ? -1.0f : 1.0f;   // (see k_mom_gather: every other row sums over negated monomials)
    float pw[3][TOP + 1];
    {
        const float c[3] = {row.x, row.y, row.z};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            pw[k][0] = 1.0f;
#pragma unroll
            for (int e = 1; e <= TOP; ++e) pw[k][e] = k < DIM ? pw[k][e - 1] * c[k] : 1.0f;
        }
    }
    constexpr int st = pow_stride(DIM);
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        float v[8];
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
            const float4 c4 = *reinterpret_cast<const float4 *>(cf + 16 * k + 8 * lh + h);
            const float cc[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const uint32_t e0 = kBasisHost.e[KIND][16 * k + h + z], e1 = kBasisHost.e[KIND][16 * k + 8 + h + z];
                const float x0 = pw[0][row_power(e0, 0, st)], x1 = pw[0][row_power(e1, 0, st)];
                const float y0 = pw[1][row_power(e0, 1, st)] * pw[2][row_power(e0, 2, st)];
                const float y1 = pw[1][row_power(e1, 1, st)] * pw[2][row_power(e1, 2, st)];
                v[h + z] = sign * cc[z] * (lh ? x1 : x0) * (lh ? y1 : y0);
            }
        }
        split8(v, psi[k]);
        // (sixteen at a time: the reads of all of them in flight would take the registers)
        if (k & 1) asm volatile("" : "+v"(psi[k][0]), "+v"(psi[k][1]), "+v"(psi[k - 1][0]), "+v"(psi[k - 1][1])::"memory");
    }
    const double dx[3] = {(double)row.x * 0.5 * a.tg.h[0], DIM > 1 ? (double)row.y * 0.5 * a.tg.h[1] : 0.0,
                          DIM > 2 ? (double)row.z * 0.5 * a.tg.h[2] : 0.0};
    const float r0 = (float)(a.cscale * dx[0]), r1 = (float)(a.cscale * dx[1]), r2 = (float)(a.cscale * dx[2]);

    // (8 RT units per cell: leading pieces, then trailing ones)
    const int rot = unit_rot<RT>(lj) % UN;
    double sum = 0.0;
    const bool busy = 32 * w < grp.z, late = w >= 4;
    f16v acc;
    auto settle = [&](int k0) __attribute__((always_inline)) {
        constexpr int B = RT <= 2 ? 4 : 8;   // reads at a time (at RT <= 2 eight would take a CU's second workgroup: 27 -> 37 us at 1040 groups)
        float s = 0.0f;
#pragma unroll
        for (int h = 0; h < 16; h += B) {
            float4 e[B];
#pragma unroll
            for (int r = 0; r < B; ++r) e[r] = pair[k0 + 8 * ((h + r) >> 2) + 4 * lh + (r & 3)];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < B; ++r)
                s = fmaf(acc[h + r], __builtin_amdgcn_exp2f(fmaf(r0, e[r].x, fmaf(r1, e[r].y, fmaf(r2, e[r].z, e[r].w)))), s);
        }
        sum += (double)s;
    };
    for (int s0 = 0; s0 < a.ncell; s0 += kSeg) {
        const int n = min(kSeg, a.ncell - s0);
        if (s0) {
            __syncthreads();
            segment(s0);
            __syncthreads();
            fetch(0, 0);
            if (n > 32) fetch(32, 1);
        }
        int buf = 0;
        for (int k0 = 0; k0 < n; k0 += 32, buf = buf == 2 ? 0 : buf + 1) {
            // this tile has landed (the next one may be on its way), and its predecessor's place is read
            if (k0 + 32 < n)
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NF) : "memory");
            else
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (k0 + 64 < n) fetch(k0 + 64, buf == 0 ? 2 : buf - 1);
            if (!busy) continue;
            if (late && k0) settle(k0 - 32);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
            const unsigned char *src = ring + buf * kTile + lj * (RP * 4);
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                h8 v[2];
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    int u = 2 * k + lh + 4 * RT * z + rot;
                    u = u >= UN ? u - UN : u;
                    v[z] = *reinterpret_cast<const h8 *>(src + u * 16);
                }
                acc = mm2(v, psi[k], acc);
            }
            if (!late) settle(k0);
        }
        if (late && busy) settle((n - 1) / 32 * 32);
    }
    sum += __shfl_xor(sum, 32);
    sum *= (double)sign;
    if (has_row) {
        const double shift = a.cscale * (dx[0] * yr.x + dx[1] * yr.y + dx[2] * yr.z), fl = floor(shift);
        const int64_t i = a.perm[grp.y + 32 * w + lj];
        sum *= exp2(shift - fl);
        if (blockIdx.z)
            a.opart[i * a.p + blockIdx.z - 1] = (float)(sum * exp2(mc - m));   // (against the maximum that column 0 leaves)
        else
            a.partial[i] = make_double2(m + fl, sum);
    }
}

// coefficients of the truncated Chebyshev series of e^t on [-tau, tau], in powers of t
void series(double tau, int p, double *a)
{
    if (tau < 0.2) tau = 0.2;   // (the powers of a short interval cancel)
    double c[16], prev[16] = {}, cur[16] = {}, out[16] = {};
    for (int k = 0; k <= p; ++k) {   // 2 I_k(tau), I_0(tau)
        double term = 1.0;
        for (int j = 1; j <= k; ++j) term *= 0.5 * tau / j;
        double s = 0.0;
        for (int j = 0; j < 40; ++j) {
            s += term;
            term *= 0.25 * tau * tau / ((j + 1.0) * (j + 1.0 + k));
        }
        c[k] = k ? 2.0 * s : s;
    }
    // T_0, T_1, T_(k+1) = 2 z T_k - T_(k-1)
    prev[0] = 1.0;
    cur[1] = 1.0;
    for (int n = 0; n <= p; ++n) out[n] = c[0] * prev[n] + (p >= 1 ? c[1] * cur[n] : 0.0);
    for (int k = 2; k <= p; ++k) {
        double next[16] = {};
        for (int n = 0; n <= p; ++n) next[n] = (n ? 2.0 * cur[n - 1] : 0.0) - prev[n];
        for (int n = 0; n <= p; ++n) {
            prev[n] = cur[n];
            cur[n] = next[n];
            out[n] += c[k] * next[n];
        }
    }
    double q = 1.0;
    for (int n = 0; n <= p; ++n) {
        a[n] = out[n] / q;
        q *= tau;
    }
}

// cells of both clouds for one kind of expansion at eps; false where there would be too many of them, or where a tilt between
// cells leaves the range of a float's exponent
bool geometry(const MomState &S, int d, double eps, double tau, MomGeom (&g)[2], double (&s)[3])
{
    int active = 0;
    for (int k = 0; k < d; ++k) active += S.hi[0][k] > S.lo[0][k] && S.hi[1][k] > S.lo[1][k];
    const double h = active ? sqrt(2.0 * eps * tau / active) : 0.0;
    const double cs = 2.0 * kLog2e / eps;
    for (int side = 0; side < 2; ++side) {
        double cells = 1.0;
        for (int k = 0; k < 3; ++k) {
            double ext = k < d ? S.hi[side][k] - S.lo[side][k] : 0.0;
            const double mid = k < d ? 0.5 * (S.hi[side][k] + S.lo[side][k]) : 0.0;
            ext *= 1.0 + 1e-6;   // (points on the bounds fall inside, whatever the corner and the edges round to)
            const bool cut = k < d && S.hi[0][k] > S.lo[0][k] && S.hi[1][k] > S.lo[1][k];
            const double n = cut ? ceil(ext / h) : 1.0;
            cells *= n;
            if (!(cells <= kMomMaxCells)) return false;
            g[side].nc[k] = (int)n;
            g[side].h[k] = ext / n;
            g[side].lo[k] = mid - 0.5 * ext;
        }
    }
    for (int side = 0; side < 2; ++side) {   // rows on this side, the streamed points on the other
        double gather = 0.0, row = 0.0;
        for (int k = 0; k < d; ++k) {
            gather += cs * fmax(fabs(S.lo[side][k]), fabs(S.hi[side][k])) * 0.5 * g[1 - side].h[k];
            row += cs * (S.hi[1 - side][k] - S.lo[1 - side][k]) * 0.5 * g[side].h[k];
        }
        if (!(gather <= 48.0 && row <= 96.0)) return false;
    }
    for (int k = 0; k < 3; ++k) s[k] = g[0].h[k] * g[1].h[k] / (2.0 * eps);
    return true;
}

// Time of a pass (us).  nt, ct, gt: rows, their cells and groups; ns, cs, bs: streamed points, their cells and blocks; cols: 1 and the
// value columns of an application.  A launch takes as many row cells as the slab has place for, and its workgroups run in rounds of
// one per CU: k_mom_gather's take 2.1 us and 0.64 us per tile of monomials and stage of 32 points (half of that where `halves` is set),
// k_mom_rows' 3.6 us and 0.34 us per tile and 32 streamed cells, on top of what the chip's matrix cores and the moments' way
// through memory take.  Fitted to 887 passes (150 problems, d = 1..3, n m = 3e8 .. 3e10, cells from 1 to 7000, 33 us to 62 ms): half of the
// passes within 0.9 to 1.1 times, nine out of ten within 0.75 to 1.2 times what this says.  (The kernels take a tenth to a fifth less since;
// the line to the passes over the pairs was left where it is.)
double mom_cost(int rt, double nt, double ct, double gt, double ns, double cs, double bs, int cols, size_t slab, int num_cu)
{
    const double span = floor((double)slab / (cols * bs * (128.0 * rt + 4.0)) / 32.0) * 32.0;
    if (!(span >= 32.0)) return INFINITY;   // (moments of 32 row cells are the least that a launch forms)
    const double launches = ceil(ct / span), cells = ceil(ct / launches), tiles = ceil(cs / 32.0);
    const bool halves = cells <= 128.0;
    const double gather = ceil(cols * bs * ceil(cells / (halves ? 128.0 : 256.0)) / num_cu) * (2.1 + 0.64 * rt * (halves ? 0.5 : 1.0) * ceil(ns / bs / 32.0));
    const double rows = ceil(cols * gt / launches / num_cu) * (3.6 + 0.34 * rt * tiles);
    const double reduce = bs > cs ? 9.0 + 0.06 * bs / cs : 0.0;
    return 8.0 + launches * (gather + rows + reduce) + cols * (1.45e-4 * (nt / 32.0 + 0.5 * ct) * tiles + 5.4e-5 * ct * bs) * rt;
}
// streamed points of a block: longer ones, where there are workgroups enough for them (one per block and 32 cells of the other
// cloud), have fewer moments to write
int block_points(double cells, double other_cells, int64_t cnt, int num_cu)
{
    int block = 4 * kMomBlock;
    while (block > kMomBlock && ceil(other_cells / 32.0) * fmax(cells, (double)cnt / block) < 1.5 * num_cu) block /= 2;
    return block;
}
// The passes of a call at one eps: of P->mom.passes passes with rows on side t where there is only one, otherwise on either side in
// turn.  cells: those that hold points; blocks, groups: of either side, 0: not known yet.
double mom_cost_of(const Prepared *P, int t, int rt, const double (&cells)[2], const int (&blocks)[2], const int (&groups)[2], size_t slab,
                   int num_cu)
{
    const int64_t cnt[2] = {P->X.cnt, P->Y.cnt};
    double cost = 0.0;
    for (int side = 0; side < 2; ++side) {   // of the rows
        if (P->mom.passes == 1 && side != t) continue;
        const int o = 1 - side;
        const double g = groups[side] ? groups[side] : fmax(cells[side], 0.5 * cells[side] + (double)cnt[side] / kMomRows);
        const double b = blocks[o] ? blocks[o] : fmax(cells[o], 0.5 * cells[o] + (double)cnt[o] / block_points(cells[o], cells[side], cnt[o], num_cu));
        cost += mom_cost(rt, (double)cnt[side], cells[side], g, (double)cnt[o], cells[o], b, P->mom.cols, slab, num_cu);
    }
    return P->mom.passes == 1 ? cost : 0.5 * P->mom.passes * cost;
}

// bytes for the moments of a launch: at n = m = 262144 what a hundred row cells take, less where there are fewer blocks
size_t slab_bytes(int64_t n, int64_t m)
{
    const double mb = 256.0 * ((double)n / 262144.0) * ((double)m / 262144.0);
    return (size_t)(mb < 64.0 ? 64.0 : mb > 256.0 ? 256.0 : mb) << 20;
}
constexpr size_t kHostInts = 8 + 2 * (kMomMaxCells + 1);
struct Layout {
    size_t slab;
    size_t key[2], perm[2], xi[2], hist[2], total[2], cell[2], block[2], rows[2], centre[2], several[2], fb[2], fr[2], counts, M, bytes;
    int64_t chunk[2];
    int chunks[2], max_blocks[2], max_rows[2];
};
Layout lay(int64_t n, int64_t m)
{
    Layout L;
    Arena A;
    for (int s = 0; s < 2; ++s) {
        const int64_t cnt = s ? m : n;
        const int64_t cells = cnt < kMomMaxCells ? cnt : kMomMaxCells;
        // (at most 512 chunks; clouds have at most 2^24 points, chunks at most 2^15)
        L.chunk[s] = cnt > 256 * 1024 ? round_up(ceil_div(cnt, cnt > (1 << 22) ? 512 : 256), 256) : 1024;
        L.chunks[s] = (int)ceil_div(cnt, L.chunk[s]);
        L.max_blocks[s] = (int)(cells + ceil_div(cnt, kMomBlock));
        L.max_rows[s] = (int)(cells + ceil_div(cnt, kMomRows));
        L.key[s] = A.take((size_t)cnt * 2);
        L.perm[s] = A.take((size_t)cnt * 4);
        L.xi[s] = A.take((size_t)cnt * 16);
        L.hist[s] = A.take((size_t)L.chunks[s] * kMomMaxCells * 4);
        L.total[s] = A.take((size_t)kMomMaxCells * 4);
        L.cell[s] = A.take((size_t)kMomMaxCells * 16);
        L.block[s] = A.take((size_t)L.max_blocks[s] * 16);
        L.rows[s] = A.take((size_t)L.max_rows[s] * 16);
        L.centre[s] = A.take((size_t)kMomMaxCells * 32);
        L.several[s] = A.take((size_t)kMomMaxCells * 4);
        L.fb[s] = A.take((size_t)(kMomMaxCells + 1) * 4);
    }
    // what the host reads back, in one piece: counts of both sides (four each), the first group of rows of every cell
    L.counts = A.take(kHostInts * 4);
    for (int s = 0; s < 2; ++s) L.fr[s] = L.counts + (size_t)(8 + s * (kMomMaxCells + 1)) * 4;
    L.slab = slab_bytes(n, m);
    L.M = A.take(L.slab);
    L.bytes = A.off;
    return L;
}

MomSide side_of(const Layout &L, char *base, int s)
{
    MomSide o{};
    o.key = reinterpret_cast<uint16_t *>(base + L.key[s]);
    o.perm = reinterpret_cast<int *>(base + L.perm[s]);
    o.xi = reinterpret_cast<float4 *>(base + L.xi[s]);
    o.hist = reinterpret_cast<int *>(base + L.hist[s]);
    o.total = reinterpret_cast<int *>(base + L.total[s]);
    o.cell = reinterpret_cast<int4 *>(base + L.cell[s]);
    o.block = reinterpret_cast<int4 *>(base + L.block[s]);
    o.rows = reinterpret_cast<int4 *>(base + L.rows[s]);
    o.first_block = reinterpret_cast<int *>(base + L.fb[s]);
    o.first_rows = reinterpret_cast<int *>(base + L.fr[s]);
    o.several = reinterpret_cast<int *>(base + L.several[s]);
    o.centre = reinterpret_cast<double4 *>(base + L.centre[s]);
    o.counts = reinterpret_cast<int *>(base + L.counts) + 4 * s;
    return o;
}

#define FS_MOM_DISPATCH(rt, ...)                         \
    switch (rt) {                                          \
    case 1: { constexpr int RT_ = 1; __VA_ARGS__; } break;        \
    case 2: { constexpr int RT_ = 2; __VA_ARGS__; } break;        \
    case 4: { constexpr int RT_ = 4; __VA_ARGS__; } break;        \
    default: { constexpr int RT_ = 7; __VA_ARGS__; } break;       \
    }

}  // namespace

size_t mom_bytes(int64_t n, int64_t m) { return lay(n, m).bytes; }

// Decides whether the passes at `eps` (rows on side t) go through moments and, if so, deals the clouds to their cells.
fs_status mom_ready(Ctx *c, const Prepared *P, double eps, int t, bool *use)
{
    MomState &S = P->mom;
    *use = false;
    if (!S.base || c->dbg_lowd_moments == 2) return FS_OK;
    // (the other low-d switches ask for kernels over the pairs)
    if (c->dbg_lowd_moments == 0 && (c->dbg_lowd_score || c->dbg_lowd_splits || c->dbg_lowd_precise_valu)) return FS_OK;
    // Moments stand for passes over the pairs with fp32 scores.  Where float64-grade ones are asked for they are not accurate enough:
    // after 50 iterations at n = 3000, m = 2500 in the unit cube at eps = 0.005 f and g are off by 4e-7 eps and, over the pairs, by
    // 2e-7 and 7e-8 (d = 3), after 1000 at d = 1 by 3.5e-6 and 5e-8; the dual value (unit cube, d = 2 and 3, eps = 0.03 to 0.1, n m = 6e8 to
    // 5e9) is off by up to 2e-8 of itself and by 2e-9, marginal errors by up to 3e-8 and 6e-10.  (The switch that forces moments does so
    // for solves and gradients of any size, measurements are never taken through them.)
    if (P->force_precise || (c->dbg_lowd_moments == 0 && lowd_precise(P, eps))) return FS_OK;
    if (S.eps == eps) {
        *use = S.on;
        return FS_OK;
    }
    S.eps = eps;
    S.on = false;
    const int d = (int)P->d;
    bool finite = P->pot_mag_eps < INFINITY;
    for (int s = 0; s < 2; ++s)
        for (int k = 0; k < d; ++k) finite = finite && S.hi[s][k] >= S.lo[s][k] && S.hi[s][k] - S.lo[s][k] < 1e30;
    if (!finite) return FS_OK;
    const int64_t n = P->X.cnt, m = P->Y.cnt;
    const bool force = c->dbg_lowd_moments == 1;
    // What moments may take at most.  (The model of their time and that of the pairs are each off by up to a quarter.)
    const double limit = 0.85 * S.passes * mom_pair_cost(n, m, d, S.cols);
    const size_t slab = slab_bytes(n, m);
    const int unknown[2] = {0, 0};
    // The kind of expansion that is cheapest between the two cases that all cells hold points and half of many do.
    int best = -1;
    double half_cost = 0.0, all_cost = 0.0;
    MomGeom g[2];
    for (int k = 0; k < kKinds; ++k) {
        if (kKind[k].d != d || (c->dbg_moment_kind && c->dbg_moment_kind != 1 + k)) continue;
        MomGeom geo[2];
        double s[3], all[2], half[2];
        if (!geometry(S, d, eps, kKind[k].tau, geo, s)) continue;
        for (int q = 0; q < 2; ++q) {
            const double grid = (double)geo[q].nc[0] * geo[q].nc[1] * geo[q].nc[2], most = (double)(q ? m : n);
            all[q] = fmin(grid, most);
            half[q] = fmin(grid > 64.0 ? fmax(64.0, 0.5 * grid) : grid, most);
        }
        const double hc = mom_cost_of(P, t, kKind[k].rt, half, unknown, unknown, slab, c->num_cu);
        const double ac = mom_cost_of(P, t, kKind[k].rt, all, unknown, unknown, slab, c->num_cu);
        if (best < 0 || hc + ac < half_cost + all_cost) {
            best = k;
            half_cost = hc;
            all_cost = ac;
            g[0] = geo[0];
            g[1] = geo[1];
            for (int q = 0; q < 3; ++q) S.s[q] = s[q];
        }
    }
    if (best < 0) return FS_OK;
    // Dealing the points to their cells (four launches and a read-back) takes some time as well.  It is spent where moments pay even if
    // every cell holds points (as in a cube full of them), and where they do if half of them hold any and it is little beside the
    // passes: how many do is not known before.
    const double setup = 45.0 + 1.0e-4 * (double)(n + m);
    if (!force && setup + all_cost > limit && (setup + half_cost > limit || setup > 0.04 * limit)) return FS_OK;

    const Layout L = lay(n, m);
    if (L.bytes > S.bytes) return fail(c, FS_ERR_DEVICE, "internal: moment buffers");
    if (!S.host) S.host.reset(new (std::nothrow) int[kHostInts]);   // (no exception may leave an entry point)
    if (!S.host) return fail(c, FS_ERR_ALLOC, "host memory for the cells of the moment passes");
    SortSide a[2];
    int most_cells = 0;
    double many[2];   // (half of many cells hold points)
    for (int q = 0; q < 2; ++q) {
        many[q] = (double)g[q].nc[0] * g[q].nc[1] * g[q].nc[2];
        if (many[q] > 256.0) many[q] = fmax(256.0, 0.5 * many[q]);
    }
    for (int s = 0; s < 2; ++s) {
        const Side &sd = s ? P->Y : P->X;
        const int block = block_points(many[s], many[1 - s], sd.cnt, c->num_cu);
        a[s] = SortSide{sd.packed_d, sd.cnt, L.chunk[s], g[s].nc[0] * g[s].nc[1] * g[s].nc[2], L.chunks[s], block, g[s], side_of(L, S.base, s)};
        if (a[s].ncell > most_cells) most_cells = a[s].ncell;
    }
    const unsigned chunks = (unsigned)(L.chunks[0] > L.chunks[1] ? L.chunks[0] : L.chunks[1]);
    hipLaunchKernelGGL(k_mom_hist, dim3(chunks, 2), dim3(256), 0, c->stream, a[0], a[1], d, P->dpd);
    hipLaunchKernelGGL(k_mom_scan, dim3((unsigned)ceil_div(most_cells, 256), 2), dim3(256), 0, c->stream, a[0], a[1]);
    hipLaunchKernelGGL(k_mom_lists, dim3(1, 2), dim3(1024), 0, c->stream, a[0], a[1]);
    hipLaunchKernelGGL(k_mom_scatter, dim3(chunks, 2), dim3(256), 0, c->stream, a[0], a[1], d, P->dpd);
    FS_HIP(c, hipGetLastError());
    FS_HIP(c, hipMemcpyAsync(S.host.get(), S.base + L.counts, kHostInts * 4, hipMemcpyDeviceToHost, c->stream));
    FS_HIP(c, hipStreamSynchronize(c->stream));
    for (int s = 0; s < 2; ++s) {
        S.g[s] = g[s];
        S.side[s] = a[s].s;
        S.cells[s] = S.host[4 * s];
        S.blocks[s] = S.host[4 * s + 1];
        S.groups[s] = S.host[4 * s + 2];
        S.several[s] = S.host[4 * s + 3];
        if (S.cells[s] < 1 || S.cells[s] > a[s].ncell || S.blocks[s] < S.cells[s] || S.blocks[s] > L.max_blocks[s] ||
            S.groups[s] < S.cells[s] || S.groups[s] > L.max_rows[s] || S.several[s] < 0 ||
            S.several[s] > S.cells[s])
            return fail(c, FS_ERR_DEVICE, "internal: cells of the moment passes");
    }
    S.kind = best;
    double tau = 0.0;
    for (int k = 0; k < 3; ++k) tau += S.s[k];
    {
        double co[16];
        series(tau, kKind[best].p, co);
        for (int q = 0; q < kMaxTerms; ++q) {
            const uint32_t e = kBasisHost.e[best][q];
            const int st = pow_stride(d);
            double v = 0.0;
            if (e >> 24 != 255) {
                const int n = e >> 24, ex[3] = {(int)(e & 255), d > 1 ? (int)(e >> 8 & 255) - st : 0, d > 2 ? (int)(e >> 16 & 255) - 2 * st : 0};
                v = co[n];
                for (int k = 2; k <= n; ++k) v *= k;
                for (int k = 0; k < 3; ++k)
                    for (int z = 1; z <= ex[k]; ++z) v *= S.s[k] / z;
            }
            S.coef[q] = (float)ldexp(v, kCoefShift);
        }
    }
    const double cells[2] = {(double)S.cells[0], (double)S.cells[1]};
    const double cost = mom_cost_of(P, t, kKind[best].rt, cells, S.blocks, S.groups, L.slab, c->num_cu);
    if (!(cost < INFINITY)) return FS_OK;
    S.M = reinterpret_cast<unsigned char *>(S.base + L.M);
    S.slab = L.slab;
    S.on = force || cost < limit;
    *use = S.on;
    return FS_OK;
}

fs_status mom_pass(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, const float *V, int p, int64_t ldv, float *opart)
{
    const MomState &S = P->mom;
    const int t = res == &P->Y, s = 1 - t;
    const int rt = kKind[S.kind].rt, RP = 32 * rt;
    const unsigned cols = 1 + (V ? (unsigned)p : 0u);
    const MomSide &ts = S.side[t], &ss = S.side[s];
    int64_t span = (int64_t)(S.slab / ((size_t)cols * S.blocks[s] * (RP * 4 + 4))) / 32 * 32;
    if (span < 32 || cols > 1 + kMomMaxP) return fail(c, FS_ERR_DEVICE, "internal: moment slab");
    if (span > 65535 / cols / 32 * 32) span = 65535 / cols / 32 * 32;   // (grid of k_mom_reduce)
    if (span > S.cells[t]) span = S.cells[t];
    const int *first_rows = S.host.get() + 8 + t * (kMomMaxCells + 1);
    if (!V) prof_begin(c, 0.0, 2);   // (no pairs are evaluated)
    float *ex = reinterpret_cast<float *>(S.M + (size_t)cols * span * S.blocks[s] * RP * 4);   // (behind the moments)
    for (int64_t x0 = 0; x0 < S.cells[t]; x0 += span) {
        const int cells = (int)(S.cells[t] - x0 < span ? S.cells[t] - x0 : span);
        GatherArgs ga{};
        ga.block = ss.block;
        ga.centre = ts.centre + x0;
        ga.xi = ss.xi;
        ga.perm = ss.perm;
        ga.bias = str->packed_d + P->d;
        ga.bstride = P->dpd;
        ga.nblock = S.blocks[s];
        ga.ncells = cells;
        ga.sg = S.g[s];
        ga.cscale = 2.0 * kLog2e / eps;
        ga.d = (int)P->d;
        ga.kind = S.kind;
        ga.V = V;
        ga.ldv = ldv;
        ga.ex = ex;
        ga.M = S.M;
        // Workgroups: four tiles of cells at a time where there are no more; the monomials over two workgroups where there are
        // not enough of them for the chip.
        ga.rt = rt;
        ga.halves = cells <= 128;
        const int64_t ytiles = ceil_div(cells, ga.halves ? 128 : 256);
        ga.tsplit = (int64_t)S.blocks[s] * ytiles * cols < c->num_cu && rt > 1 ? 2 : 1;
        const int tw = (rt + ga.tsplit - 1) / ga.tsplit;
        const dim3 grid((unsigned)S.blocks[s], (unsigned)ytiles, cols * ga.tsplit);
        FS_MOM_DISPATCH(tw, hipLaunchKernelGGL(k_mom_gather<RT_>, grid, dim3(512), 0, c->stream, ga))
        if (S.several[s])
            hipLaunchKernelGGL(k_mom_reduce, dim3((unsigned)S.several[s], (unsigned)(cells * cols)),
                               dim3(S.blocks[s] - S.cells[s] > 16 * S.several[s] ? 1024 : 256), 0, c->stream, S.M, ex, ss.several,
                               ss.first_block, S.blocks[s], RP);
        RowArgs ra{};
        ra.rows = ts.rows + first_rows[x0];
        ra.tcentre = ts.centre;
        ra.scentre = ss.centre;
        ra.first_cell = (int)x0;
        ra.ncell = S.cells[s];
        ra.xi = ts.xi;
        ra.perm = ts.perm;
        ra.tg = S.g[t];
        ra.cscale = ga.cscale;
        for (int k = 0; k < kMaxTerms; ++k) ra.coef[k] = S.coef[k];
        ra.first_block = ss.first_block;
        ra.nblock = S.blocks[s];
        ra.cells = cells;
        ra.M = S.M;
        ra.ex = ex;
        ra.partial = (double2 *)P->partial;
        ra.opart = opart;
        ra.p = p;
        ra.groups = first_rows[x0 + cells] - first_rows[x0];
        const dim3 groups((unsigned)round_up(ra.groups, 8), 1, cols);
        c->moment_kind = 1 + S.kind;
        switch (S.kind) {
        case 0: hipLaunchKernelGGL(k_mom_rows<0>, groups, dim3(512), 0, c->stream, ra); break;
        case 1: hipLaunchKernelGGL(k_mom_rows<1>, groups, dim3(512), 0, c->stream, ra); break;
        case 2: hipLaunchKernelGGL(k_mom_rows<2>, groups, dim3(512), 0, c->stream, ra); break;
        case 3: hipLaunchKernelGGL(k_mom_rows<3>, groups, dim3(512), 0, c->stream, ra); break;
        case 4: hipLaunchKernelGGL(k_mom_rows<4>, groups, dim3(512), 0, c->stream, ra); break;
        case 5: hipLaunchKernelGGL(k_mom_rows<5>, groups, dim3(512), 0, c->stream, ra); break;
        default: hipLaunchKernelGGL(k_mom_rows<6>, groups, dim3(512), 0, c->stream, ra); break;
        }
        static_assert(kKinds == 7, "kinds of k_mom_rows");
    }
    if (!V) prof_end(c);
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

}  // namespace fs
