// Internal declarations shared by the translation units of libflashsink.
// Nothing here is part of the C ABI (see include/flashsink.h).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <memory>
#include <string>
#include <vector>

#include "flashsink.h"

namespace fs {

// ---------------------------------------------------------------------------------------
// constants
// ---------------------------------------------------------------------------------------
constexpr double kLog2e = 1.4426950408889634074;   // log2(e)
constexpr double kLn2 = 0.69314718055994530942;    // ln(2)
constexpr float kNegInit = -3.0e38f;               // finite "-inf" seed of the running max
constexpr int kLowdMaxD = 16;                      // d <= 16: fp32 vector-ALU path
// Most column splits of one streaming pass over `n_res` resident rows: as many as fill the chip
// even for a handful of rows (n << m), as long as the [splits][rows] partial records stay at 64 MB.
// (`budget`: bytes the records may take; the context's Ctx::partial_budget)
inline int max_splits(size_t budget, int64_t n_res)
{
    const int64_t pad = (n_res + 1023) / 1024 * 1024;
    const int64_t s = (int64_t)budget / (pad * 16);
    return s < 1 ? 1 : (s > 1024 ? 1024 : (int)s);
}

// Direct global -> LDS loads (no registers in between): lane l's 16 (4) bytes land at
// lds_off + 16 l (4 l); lds_off must be wave-uniform.  Issued as inline assembly so that the
// compiler does not serialise them against the LDS reads of OTHER ring slots; completion is
// tracked by hand with s_waitcnt vmcnt (VMEM operations retire in order).
__device__ inline void dma16(const void *g, unsigned lds_off)
{
    unsigned m = __builtin_amdgcn_readfirstlane(lds_off);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(m) : "memory", "m0");
}
__device__ inline void dma4(const void *g, unsigned lds_off)
{
    unsigned m = __builtin_amdgcn_readfirstlane(lds_off);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(g), "s"(m) : "memory", "m0");
}

// The same with a wave-uniform base address (it stays in scalar registers, and so does all the
// arithmetic that leads to it) and a per-lane byte offset.
__device__ inline void dma16s(const void *g_uniform, unsigned lane_off, unsigned lds_off)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(g_uniform), "s"(lds_off)
                 : "memory", "m0");
}
__device__ inline void dma4s(const void *g_uniform, unsigned lane_off, unsigned lds_off)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(lane_off), "s"(g_uniform), "s"(lds_off)
                 : "memory", "m0");
}

// Split records (fp32-grade scores on the bf16 matrix cores, d <= kLowdMaxD): 8 ks words of two bf16 slots.  A coordinate is the sum
// of three bf16 pieces p0, p1, p2 (split3), and the six products with a resident row's that count (streamed x resident, words of
// consecutive slots; p1 p2 and p2 p1 are below 2^-25 of a product),
//     (p0, p1) x (p1, p0)   (p1, p0) x (p1, p2)      words 2 k, 2 k + 1
//     (p2, .) x (p0, .)                              word 2 d + k / 2, two coordinates each
//     (p0, .) x (p0, .)                              word split_lead(ks, d) + k / 2
// come before the bias (three pieces and a one for the running max: the last two words, see split_bias_words).  In this order
// the sums are small until the last k-step or two, where the leading products meet the bias and what is left of both is small
// again: the matrix cores round (and where they align a product, truncate) at the size of the sum so far.  Errors against 64 bits
// (n = 3001, m = 2500; normal and cube, d = 1 .. 16) beside those of eight products a coordinate (p1 p2 and p2 p1 as well) in order with
// the bias behind them: half-steps and short solves 0.16 to 0.99 times, mostly 0.6 to 0.8 times, gradients, which keep exponentials
// to 2^-17, up to 1.05 times; with the bias before the products they were 1.0 to 2.6 times those.
// Measured (both half-steps of an averaged iteration, n = m = 20011, d = 10): 8 d + 6 slots 157 us, 6 d + 4 131.  Three fp16
// pieces, whose products carry more digits, took 140 us and a common scale of the coordinates; two of them 125 us, at 1.1 to 1.8 times
// the errors.
__host__ __device__ inline int split_pairs(int64_t d) { return (int)(d + 1) / 2; }
inline int split_ksteps(int64_t d) { return (int)(2 * d + 2 * split_pairs(d) + 2 + 7) / 8; }   // 1..7 for d = 1..16
__host__ __device__ inline int split_lead(int ks, int64_t d) { return 8 * ks - 2 - split_pairs(d); }
// The records of odd groups of 32 points are stored negated, so their scores come out of the matrix cores negated: the cores truncate
// towards minus infinity where they align a product, which pulls the scores of even groups down and of odd ones up.
__host__ __device__ inline bool split_negated(int64_t point) { return point >> 5 & 1; }
// Position (in 16-byte units) of piece `piece` of the record of point `point`: records lie in groups of 32 points, piece by
// piece, so that the lanes that read (from LDS or memory) or write one piece of consecutive points touch consecutive units.
// Point by point, a wave's LDS reads met in 2 (odd ks) to 16 (ks = 8) ways on a bank: six averaged iterations and the
// gradient at n = 15000, m = 14000, d = 14 (ks = 8) took 2147 us, 985 here; n = 12000, m = 20011, d = 5 (ks = 3) 778 and 656.
__host__ __device__ inline int64_t split_unit(int ks, int64_t point, int piece)
{
    return (point >> 5) * (64 * ks) + piece * 32 + (point & 31);
}
__device__ inline void split3(float v, __bf16 (&p)[3])
{
    p[0] = (__bf16)v;
    const bool fin = fabsf(v) < INFINITY;   // an infinite bias (padding) stays in the first piece
    float r = fin ? v - (float)p[0] : 0.0f;
    p[1] = (__bf16)r;
    r -= (float)p[1];
    p[2] = (__bf16)r;
}
__device__ inline void split3d(double v, __bf16 (&p)[3])   // three bf16 pieces of a finite double
{
    p[0] = (__bf16)(float)v;
    double r = v - (double)(float)p[0];
    p[1] = (__bf16)(float)r;
    r -= (double)(float)p[1];
    p[2] = (__bf16)(float)r;
}
// Grids of the leading digits of the "precise" split records (d <= 3, see k_lse_lowd_split):
// gy = 2^(Ey-7) with 2^Ey > max |y_k| (from rho_max, the largest squared norm after centring) and
// gx = 2^(Ex-7) with 2^Ex > (2 log2e/eps) max |x_k|; leading digits are multiples of the grid with
// at most 8 significant bits.
__host__ __device__ inline void split_grids(double rho_max, double eps, double *gx, double *gy)
{
    const double r = sqrt(rho_max > 1e-60 ? rho_max : 1e-60);
    *gy = exp2(floor(log2(r)) + 1.0 - 7.0);
    *gx = exp2(floor(log2(r * 2.0 * kLog2e / eps)) + 1.0 - 7.0);
}
__device__ inline uint32_t bf16_pair(__bf16 lo, __bf16 hi)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
}

enum class Path { LowD, F64, BF16 };

// Fixed-point scores (fs_fx.hip): k-steps of 32 coordinates, 0 where the path does not exist.  128 coordinates is what
// the resident digits of a wave may take in registers, and what keeps its integer sums inside 32 bits.
constexpr int kFxMaxKs = 4;
__host__ __device__ inline int fx_ksteps(int64_t d) { return d > kLowdMaxD && d <= 32 * kFxMaxKs ? (int)((d + 31) / 32) : 0; }

// Decides on the device which of the two kernels of a pass runs, fixed point or float64: the scale of the clouds is known there
// first.  Where it has reached the host's pinned box by the time of a launch (fx_known) only the kernel that runs is launched,
// otherwise both are, and one of them leaves at once: no call waits for it.  cscale r2^2 is the size of a score's unit-scale product in base-2
// units, v below; r2 covers the distance of the coordinates from the middle of their range, where k_prep_fx puts the origin.
//
// The upper line lies where the error of a score reaches the rounding of the exponential's float argument.  What counts there
// is that a coordinate below 2^-7 r2 loses bits of its float; at d = 128 (rms over pairs, in base-2 units) normal points have
// 2^-23.4 at v = 1846 and 2^-20.1 at v = 18466, unit-cube points 2^-26 at v = 288.  Plan sums of normal points at v = 1846 are
// off by 5.3e-8 of their size at d = 64 and 6.5e-8 at d = 128, where float64 scores leave 5.0e-8 and 3.7e-8 and the rounding of the
// output alone 3.4e-8; at v = 500 by 4.6e-8 where float64 scores leave 1.4e-7 to 2.2e-7; at v = 16000 it was 2.5e-7 to 7e-7.  Bounds for data whose
// digits conspire: the products left out at most 2 d 2^14 2^-54 v (2^-21 at the line, d = 128), the coordinates' rounding
// d 2^-31 v (one cloud within 2^-7 r2 of the origin and rounded one way, the other at the far end).
// Below v = 1/2 weights of 2^-60 no longer fit the bias records (every tile with one would take the slow epilogue), and
// the fp64 kernels take over.  A scale that is not finite is off as well.
//
// Up to kFxFull, ten products: those left out are 2^-24.3 rms at that line for random digits and d = 128, and for two-valued
// coordinates; d 2^-30.4 v at most (2^-18.4, every digit at its largest and of one sign).  At four times the line, two-valued
// coordinates already cost plan sums a digit against the fp64 kernels.
constexpr double kFxLow = 0.5, kFxHigh = 2048.0, kFxFull = 32.0;
struct FxGate {
    const double *r2 = nullptr;   // common scale of both clouds (device), see k_prep_fx; nullptr: no digit images
    double cscale = 0.0;          // 2 log2(e) / eps
    __device__ bool on() const
    {
        const double r = *r2, v = cscale * r * r;
        return v >= kFxLow && v <= kFxHigh;
    }
    // all thirteen digit products (see fs_fx.hip)
    __device__ bool full() const
    {
        const double r = *r2;
        return cscale * r * r > kFxFull;
    }
    __device__ double unit(int k) const { return ldexp(cscale * *r2 * *r2, -k); }
    __device__ double per_unit(int k) const { return ldexp(1.0 / (cscale * *r2 * *r2), k); }
};

// the four balanced base-256 digits of sixteen coordinates in fixed point
__device__ inline void fx_digits16(const int *v, uint4 (&out)[4])
{
    uint32_t o[4][4];
#pragma unroll
    for (int z = 0; z < 16; ++z) {
        int X = v[z];
#pragma unroll
        for (int dg = 3; dg >= 0; --dg) {
            const int t = dg > 0 ? (int)(signed char)(X & 255) : X;   // balanced: what is left is a multiple of 256
            o[dg][z >> 2] = (z & 3) ? o[dg][z >> 2] | ((uint32_t)(t & 255) << (8 * (z & 3))) : (uint32_t)(t & 255);
            X = (X - t) >> 8;
        }
    }
#pragma unroll
    for (int dg = 0; dg < 4; ++dg) out[dg] = make_uint4(o[dg][0], o[dg][1], o[dg][2], o[dg][3]);
}

// Splits of the streamed side that a pass wrote, as the merges need them: n of the main kernel, and, where the gate
// chooses between two kernels, alt of the float64 one (0: only one kernel was launched)
struct Splits {
    int n, alt;
    Splits(int n_ = 1, int alt_ = 0) : n(n_), alt(alt_) {}
};

// ---------------------------------------------------------------------------------------
// context
// ---------------------------------------------------------------------------------------
struct Ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    int num_cu = 256;
    // grow-only device workspace
    char *ws = nullptr;
    size_t ws_bytes = 0;
    bool ws_static = false;          // ws is the library's static scratch array for the duration of a call: never freed or grown
    char *static_ws = nullptr;       // this device's address of the static scratch array (resolved in fs_create)
    size_t partial_budget = size_t(64) << 20;   // bytes the [splits][rows] partial records of a pass may take
    // grow-only second buffer for entry points that call other entry points (which lay the workspace out anew)
    char *aux = nullptr;
    size_t aux_bytes = 0;
    // numbers that a kernel hands to the host (pinned), and when they are there: the conjugate gradients' (made when first used)
    double *pin = nullptr;
    hipEvent_t pin_ready = nullptr;
    // Scalars that decide what the host launches next, written there by the kernels that have them (pinned; every word carries the
    // stamp of its call in the upper half, so no order of the writes is asked for; nullptr: copies instead).  Made by the first call
    // that uses it (in fs_create it took 10 to 35 us of every context, and as much of its fs_destroy, also where only bf16 problems
    // follow); calls in the static scratch array, which may not allocate, have this device's one that lives as long as that array.
    unsigned long long *box = nullptr;
    unsigned long long *static_box = nullptr;
    std::string err;
    // Derived copies kept across entry calls (fs_points_keep): what identifies the clouds the caller has declared
    // unchanged, whether the workspace currently holds their derived copies, and the host-side value that belongs
    // to them (largest squared norm after centring, low-d path)
    struct PointsKey {
        const void *x = nullptr, *y = nullptr;
        int dtype = 0, compute = 0;
        int64_t n = 0, m = 0, d = 0, ldx = 0, ldy = 0;
        const char *ws = nullptr;      // the workspace the copies live in
        size_t partial_budget = 0;     // (the offsets of the device scalars depend on it)
        bool same(const PointsKey &o) const
        {
            return x == o.x && y == o.y && dtype == o.dtype && compute == o.compute && n == o.n && m == o.m && d == o.d &&
                   ldx == o.ldx && ldy == o.ldy && ws == o.ws && partial_budget == o.partial_budget;
        }
    };
    bool keep_on = false;
    PointsKey keep_key;                // declared by the caller (ws and partial_budget unset)
    bool kept_valid = false;
    bool kept_bounds = false;   // ... and whether the bounds that the cell moments need are there as well
    size_t mom_denied = SIZE_MAX;   // bytes of moment buffers that there was no memory for
    size_t seeds_denied = SIZE_MAX; // ... of a workspace with FxSeed buffers
    PointsKey kept_key;
    double kept_rho_max = -1.0;
    uint32_t kept_fx_stamp = 0;
    // test and experiment switches of this context (fs_debug_set); 0 = the library decides
    int dbg_lowd_splits = 0;         // forced split count of the streamed side of a low-d pass
    int dbg_lowd_score = 0;          // 32: fp32 scores, 64: float64 scores in every low-d half-step
    int dbg_lowd_precise_valu = 0;   // 1: float64 scores at d <= 3 on the vector ALU instead of the precise records
    int dbg_lowd_any_bias = 0;       // 1: the precise records also for biases beyond their digit range (tests of that case)
    int dbg_lowd_moments = 0;        // d <= 3: 1: half-steps through cell moments wherever they can be, 2: never
    int dbg_fx_any_size = 0;         // 1: digit images for problems of any size
    size_t dbg_ws_limit = 0;         // the workspace does not get more bytes than this (0: no limit)
    int dbg_fx_splits = 0;           // forced split count of the streamed side of a fixed-point pass
    int dbg_fx_long = 0;             // 1: fixed-point half-steps of any length as long ones (MODE 3 or 4), 2: none
    unsigned long long *fx_count = nullptr;   // device: tiles that long half-steps have left at their leading products, and all of theirs
    int dbg_moment_kind = 0;         // 1 + the expansion that passes through cell moments take
    int moment_kind = 0;             // 1 + the one that the last such pass took
    // profiling of the streaming LSE launches
    bool prof_on = false;
    std::vector<hipEvent_t> ev_pool;   // pairs (start, stop)
    size_t ev_used = 0;
    std::vector<int> ev_kind;          // per recorded launch: which kernel it was (0 = the path's main
                                       // kernel, 1 = the low-d float64-score kernel, 2 = a pass through cell moments)
    std::vector<double> ev_pairs;      // per recorded launch: pair evaluations
};

fs_status fail(Ctx *c, fs_status s, const char *fmt, ...);

#define FS_HIP(ctx, expr)                                                                     \
    do {                                                                                      \
        hipError_t e__ = (expr);                                                              \
        if (e__ != hipSuccess)                                                                \
            return fs::fail((ctx), FS_ERR_DEVICE, "%s failed: %s", #expr, hipGetErrorString(e__)); \
    } while (0)

// Linear sub-allocator over the workspace (256-byte aligned pieces).
struct Arena {
    size_t off = 0;
    size_t take(size_t bytes)
    {
        size_t o = off;
        off += (bytes + 255) & ~size_t(255);
        return o;
    }
};

inline int64_t round_up(int64_t v, int64_t q) { return (v + q - 1) / q * q; }
inline int64_t ceil_div(int64_t v, int64_t q) { return (v + q - 1) / q; }

// ---------------------------------------------------------------------------------------
// One side (x or y) of a prepared problem: the derived copy the kernels read, its squared
// norms, the shifted potential and the bias it contributes when it is the streamed side.
// ---------------------------------------------------------------------------------------
struct Side {
    int64_t cnt = 0;       // real points
    int64_t cnt_pad = 0;   // rows of the derived copy (padding rows: zero coordinates, bias -inf)
    const float *w = nullptr;   // weights (device) or nullptr = uniform
    double log_uniform = 0.0;   // log(1/cnt)
    // LowD: packed [cnt_pad][dp] floats, dp = round_up(d+1, 4), and [cnt_pad][dpd] doubles,
    // dpd = round_up(d+1, 2); slot d of each point holds its bias
    float *packed = nullptr;
    double *packed_d = nullptr;
    double *norm_f = nullptr;  // [cnt_pad] squared norms of the float-rounded centred points
    // LowD: the packed floats again as [cnt_pad][16 ks] bf16 "split" records for the
    // matrix cores (layout: see split_ksteps)
    uint16_t *split = nullptr;
    // LowD, d <= 3: "precise" split records [cnt_pad][48] bf16 built from the float64 copy
    uint16_t *split_p = nullptr;
    // F64: double [cnt_pad][kp], kp = round_up(d, 32) (zero filled), bias in bias_d[cnt_pad].
    // LowD with d > 3 keeps the same two arrays (centred coordinates, kp = 32) for its float64-score
    // passes, which run on the fp64 matrix-core kernels.
    double *pts_d = nullptr;
    double *bias_d = nullptr;
    // BF16: uint16 [cnt_pad][kp], kp = round_up(d, 32), bias in bias_f[cnt_pad]
    uint16_t *pts_b = nullptr;
    float *bias_f = nullptr;
    // F64 with digit images (16 < d <= 128): [cnt_pad / 32][fx_ks][4][1024] bytes, and the bias records
    // [cnt_pad / 32][128] ints (see store_fx_record)
    unsigned char *dig = nullptr;
    int *brec = nullptr;
    double *norm = nullptr;   // [cnt_pad] squared norms of the derived points
    double *pot = nullptr;    // [cnt_pad] UNSHIFTED potential (f or g) in float64
};

// Half-steps through cell moments (fs_moments.hip, d <= 3).  A grid of cells over one cloud: corner, edges, cells per coordinate.
constexpr int kMomMaxCells = 8192;   // per cloud
constexpr int kMomBlock = 256;       // streamed points a workgroup takes at a time; a block of a cell is one to four times that
constexpr int kMomTerms = 224;       // monomials at most
constexpr int kMomRows = 256;        // rows per workgroup
struct MomGeom {
    double lo[3], h[3];
    int nc[3];
};
// one cloud dealt to its cells (device)
struct MomSide {
    uint16_t *key;          // [cnt] cell of a point
    int *perm;              // [cnt] point at a place of the sorted order
    float4 *xi;             // [cnt] sorted: coordinates in half cells
    int *hist, *total;      // of the sort
    int4 *cell;             // cells that hold points: (cell, first place, points, -)
    int4 *block, *rows;     // blocks and groups of rows: (number of their cell among those, first place, points, -)
    double4 *centre;        // [cells]
    int *several;           // cells of several blocks
    int *first_block, *first_rows;   // [cells + 1]
    int *counts;
};
// What the passes of one entry call share: the grids belong to one eps and are laid out when it is first met.
struct MomState {
    char *base = nullptr;   // nullptr: no buffers
    size_t bytes = 0;
    // Set by the entry points whose passes may take them (half-steps of the alternating schedule, gradients), for which alone buffers
    // and bounds are made: how many passes the call makes at one eps, and their columns (1, and the values' of an application).  An
    // application may where its values are points of a cloud, which the bounds say are finite (an infinite value would reach whole
    // cells as NaN).
    int passes = 0, cols = 1;
    double lo[2][3], hi[2][3];   // bounds of both centred clouds (host)
    double eps = 0.0;
    bool on = false;        // ... whether half-steps at that eps run through moments
    int kind = 0;
    MomGeom g[2];
    MomSide side[2];
    int cells[2], blocks[2], groups[2], several[2];
    size_t slab = 0;        // bytes of M
    float coef[kMomTerms];
    double s[3];
    unsigned char *M = nullptr;
    std::unique_ptr<int[]> host;   // what the host has read back of the cells (see Layout::counts in fs_moments.hip)
};

// Launch-shape decision of one streaming pass.
struct PassShape {
    int rows_per_block = 0;
    int row_blocks = 0;
    int splits = 1;
    int64_t cols_per_split = 0;   // multiple of the column tile
    double cost = 0.0;            // fixed-point passes: what the model of fx_shape expects
};

constexpr int kScalars = 32, kScalarBounds = 16;   // Prepared::scalars
struct Prepared {
    Path path = Path::LowD;
    int64_t d = 0;
    int dp = 0;   // LowD: floats per packed point
    int dpd = 0;  // LowD: doubles per packed point (float64 score mode)
    int ks = 0;   // LowD: 16-wide contraction steps of a split record
    double rho_max = 0.0;   // LowD: largest squared norm of a centred point (host copy)
    // LowD: size of the biases that the caller's potentials give, in base-2 units:
    //   |bias| <= pot_mag_eps / eps + logw_mag   (potential part, scaling like 1/eps, and log-weight part)
    double pot_mag_eps = 0.0, logw_mag = 0.0;
    int halfsteps_per_eps = 2;    // LowD: half-steps the caller runs at one eps (error budget)
    bool force_precise = false;   // LowD: float64 scores regardless (marginal error evaluation)
    int dbg_score = 0;            // LowD: the context's score switch (see Ctx::dbg_lowd_score)
    bool dbg_precise_valu = false;   // LowD: the context's kernel switch (see Ctx::dbg_lowd_precise_valu)
    bool dbg_any_bias = false;       // LowD: see Ctx::dbg_lowd_any_bias
    mutable MomState mom;            // LowD, d <= 3
    int kp = 0;   // F64 / BF16: padded contraction length
    int fx_ks = 0;   // F64: k-steps of the digit images, 0: none
    unsigned long long *box = nullptr;   // where kernels of this call write for the host (Ctx::box or Ctx::static_box), or nullptr
    uint32_t fx_stamp = 0;           // the stamp under which r2 comes to the host (see fx_known), 0: it does not
    // fixed-point passes: what the last pass over the rows of X [0] and Y [1] left about them (FxSeed), two buffers a side in turn
    struct Seeds {
        char *buf[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};
        int last[2] = {-1, -1};   // which of the two holds the last pass's, -1: neither
        int splits[2] = {0, 0};   // ... and its splits
        size_t bytes[2] = {0, 0};
    };
    bool want_seeds = false;      // set by the entry points that pass over the same rows several times
    bool pairs = false;           // ... two passes a launch (fs_solve_symmetric)
    mutable Seeds seeds;
    mutable PassShape fx_shapes[2][3];   // of half-steps over the rows of X [0] and Y [1] in MODE 0, 3 and 4, once asked for
    Side X, Y;
    // partial reductions of a streaming pass: [splits][max(n,m)_pad] records
    void *partial = nullptr;
    size_t partial_bytes = 0;
    double *dev_part = nullptr;  // [ceil(max(n,m)/256)] per-block sums of the marginal deviation
    double *gauge_part = nullptr;   // [2][ceil(max(n,m)/256)] per-block sums of the plan's mass seen by a g-update
    double *gauge_part_x = nullptr; // the same for an f-update (averaged schedule: both passes measure, halves by parity)
    double *scalars = nullptr;   // [kScalars] device doubles (marginal errors, centring sums...; [8], [9]: gauge drift, see GaugeMode; [10], [11]: FxGate::r2 and the origin of the digits; from kScalarBounds on: bounds of the centred clouds, see k_mean_final)
    double *mean = nullptr;      // [kLowdMaxD] common mean (LowD)
    char *extra = nullptr;       // entry-point specific scratch (plan application partials)
    size_t extra_bytes = 0;
};

// For each row of a pass of the fixed-point kernels and each split of the streamed side, a point whose score was within a few base-2
// units of the split's largest: point, or -1 where there is none, and the leading part of <x_i, y_point> in units of r2^2 2^-22.  The next
// pass over the same rows starts from the score of that point at its own biases (see fs_fx.hip).
struct FxSeed {
    int dot, point;
};

// Prepared::box: one word for the exponent of r2, two for each scalar of the low-d prologue (see launch_bias_from_user)
constexpr int kBoxFx = 0, kBoxLowd = 8, kBoxWords = 64;
constexpr int kFxNoScale = 0x4000;   // instead of the exponent: the scale is not finite

// whether the context's stream records a graph (or may not be asked: the default stream while another one records)
inline bool capturing(const Ctx *c)
{
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &s) == hipSuccess) return s != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// the gate of a pass at `eps` (r2 sits in scalars[10])
inline FxGate fx_gate(const Prepared *P, double eps)
{
    FxGate g;
    g.r2 = P->fx_ks ? P->scalars + 10 : nullptr;
    g.cscale = 2.0 * kLog2e * (1.0 / eps);   // (as store_fx_record forms it)
    return g;
}

// Which of the two kernels of a pass runs, as far as the host knows: 1 the fixed-point one, 0 the other, -1 not known yet, launch both.
// The scale arrives while the first passes of a call run; nothing waits for it.
inline int fx_known(const Prepared *P, double eps)
{
    if (!P->box || !P->fx_ks || !P->fx_stamp) return -1;
    const unsigned long long w = __atomic_load_n(P->box + kBoxFx, __ATOMIC_RELAXED);
    if ((uint32_t)(w >> 32) != P->fx_stamp) return -1;
    const int ex = (int)(int16_t)(w & 0xffff);
    if (ex == kFxNoScale) return 0;
    const double r = ldexp(1.0, ex), v = 2.0 * kLog2e * (1.0 / eps) * r * r;   // (as FxGate::on has it)
    return v >= kFxLow && v <= kFxHigh;
}

// Where the bias of point i of a side lives, by path, and the squared norms that turn the
// unshifted potential into the shifted one of Prop. 1 (fhat = f - alpha, ghat = g - beta).
struct BiasSink {
    float *packed;          // LowD float copy: packed[i*dp + d], shifted by norm_f
    uint16_t *split;        // LowD split records (same value as the float copy), ks > 0
    int ks;
    uint16_t *split_p;      // LowD precise split records (d <= 3) and the grid of their bias digits:
    double q;               // q itself, or (q == 0) the device scalar rho_max and the eps it is derived from
    const double *rho_dev;
    double q_eps;
    double *packed_d;       // LowD double copy: packed_d[i*dpd + d], shifted by norm
    int dp, dpd, d;
    float *bias_f;          // BF16 path
    double *bias_d;         // F64 path
    int *brec;              // F64 path: bias records of the fixed-point kernels and the scale r2 they refer to
    const double *r2;
    const double *norm_f;
    const double *norm;
};

// ---- merge the per-split (max, sum) statistics of a streaming pass -----------------------
//   LSE_2 = M + log2(sum_k s_k 2^(m_k - M)),  pot_new = -eps * ln2 * LSE_2      (Alg. 1, last lines)
// and, as asked: store pot_new, the bias for the pass that streams this side next, the
// unshifted potential for the caller, or the marginal deviation |w e^((pot_old-pot_new)/eps) - w|.
struct FinalizeArgs {
    const double2 *partial;
    int64_t stride;
    int splits, splits_alt;   // (splits_alt: where the gate chose the float64 kernel)
    FxGate gate;
    int64_t cnt;
    double eps, inv_eps_next;
    const float *w;
    double log_uniform;
    const double *res_norm;
    double *pot;
    BiasSink sink;
    float *user_out;
    double *dev_part;
    double mix;
    double *save_old;
    int blocks;   // workgroups of this side
    // gauge drift (see GaugeMode): where a g-update leaves the block sums of the plan's column marginals, and what
    // a workgroup of the following f-update collects
    double *gauge_out;
    const double *gauge_prev;
    int64_t gauge_prev_cnt;
    double gauge_prev_eps;
    double *gauge_scalars;   // [0]: the sum so far, [1]: the sum without its last term
    const double *gauge_prev_x;   // averaged schedule: the f-pass's block sums of the previous iteration
    int64_t gauge_prev_x_cnt;
};

// ---------------------------------------------------------------------------------------
// kernel launchers (implemented in the path-specific translation units)
// ---------------------------------------------------------------------------------------

// fs_prep.hip
fs_status launch_prepare(Ctx *c, const fs_problem *p, Prepared *P);
// cnt doubles (at most kMostReadBack) of the device to the host, once everything before on the stream has run
constexpr int kMostReadBack = 28;
fs_status read_back(Ctx *c, const double *src, int cnt, double *dst);
// `first` / `last`: an entry point that brings in both potentials passes (true, false) and then
// (false, true); the low-d read-back of the sizes that choose the score arithmetic (largest squared
// norm, size of the biases) happens once, in the call with last = true.
fs_status launch_bias_from_user(Ctx *c, Prepared *P, Side *side, const float *pot_user, double eps, bool first = true,
                                bool last = true);
// `res_norm` is the norm array matching the coordinates the pass used (Side::norm or norm_f).
// `mix`: the new potential is (1 - mix) * old + mix * update (1: plain update, 1/2: averaged schedule).
// `abs_dev_sum` != nullptr measures the marginal deviation instead of storing the update; with
// `save_old` it does both and leaves the replaced potential in save_old[0..cnt).
// Drift of the alternating iteration along its neutral direction (f + t, g - t), and how it is taken out.
// The exact iterates keep the plan's total mass at 1: after "f from g" the row marginals are exact.  A g-update
// measures that mass on its way (Prop. 3: c_j = b_j exp((g_j - g_j^+)/eps) are the column sums of the plan that
// (f, g) induce).  When the f-pass and the g-pass carry different systematic rounding biases u_f, u_g (the matrix
// cores truncate when they align the products of a score), the computed mass is exp((u_f - u_g)/eps), and the
// difference is exactly what one iteration adds to t: a random error would be damped, this one accumulates linearly
// (measured on the annealed low-dimension workload: 8e-5 eps at n = 16384, 2.5e-4 eps at n = 32768 after 200
// iterations, with a scatter around that constant of 8e-6).  So a solve adds up eps ln(mass) over its g-updates
// (scalars[8]; scalars[9] keeps the sum without the last term) and hands f - scalars[9], g + scalars[8] to the caller.
//   Measure: this merge is a g-update of an alternating solve: leave the block sums of c_j in gauge_part
//   Collect: this merge is the f-update after one: one of its workgroups adds eps_prev ln(sum gauge_part) to scalars[8]
//            (gauge_prev_cnt: how many sums that g-update left)
enum class GaugeMode { None, Measure, Collect };
fs_status launch_finalize(Ctx *c, const Prepared *P, Side *res, const double *res_norm, Splits splits,
                          double eps_cur, double eps_next_bias, float *user_out, double *abs_dev_sum,
                          double mix = 1.0, double *save_old = nullptr, GaugeMode gauge = GaugeMode::None,
                          int64_t gauge_prev_cnt = 0, double gauge_prev_eps = 0.0);
// the same merge's arguments, for a half-step kernel that merges on its own
FinalizeArgs make_finalize_args(const Prepared *P, Side *res, const double *res_norm, double eps_cur, double eps_next_bias,
                                float *user_out, GaugeMode gauge, int64_t gauge_prev_cnt, double gauge_prev_eps);
// the last g-update's term, then f_user = (float)(X.pot - scalars[9]) and g_user = (float)(Y.pot + scalars[8])
// (x_pot: the f to hand out, X.pot or a saved copy of it)
// (collect_last: how many sums the last g-update left in gauge_part, 0: nothing to collect)
fs_status launch_gauge_export(Ctx *c, const Prepared *P, int64_t collect_last, double eps_last, const double *x_pot,
                              float *f_user, float *g_user);
// `gauge`: the averaged schedule's form of the drift removal (see GaugeMode): both passes of an iteration read the
// same old potentials, so the plan's mass as the f-pass sees it (row sums) and as the g-pass sees it (column sums)
// differ by exp((u_f - u_g)/eps) exactly, and an averaged iteration moves t by a quarter of u_f - u_g.  With
// gauge_parity >= 0 (the iteration number) both merges leave their block sums in half `gauge_parity & 1` of
// gauge_part_x / gauge_part, and, `collect_prev`, one workgroup adds the previous iteration's term
// eps (ln mass_g - ln mass_f) / 4 to scalars[8] and [9] from the other half; the caller hands out f - scalars[9],
// g + scalars[8] (launch_gauge_collect_pair for the last iteration, then launch_gauge_export with collect_last = false).
fs_status launch_finalize_pair(Ctx *c, const Prepared *P, Side *X, const double *norm_x, const void *partial_x, Splits splits_x,
                               float *f_out, Side *Y, const double *norm_y, const void *partial_y, Splits splits_y,
                               float *g_out, double eps_cur, double eps_next_bias, double mix, int gauge_parity = -1,
                               bool collect_prev = false);
fs_status launch_gauge_collect_pair(Ctx *c, const Prepared *P, double eps, int gauge_parity);
fs_status launch_export_f32(Ctx *c, const double *src, int64_t cnt, float *dst);
// label-augmented cost: augmented copy [rows][d + V] of one cloud (see k_label_augment) and the map between the
// potentials of the labelled and of the augmented problem
fs_status launch_label_augment(Ctx *c, const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld,
                               const int32_t *labels, const float *W, int V, bool target_side, double l1, double l2,
                               bool round_bf16, float *out, float *vconst, unsigned *bad);
fs_status launch_label_potential(Ctx *c, const float *src, const float *vconst, double cshift, double l1, bool to_augmented,
                                 int64_t cnt, float *dst);
fs_status launch_pts_to_f32(Ctx *c, const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld, float *dst);
fs_status launch_grad_assemble(Ctx *c, float *g, int64_t ldg, const void *pts, int dtype, int64_t ld, int64_t rows,
                               int64_t d, const float *w, const float *mass, int mode);
fs_status launch_value_terms(Ctx *c, const Prepared *P, const Side *res, const double *res_norm, const Side *str,
                             Splits splits, double eps, double *scratch, double *dst);
fs_status launch_row_norms(Ctx *c, const void *pts, int dtype, int64_t rows, int64_t d, int64_t ld,
                           float *out);
fs_status launch_fill_f64(Ctx *c, double *dst, double v, int64_t cnt);
fs_status launch_weight_stats(Ctx *c, const float *w, int64_t cnt, double *scratch, double *dst);
fs_status launch_count_nonfinite(Ctx *c, const float *v, int64_t cnt, double *scratch, double *dst);
// merge the splits of an application pass (partial (max,sum) + opart[split][row][PC]) and apply
// the epilogue  out_i = w_i exp(pot_shifted_i/eps + m_i) O_i  for columns p0 .. p0+PC-1 (PC_alt: row length of the
// accumulators where the gate chose the other kernel)
fs_status launch_apply_finalize(Ctx *c, const Prepared *P, const Side *res, const double *res_norm, Splits splits,
                                double eps, const float *opart, int PC, int p0, int p, float *out, int64_t ldo,
                                float *mass_out, int PC_alt = 0);

// fs_hvp.hip
size_t hvp_scratch_bytes(int64_t n, int64_t m, int64_t d);
fs_status hvp_run(Ctx *c, Prepared *P, const float *x, int64_t ldx, const float *y, int64_t ldy, double eps,
                  const float *A, int64_t lda, double tau, double eta, int max_cg, float *out, int64_t ldo,
                  char *scratch, int *cg_iters);

// out (n x p, ldo) += <A_i, mean> PV_i (PV: n x p, dense): the mean's share of the Hadamard weights
fs_status launch_add_mean_share(Ctx *c, const float *A, int64_t lda, const double *mean, const float *PV, int64_t n, int d,
                                int p, float *out, int64_t ldo);

// fs_lowd.hip
PassShape lowd_shape(const Ctx *c, int64_t n_res, int64_t n_str);
// true: this half-step runs the low-d pass with float64 scores (norm), false: float (norm_f)
bool lowd_precise(const Prepared *P, double eps);
fs_status lowd_lse(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps,
                   Splits *splits_out);
// the squared norms that belong to the coordinates of the half-steps at eps (Side::norm or norm_f)
inline const double *lowd_norm(const Prepared *P, const Side *res, double eps)
{
    return (P->mom.on && P->mom.eps == eps) || lowd_precise(P, eps) ? res->norm : res->norm_f;
}
// fs_moments.hip
size_t mom_bytes(int64_t n, int64_t m);
// time of a pass over the pairs on the split records (us): 9 to 12 pairs a ns, in an application 7 to 9.3 (d = 1) and 5.1 to 6.5
inline double mom_pair_cost(int64_t n, int64_t m, int64_t d, int cols)
{
    return (double)n * (double)m / (cols == 1 ? 11.4e6 : d == 1 ? 9.0e6 : 6.2e6) + 8.0;
}
// Whether moments can pay for `passes` passes at one eps: dealing the clouds to cells takes some 70 us, a pass through few cells 30 (and 10 a column).
// (Where they can't, the clouds' bounds would only cost: 4 of 100 us of a half-step call at n = 43577, m = 7343.)
inline bool mom_size(const Ctx *c, const MomState &S, int64_t n, int64_t m, int64_t d)
{
    if (!S.passes || d > 3 || c->ws_static || c->dbg_lowd_moments == 2) return false;
    return c->dbg_lowd_moments == 1 || ((double)n * (double)m >= 3.0e8 && S.passes * (mom_pair_cost(n, m, d, S.cols) - 20.0 - 10.0 * S.cols) > 40.0);
}
// (t: side of the rows, 0: X)
fs_status mom_ready(Ctx *c, const Prepared *P, double eps, int t, bool *use);
// V != nullptr: the plan application to the p columns of V as well, accumulators [rows][p] in opart
fs_status mom_pass(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, const float *V, int p, int64_t ldv, float *opart);
constexpr int kMomMaxP = 8;   // columns of an application through moments
// a half-step and its merge in one launch (small problems); *done = false: not applicable.  It leaves one gauge sum per 32
// rows, the merge kernels one per 256.
// The line, from half-steps in two launches and in one (us, of solves): d = 2: n = m = 3000 12.9 / 9.7, 8000 16.9 / 16.1; d = 4: 5400
// 15.4 / 13.2, 7000 17.0 / 15.6; d = 7: 5400 16.3 / 14.0; d = 10: 4900 16.6 / 14.2; d = 12: 4400 17.5 / 17.1, 5400 18.3 / 19.4; d = 14: 4000
// 19.8 / 17.9, 8000 27.9 / 28.7; d = 16: 3700 18.5 / 18.2, 4400 19.0 / 20.2, 8000 26.0 / 31.4.  (Below twelve dimensions one launch
// would also win a little beyond it: d = 10, n = m = 7000 19.1 / 17.4.)
inline bool lowd_small(int64_t n, int64_t m, int64_t d)
{
    return n <= 8192 && m <= 8192 && (double)n * (double)m * split_ksteps(d) <= 1.0e8;
}
fs_status lowd_half_small(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, const FinalizeArgs &fz, bool *done);
// both half-steps of an averaged iteration (Eq. 4-5) in one launch; *done = false: not applicable
fs_status lowd_lse_pair(Ctx *c, const Prepared *P, double eps, void *partial_x, void *partial_y, Splits *splits_x,
                        Splits *splits_y, bool *done);
size_t lowd_apply_ws(const Ctx *c, int64_t n_res, int64_t n_str, int64_t d, int64_t p);
// had_A != nullptr: Hadamard-weighted transport (Alg. 5), every plan entry times <had_A row i, centred
// streamed point j>; had_A is [res->cnt][lda] floats.
fs_status lowd_apply(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps,
                     const float *V, int64_t p, int64_t ldv, float *out, int64_t ldo, float *mass_out,
                     const float *had_A = nullptr, int64_t lda = 0);

// fs_f64.hip
// (prof_kind: how the launch is booked by the profiling hooks, see Ctx::ev_kind)
fs_status f64_lse(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps,
                  Splits *splits_out, int prof_kind = 0);
fs_status f64_lse_pair(Ctx *c, const Prepared *P, double eps, void *partial_x, void *partial_y, Splits *splits_x,
                       Splits *splits_y);
size_t f64_apply_ws(const Ctx *c, int64_t n_res, int64_t n_str, int64_t d, int64_t p);
fs_status f64_apply(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps,
                    const float *V, int64_t p, int64_t ldv, float *out, int64_t ldo, float *mass_out,
                    const float *hadA = nullptr, int64_t lda = 0);

// fs_fx.hip: the fixed-point kernels of a pass (P->fx_ks > 0); they leave at once where the gate is off
// (launch = false: the host knows that the gate is off, only the shapes are asked for)
fs_status fx_lse(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, int *splits, bool launch);
fs_status fx_lse_pair(Ctx *c, const Prepared *P, double eps, void *partial_x, void *partial_y, int *splits_x, int *splits_y, bool launch);
// bytes of one buffer of seeds of the rows of side t (0: X) in a call that passes over them several times; pairs: two passes a launch
size_t fx_seed_bytes(const Ctx *c, const Prepared *P, int t, bool pairs);
size_t fx_apply_ws(const Ctx *c, int64_t n_res, int64_t n_str, int64_t d, int64_t p);
fs_status fx_apply_pass(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, const float *V, int64_t p, int64_t ldv,
                        int p0, const float *hadA, int64_t lda, int *splits, int *pc, const double **had_add, bool launch);

// fs_bf16.hip
fs_status bf16_lse(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps,
                   Splits *splits_out);
fs_status bf16_lse_pair(Ctx *c, const Prepared *P, double eps, void *partial_x, void *partial_y, Splits *splits_x,
                        Splits *splits_y);
// plan application in bf16 mode (Alg. 2 / Alg. 4): workspace bytes and the pass itself
size_t bf16_apply_ws(const Ctx *c, int64_t n_res, int64_t n_str, int64_t d, int64_t p, size_t *least);
fs_status bf16_apply(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, const float *V, int64_t p,
                     int64_t ldv, float *out, int64_t ldo, float *mass_out);

// profiling helpers (fs_api.hip)
void prof_begin(Ctx *c, double pairs, int kind = 0);
void prof_end(Ctx *c);

}  // namespace fs
