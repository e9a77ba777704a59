// The merge of a pass's statistics into the new potential, and the biases it leaves for the pass that streams the side
// next: shared by the merge kernels (fs_prep.hip) and by the half-step kernel that merges on its own (fs_lowd.hip).
#pragma once

#include "fs_internal.h"

namespace fs {
namespace {

// block-wide sum of one double per thread (blockDim.x == 256); result valid in thread 0
__device__ inline double block_sum_256(double v, double *sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    return sh[0];
}

// the last four slots of a streamed-role split record: the bias in three pieces, and a one that picks up the resident row's
// (negated) running max
__device__ inline uint2 split_bias_words(float bias, bool negated)
{
    __bf16 b[3];
    split3(negated ? -bias : bias, b);
    return make_uint2(bf16_pair(b[0], b[1]), bf16_pair(b[2], (__bf16)(negated ? -1.0f : 1.0f)));
}

// The three 8-bit digits of a bias on the grid q and what they leave.  Inside the digit range (|bias| < 2^21 q: the
// launcher checks the biases it can foresee) every digit is exact in bf16 and the residual is bias - rint(bias/q) q.
// Each digit is taken from what the ROUNDED digits before it leave, and the residual from all three as stored, so a
// bias beyond the range (potentials that grew during a solve) still has pieces that sum to it to double precision:
// the exact window of the first k-step is lost there and the score falls back to fp32-grade accuracy instead of
// carrying a silently rounded digit.
__device__ inline void split_precise_bias(double bias, double q, uint4 *digits, uint2 *residual)
{
    const __bf16 one = (__bf16)1.0f, z = (__bf16)0.0f;
    if (!(fabs(bias) < INFINITY)) {   // padding and zero-weight points: -inf
        *digits = make_uint4(bf16_pair((__bf16)(float)bias, z), bf16_pair(z, one), bf16_pair(one, one), 0u);
        if (residual) *residual = make_uint2(0u, 0u);
        return;
    }
    const double iq = 1.0 / q;   // (q is a power of two: the products below are exact quotients)
    const double B = rint(bias * iq);
    const __bf16 da = (__bf16)(float)(rint(B * (1.0 / 65536.0)) * 65536.0 * q);
    const double ra = B * q - (double)(float)da;
    const __bf16 db = (__bf16)(float)(rint(ra * (iq * (1.0 / 256.0))) * 256.0 * q);
    const double rb = ra - (double)(float)db;
    const __bf16 dc = (__bf16)(float)rb;
    *digits = make_uint4(bf16_pair(da, db), bf16_pair(dc, one), bf16_pair(one, one), 0u);
    if (residual) {
        __bf16 r[3];
        split3d(bias - ((double)(float)da + (double)(float)db + (double)(float)dc), r);
        *residual = make_uint2(bf16_pair(r[0], r[1]), bf16_pair(r[2], z));
    }
}

// bias in base-2 units of a streamed point:  ((pot_shifted)/eps + log w) * log2(e)
// (Alg. 1: (ghat_j + delta_j)/eps with delta = eps*log b)
// (returns the float64 bias)
__device__ inline double store_bias(const BiasSink &s, int64_t i, double pot, double inv_eps, double lw, double norm, double norm_f)
{
    double b = ((pot - norm) * inv_eps + lw) * kLog2e;
    if (s.packed) {
        const float bf = (float)(((pot - norm_f) * inv_eps + lw) * kLog2e);
        s.packed[i * s.dp + s.d] = bf;
        if (s.split) reinterpret_cast<uint2 *>(s.split)[2 * split_unit(s.ks, i, 2 * s.ks - 1) + 1] = split_bias_words(bf, split_negated(i));
    }
    if (s.packed_d) s.packed_d[i * s.dpd + s.d] = b;
    if (s.split_p) {
        double q = s.q;
        if (!(q > 0.0)) {
            double gx, gy;
            split_grids(*s.rho_dev, s.q_eps, &gx, &gy);
            q = gx * gy;
        }
        uint4 *rec = reinterpret_cast<uint4 *>(s.split_p);
        split_precise_bias(b, q, rec + split_unit(3, i, 1), reinterpret_cast<uint2 *>(rec + split_unit(3, i, 5)));
    }
    if (s.bias_f) s.bias_f[i] = (float)b;
    if (s.bias_d) s.bias_d[i] = b;
    return b;
}

__device__ inline double store_bias(const BiasSink &s, int64_t i, double pot, double inv_eps, double lw)
{
    return store_bias(s, i, pot, inv_eps, lw, s.norm[i], s.packed ? s.norm_f[i] : 0.0);
}

// Bias record of the fixed-point kernels, per tile of 32 points four times 32 integers:
//   b = u2 hi + u4 lo + u6 lo2,  u2 = cscale r2^2 2^-14,  u4 = u2 2^-16,  u6 = u4 2^-16 (lo2 only where the pass forms
//   products of that weight, see FxGate::full);  the kind of the tile, and the set of its points without weight
// These are the initial values of the three accumulators.  |hi| <= 0.95 2^21 keeps 2^8 (hi + the leading digit products)
// within half of the integer range, so the difference of any two scores is representable.  Kind (rec[96]): 2 where points have
// a bias of -inf, each a bit of rec[97]; 1 (flagged, its record left zero) where another bias is beyond that range or not
// finite, or where the tile is not full; else 0.  All threads of a wave call this with consecutive i; a side's points start at a multiple of 32.
__device__ inline void store_fx_record(const BiasSink &s, int64_t i, int64_t cnt, double b, double inv_eps)
{
    FxGate gate;
    gate.r2 = s.r2;
    gate.cscale = 2.0 * kLog2e * inv_eps;
    const double B = b / gate.unit(14);
    const double hi = floor(B);
    const bool none = i < cnt && b == -INFINITY;
    const bool ok = none || (i < cnt && fabs(hi) <= 1992294.0);
    const unsigned long long all = __ballot(ok), all_none = __ballot(none);
    const bool full = (uint32_t)(threadIdx.x & 32 ? all >> 32 : all) == 0xffffffffu;
    const uint32_t set = (uint32_t)(threadIdx.x & 32 ? all_none >> 32 : all_none);
    if (i >= cnt) return;
    int *rec = s.brec + (i >> 5) * 128 + (i & 31);
    const bool in = full && !none;
    const double r = in ? (B - hi) * 65536.0 : 0.0;
    const bool fine = gate.full();
    const double lo = fine ? floor(r) : rint(r);
    rec[0] = in ? (int)hi : 0;
    rec[32] = (int)lo;
    rec[64] = fine ? (int)floor((r - lo) * 65536.0) : 0;
    rec[96] = i & 1 ? (int)set : !full ? 1 : set ? 2 : 0;   // (the set is read where the tile is full)
}

// Rescaling of a split's sums to the common maximum.  Every streaming kernel keeps integer-valued
// running maxima (and -3e38 for "nothing seen"), so the factor 2^(m_k - M) is an exact ldexp.
__device__ inline double rescale_split(double v, double mk, double M)
{
    const double dlt = mk - M;
    return dlt >= -1100.0 ? ldexp(v, (int)dlt) : 0.0;   // also 0 for a NaN difference (-inf - -inf)
}


// one workgroup: scalars[1] <- scalars[0], scalars[0] += eps ln(sum of part[0..cnt)), in a fixed order
__device__ inline void gauge_collect(const double *part, int64_t cnt, double eps, double *scalars, double *sh)
{
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < cnt; i += 256) acc += part[i];
    const double t = block_sum_256(acc, sh);
    if (threadIdx.x == 0) {
        const double prev = scalars[0];
        scalars[1] = prev;
        scalars[0] = prev + ((t > 0.0 && t < INFINITY) ? eps * log(t) : 0.0);
    }
    __syncthreads();
}

// averaged schedule, one workgroup: scalars[0] = scalars[1] += eps (ln sum(part_y) - ln sum(part_x)) / 4
__device__ inline void gauge_collect_pair(const double *part_x, int64_t cnt_x, const double *part_y, int64_t cnt_y, double eps,
                                          double *scalars, double *sh)
{
    double ax = 0.0, ay = 0.0;
    for (int64_t i = threadIdx.x; i < cnt_x; i += 256) ax += part_x[i];
    for (int64_t i = threadIdx.x; i < cnt_y; i += 256) ay += part_y[i];
    const double sx = block_sum_256(ax, sh);
    __syncthreads();
    const double sy = block_sum_256(ay, sh);
    if (threadIdx.x == 0) {
        const bool ok = sx > 0.0 && sx < INFINITY && sy > 0.0 && sy < INFINITY;
        const double v = scalars[0] + (ok ? 0.25 * eps * (log(sy) - log(sx)) : 0.0);
        scalars[0] = v;
        scalars[1] = v;
    }
    __syncthreads();
}

// What the merge needs of point i besides its statistics.  (Loaded, and its logarithm taken, before the statistics are there: behind
// them each of these loads was a round trip to memory of its own, see k_finalize.)
struct PointIn {
    double res_norm, norm, norm_f, old, wi, lw;
};
__device__ __forceinline__ PointIn load_point(const FinalizeArgs &a, const int64_t i)
{
    PointIn p{};
    p.res_norm = a.res_norm[i];
    if (a.mix != 1.0 || a.dev_part || a.gauge_out || a.save_old) p.old = a.pot[i];
    if (a.inv_eps_next > 0.0) {
        p.norm = a.sink.norm[i];
        if (a.sink.packed) p.norm_f = a.sink.norm_f[i];
    }
    if (a.w) {
        p.wi = (double)a.w[i];
        if (a.inv_eps_next > 0.0) p.lw = log(p.wi);
    } else {
        p.lw = a.log_uniform;
        if (a.dev_part || a.gauge_out) p.wi = exp(a.log_uniform);
    }
    return p;
}

// the new potential of point i from its merged statistics, and what else is asked for; *dev, *mass and *bias are left
// alone where they are not
__device__ __forceinline__ void finalize_point(const FinalizeArgs &a, const int64_t i, const PointIn &p, const double M, const double S,
                                               double *dev, double *mass, double *bias)
{
    // fhat = -eps * LSE (Alg. 1), f = fhat + alpha (Prop. 1)
    double pot_new = -a.eps * kLn2 * (M + log2(S)) + p.res_norm;
    const double pot_upd = pot_new;
    if (a.mix != 1.0) pot_new = (1.0 - a.mix) * p.old + a.mix * pot_new;   // averaged schedule (Eq. 4-5)
    if (a.dev_part) *dev = fabs(p.wi * exp((p.old - pot_new) / a.eps) - p.wi);   // Prop. 3: r = a exp((fhat - fhat+)/eps)
    // Prop. 3: the plan's column (row) sum, from the UPDATE itself also where the stored potential is an average
    if (a.gauge_out) *mass = p.wi > 0.0 ? p.wi * exp((p.old - pot_upd) / a.eps) : 0.0;
    if (!a.dev_part || a.save_old) {
        if (a.save_old) a.save_old[i] = p.old;
        a.pot[i] = pot_new;
        if (a.inv_eps_next > 0.0) *bias = store_bias(a.sink, i, pot_new, a.inv_eps_next, p.lw, p.norm, p.norm_f);
        if (a.user_out) a.user_out[i] = (float)pot_new;
    }
}

}  // namespace
}  // namespace fs
