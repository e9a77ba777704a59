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

// piece d of a streamed-role split record: the bias in three bf16 pieces, then the three ones
// that pick up the resident row's (negated) running max
__device__ inline uint4 split_bias_piece(float bias)
{
    __bf16 b[3];
    split3(bias, b);
    const __bf16 one = (__bf16)1.0f;
    return make_uint4(bf16_pair(b[0], b[1]), bf16_pair(b[2], one), bf16_pair(one, one), 0u);
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
    const double B = rint(bias / q);
    const __bf16 da = (__bf16)(float)(rint(B * (1.0 / 65536.0)) * 65536.0 * q);
    const double ra = B * q - (double)(float)da;
    const __bf16 db = (__bf16)(float)(rint(ra / (256.0 * q)) * 256.0 * q);
    const double rb = ra - (double)(float)db;
    const __bf16 dc = (__bf16)(float)rb;
    *digits = make_uint4(bf16_pair(da, db), bf16_pair(dc, one), bf16_pair(one, one), 0u);
    if (residual) {
        __bf16 r[3];
        split3d(bias - ((double)(float)da + (double)(float)db + (double)(float)dc), r);
        *residual = make_uint2(bf16_pair(r[0], r[1]), bf16_pair(r[2], z));
    }
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

// bias in base-2 units of a streamed point:  ((pot_shifted)/eps + log w) * log2(e)
// (Alg. 1: (ghat_j + delta_j)/eps with delta = eps*log b)
// (returns the float64 bias)
__device__ inline double store_bias(const BiasSink &s, int64_t i, double pot, double inv_eps, double lw)
{
    double b = ((pot - s.norm[i]) * inv_eps + lw) * kLog2e;
    if (s.packed) {
        const float bf = (float)(((pot - s.norm_f[i]) * inv_eps + lw) * kLog2e);
        s.packed[i * s.dp + s.d] = bf;
        if (s.split) reinterpret_cast<uint4 *>(s.split)[i * (2 * s.ks) + split_piece_pos(s.ks, i, s.d)] = split_bias_piece(bf);
    }
    if (s.packed_d) s.packed_d[i * s.dpd + s.d] = b;
    if (s.split_p) {
        double q = s.q;
        if (!(q > 0.0)) {
            double gx, gy;
            split_grids(*s.rho_dev, s.q_eps, &gx, &gy);
            q = gx * gy;
        }
        uint4 *rec = reinterpret_cast<uint4 *>(s.split_p) + i * 6;
        split_precise_bias(b, q, rec + 1, reinterpret_cast<uint2 *>(rec + 5));
    }
    if (s.bias_f) s.bias_f[i] = (float)b;
    if (s.bias_d) s.bias_d[i] = b;
    return b;
}

// Bias record of the fixed-point kernels, per tile of 32 points four times 32 integers:
//   b = u2 hi + u4 lo + u6 lo2,  u2 = cscale r2^2 2^-14,  u4 = u2 2^-16,  u6 = u4 2^-16 (lo2 only where the pass forms
//   products of that weight, see FxGate::full);  the flag of the tile
// These are the initial values of the three accumulators.  |hi| <= 0.95 2^21 keeps 2^8 (hi + the leading digit products)
// within half of the integer range, so the difference of any two scores is representable.  A tile with a bias beyond
// that (or not finite), or one that is not full, is flagged and its record left zero.  All threads of a wave call this
// with consecutive i; a side's points start at a multiple of 32.
__device__ inline void store_fx_record(const BiasSink &s, int64_t i, int64_t cnt, double b, double inv_eps)
{
    FxGate gate;
    gate.r2 = s.r2;
    gate.cscale = 2.0 * kLog2e * inv_eps;
    const double B = b / gate.unit(14);
    const double hi = floor(B);
    const bool ok = i < cnt && fabs(hi) <= 1992294.0;
    const unsigned long long all = __ballot(ok);
    const bool full = (uint32_t)(threadIdx.x & 32 ? all >> 32 : all) == 0xffffffffu;
    if (i >= cnt) return;
    int *rec = s.brec + (i >> 5) * 128 + (i & 31);
    const double r = full ? (B - hi) * 65536.0 : 0.0;
    const bool fine = gate.full();
    const double lo = fine ? floor(r) : rint(r);
    rec[0] = full ? (int)hi : 0;
    rec[32] = (int)lo;
    rec[64] = fine ? (int)floor((r - lo) * 65536.0) : 0;
    rec[96] = full ? 0 : 1;
}

// Rescaling of a split's sums to the common maximum.  Every streaming kernel keeps integer-valued
// running maxima (and -3e38 for "nothing seen"), so the factor 2^(m_k - M) is an exact ldexp.
__device__ inline double rescale_split(double v, double mk, double M)
{
    const double dlt = mk - M;
    return dlt >= -1100.0 ? ldexp(v, (int)dlt) : 0.0;   // also 0 for a NaN difference (-inf - -inf)
}

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
    // the first workgroup of the following f-update collects
    double *gauge_out;
    const double *gauge_prev;
    int64_t gauge_prev_cnt;
    double gauge_prev_eps;
    double *gauge_scalars;   // [0]: the sum so far, [1]: the sum without its last term
    const double *gauge_prev_x;   // averaged schedule: the f-pass's block sums of the previous iteration
    int64_t gauge_prev_x_cnt;
};

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

// the new potential of point i from its merged statistics, and what else is asked for; *dev, *mass and *bias are left
// alone where they are not
__device__ __forceinline__ void finalize_point(const FinalizeArgs &a, const int64_t i, const double M, const double S, double *dev,
                                               double *mass, double *bias)
{
    // fhat = -eps * LSE (Alg. 1), f = fhat + alpha (Prop. 1)
    double pot_new = -a.eps * kLn2 * (M + log2(S)) + a.res_norm[i];
    const double pot_upd = pot_new;
    if (a.mix != 1.0) pot_new = (1.0 - a.mix) * a.pot[i] + a.mix * pot_new;   // averaged schedule (Eq. 4-5)
    if (a.dev_part) {
        double wi = a.w ? (double)a.w[i] : exp(a.log_uniform);
        *dev = fabs(wi * exp((a.pot[i] - pot_new) / a.eps) - wi);   // Prop. 3: r = a exp((fhat - fhat+)/eps)
    }
    if (a.gauge_out) {
        // Prop. 3: the plan's column (row) sum, from the UPDATE itself also where the stored potential is an average
        const double wi = a.w ? (double)a.w[i] : exp(a.log_uniform);
        *mass = wi > 0.0 ? wi * exp((a.pot[i] - pot_upd) / a.eps) : 0.0;
    }
    if (!a.dev_part || a.save_old) {
        if (a.save_old) a.save_old[i] = a.pot[i];
        a.pot[i] = pot_new;
        if (a.inv_eps_next > 0.0)
            *bias = store_bias(a.sink, i, pot_new, a.inv_eps_next, a.w ? log((double)a.w[i]) : a.log_uniform);
        if (a.user_out) a.user_out[i] = (float)pot_new;
    }
}

}  // namespace
}  // namespace fs
