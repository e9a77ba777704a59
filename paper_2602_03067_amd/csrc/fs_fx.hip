// fp32-accuracy path for 16 < d <= 128: the score contraction <x_i, y_j> in fixed point on the int8
// matrix cores (v_mfma_i32_32x32x32_i8), exact integer accumulation.
//
// Why: the fp64 matrix cores (fs_f64.hip) have 1/64 of the int8 rate.  A coordinate is 31-bit fixed
// point relative to the clouds' common scale r2 (a power of two), split into four balanced base-256
// digits,  x = r2 2^-31 sum_i D_i 2^(8 (4 - i)),  |D_1| <= 127, D_i in [-128, 127].  A product of two
// points is then a sum over digit pairs (i, j) of weight 2^(64 - 8 (i + j)), and the thirteen pairs
// with i + j <= 6 are kept (ten, i + j <= 5, where the scores are small): what is dropped is 2^-38 r2^2 sqrt(d / 64)
// rms for random digits, and the gate (FxGate, with the bounds for any digits) sends problems whose scores would feel
// it, or the rounding of the coordinates, to the fp64 kernels.  The clouds are shifted first (k_prep_fx).
//
// The pairs of equal weight share an accumulator, and neighbouring weights share a register by
// Horner's rule between MFMAs, so a score leaves the matrix cores as two integers:
//     H = 2^8 sum(1,1) + sum(i + j = 3)                      unit u3 = cscale r2^2 2^-22
//     L = 2^8 sum(i + j = 4) + sum(i + j = 5) + 2^-8 sum(i + j = 6)     unit u5 = u3 2^-16
// The streamed point's bias enters as the initial accumulators (three integers per point, units u2,
// u4, u6: see store_fx_record) and the resident row's running max m, a multiple of u3, as an integer
// subtraction, so cancellation happens in exact integer arithmetic and the vector ALU only converts
// what is left:  score - m = u3 H + u5 L.
//
// A tile of 32 streamed points whose biases do not fit that grid (padding, potentials far away) is flagged in its bias
// record and takes a float64 epilogue with the float64 biases; so does a row whose running max is beyond the integer
// range.  Points without weight are a bit mask of their tile, which costs it 32 vector instructions (in applications to more
// than four columns they take the float64 epilogue as well).  With 5 % of them most tiles hold one: ten iterations at
// n = m = 4000, d = 32 take 428 us with the mask, 890 with the float64 epilogue, 610 on the fp64 kernels.
//
// Mapping (32x32x32): A = streamed points (lane l: point l % 32, bytes 16 (l / 32) ..), B = resident
// rows, D: lane l, register r holds D[i = 8 (r / 4) + 4 (l / 32) + r % 4][j = l % 32]: the sixteen
// registers of a lane are sixteen streamed points of ONE resident row.  Digit images in HBM hold the
// fragments in lane order ([tile of 32 points][k-step of 32][digit][64 lanes][16 bytes]), so LDS is
// filled by linear direct loads and read without bank conflicts.
//
// A workgroup is four waves = 128 resident rows (their digits stay in registers) over a run of streamed tiles that pass
// through an LDS ring; two workgroups per CU, one where two rings do not fit, three in MODE 3 (fx_wg_per_cu).
//
// Long half-steps (MODE 3).  Where the scores of a row spread over hundreds of base-2 units, few tiles hold a point that counts
// (shifted normal points, n = m = 16384, d = 64, eps = 0.1: one tile of four holds a pair within 60 units of its row's largest).  The three
// leading products of a tile say so: a tile none of whose scores comes near m is left at them, with 7 or 10 of its products,
// the conversions and the exponentials undone.  m must be near the row's largest from the first tile on for that: it starts at the
// score, at the biases of this pass, of a point that the last pass over these rows in the same call found (FxSeed), which bounds
// the row's sum from below whatever the potentials have become.  The leading products come first and the max between them and
// the others, so a wave waits for its own products more often; three workgroups per CU fill those waits (168 registers: sums of one
// weight are shifted before the next ones join them).  Half-step with its merge (us): that case 216 -> 116, the self term of a
// divergence at n = 10000, d = 64 78 -> 53; where nothing can be left (unit cube) n = m = 16384, d = 64 197 -> 186, n = m = 10000, d = 128
// 132 -> 119, n = m = 8192, d = 64 53 -> 57, which is why short passes stay in MODE 0 (fx_long).
//
// Bound: matrix and vector instructions, and with them the chip's power.  A wave alone issues a vector instruction every 2.5 ns, two
// of a SIMD 1.3 (2.1 for conversions, shifts by an immediate, three-way maxima and whatever reads a scalar register), three or four 1.0
// (1.9); an MFMA takes 13.6 ns, 20 with random operands.  A tile of 32 x 32 scores at d = 64 is 20 or 26 MFMAs and about 175 vector
// instructions: 700 to 800 ns (n = m = 16384, ten products, three workgroups per CU: 305000 cycles per CU at 1.85 GHz, and with all points
// but two at zero 283000 at 2.19).  Four workgroups per CU in MODE 3 at d = 64 spill: 78.5 us against 76 at n = m = 10000.
// Measured (half-step with its merge, us, fp64 and here; unit cube, ten products): n = m = 10000, d = 64: 232 -> 77; n = 9973, m = 12007, d = 128:
// 545 -> 145; n = 9973, m = 12007, d = 20: 63.
// Error of plan sums against 64 bits (n = 3001, m = 2800, d = 64 and 128; cube, normal, pixel and two-valued points,
// everywhere between the gates): 3e-8 to 6.5e-8, 64 columns of both signs 7e-8 to 1.1e-7; fp64 scores with fp32 sums 3.4e-8 to
// 4.3e-7 and 5e-8 to 5.6e-7.
#include <type_traits>

#include "fs_internal.h"

namespace fs {
namespace {

typedef int i4 __attribute__((ext_vector_type(4)));
typedef int i16v __attribute__((ext_vector_type(16)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

constexpr int kRows = 128;           // resident rows per workgroup
constexpr int kRecBytes = 512;       // bias record of a tile

__device__ inline float fast_exp2(float v) { return __builtin_amdgcn_exp2f(v); }
__device__ inline void lds_done_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N> __device__ inline void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// the eight bf16 values with infinities and NaN replaced by zero
__device__ inline bf8 finite_only(bf8 v)
{
    uint4 u = __builtin_bit_cast(uint4, v);
    uint32_t *p = &u.x;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if ((p[k] & 0x7f80u) == 0x7f80u) p[k] &= 0xffff0000u;
        if ((p[k] & 0x7f800000u) == 0x7f800000u) p[k] &= 0xffffu;
    }
    return __builtin_bit_cast(bf8, u);
}

struct FxArgs {
    const unsigned char *res, *str;   // digit images
    const int *brec;                  // bias records of the streamed tiles
    const double *bias;               // the same biases in float64
    FxGate gate;
    int n_tiles, tiles_per_split;
    double2 *partial;                 // [splits][partial_stride] (max, sum)
    int64_t partial_stride;
    const FxSeed *seed_in;            // [seed_splits][partial_stride] of the last pass over these rows, or nullptr
    FxSeed *seed_out;                 // [splits][partial_stride], or nullptr
    int seed_splits;
    unsigned long long *count;        // COUNT: [0] tiles left at their leading products, [1] all tiles (of a wave each)
    // application
    const float *V;                   // MODE 1: [n_str][ldv] values, columns p0 ..
    int64_t ldv, n_str;
    int p0;
    const unsigned char *vimg;        // MODE 2: value images (see k_vimg_fx)
    const int *vflag;                 // MODE 2: [n_tiles] the tile holds values that are not finite
    float *opart;                     // [splits][partial_stride][PC]
    // HAD: digit image of the rows of the Hadamard factor and their scales (see k_had_digits)
    const unsigned char *had;
    const float *had_scale;
    const double *had_add;            // what the shift of the streamed points takes from the weights of a row
};

// MODE 0: log-sum-exp.  MODE 3: the same for long passes: a tile whose leading products show that it cannot count is left at them,
// and m starts at the score of a point that the last pass over these rows found.  MODE 1: application to NC <= 4 columns on the vector ALU (one fma per score and
// column).  MODE 2: application to 32 NC columns: the exponentials, in three bf16 pieces each, are the B
// operand of a second MFMA against the values in three bf16 pieces.  Six of the nine piece products are
// kept; those dropped are below 2^-25 of a product, less than one rounding of an fp32 accumulation.
// HAD (with MODE 2): Hadamard-weighted application (Alg. 5), every exponential times <row of A, streamed point>, which is
// a second contraction of the same streamed digits with those of A (a scale per row; thirteen products).
constexpr int fx_stage_bytes(int ks, int mode, int nc)
{
    return ks * 4096 + kRecBytes + (mode == 1 ? (nc + 1) / 2 * 256 : mode == 2 ? nc * 6 * 1024 : 0);
}
constexpr int fx_stages(int stage_bytes) { return stage_bytes <= 13 * 1024 ? 4 : 3; }
// Workgroups per CU: two where two rings fit the 160 KB of LDS, which the widest applications do not (four column blocks
// at any d, three at d > 64, two at d > 96).  HAD: one, the second set of resident digits takes the registers.  MODE 3: three, it
// holds fewer accumulators at a time.
constexpr int fx_wg_per_cu(int ks, int mode, int nc, bool had)
{
    const int stage = fx_stage_bytes(ks, mode, nc);
    return mode == 3 ? 3 : mode == 4 ? 2 : had || 2 * fx_stages(stage) * stage > 160 * 1024 ? 1 : 2;
}
template <int KS, int MODE, int NC, bool HAD = false> struct FxShape {
    static constexpr int kStage = fx_stage_bytes(KS, MODE, NC);
    static constexpr int kStages = fx_stages(kStage);
    // vector-memory instructions of a wave per stage
    static constexpr int kLoads = KS + 1 + (MODE == 1 ? 1 : MODE == 2 ? (NC * 6 + 3) / 4 : 0);
    static constexpr int kWgPerCu = fx_wg_per_cu(KS, MODE, NC, HAD);
    static constexpr int kPC = MODE == 2 ? 32 * NC : NC;
    // digits of a tile that stay in registers while it lasts: all of them, the leading two, or none, and then in one pass over the digits
    // (0) or in two (1): at four k-steps, where the resident digits take 64 registers of 168, the three accumulators of one pass were spilled, and
    // reloads in the loop wait for the ring (half-step in the unit cube, n = m = 15000, d = 120, thirteen products, 352 us; 331 in MODE 0, 335 here)
    static constexpr int kHold(bool full) { return KS <= 2 ? 4 : !full ? 2 : KS == 4 && MODE == 3 ? 1 : 0; }
};

// MODE 4: MODE 3 with two workgroups per CU, at four k-steps (see fx_mode).
// COUNT (with MODE 3): tiles are counted, in kernels of their own: a counter across the loop takes the others up to twenty registers,
// and where they have none left spills.
template <int KS, int MODE, int NC, bool FULL, bool HAD = false, bool COUNT = false>
__device__ __forceinline__ void fx_body(const FxArgs &a, unsigned char *ring, const int bx, const int by)
{
    using S = FxShape<KS, MODE, NC, HAD>;
    constexpr bool LONG = MODE >= 3;
    constexpr int NS = S::kStages;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int lh = l >> 5, lj = l & 31;
    const int64_t row0 = (int64_t)bx * kRows + 32 * w;
    const int t_begin = by * a.tiles_per_split;
    const int t_end = min(a.n_tiles, t_begin + a.tiles_per_split);
    const int G = t_end - t_begin;
    const unsigned ring_off = (unsigned)(size_t)ring;
    const unsigned l16 = l * 16, l4 = l * 4;

    const double u3d = a.gate.unit(22), u5d = a.gate.unit(38);
    float u3 = (float)u3d, u5 = (float)u5d;
    constexpr bool kOneStep = MODE == 1 && KS == 1;
    if (!kOneStep) asm volatile("" : "+v"(u3), "+v"(u5));   // (an instruction that reads a scalar register takes twice the time)
    const int lazy = (int)fmin(4.0 / u3d, 1073741824.0);   // see settle
    // A tile none of whose scores comes to m less this is left at its leading products.  What low digits and a bias's remainder add to a
    // score is between -193 d and 193 d + 257 of the leading digits' units (three products of 2^14 per coordinate and 2^8, the others a
    // 1/192 of that), and m is the leading part of a score or, from a seed, one with its whole bias and 15 units at most above it,
    // so with this slack an exponential that is left is less than 2^-59 of the row's largest, over all splits and whatever the digits.
    // Half-steps only: the values of an application may be of any size.
    const int skip = -(int)fmin(60.0 / u3d + (2.0 * 193.0 * 32.0 * KS + 273.0), 2147483647.0);

    int issued = 0;
    auto issue = [&]() __attribute__((always_inline)) {
        const int64_t t = t_begin + issued;
        const unsigned lds = ring_off + (issued % NS) * S::kStage;
        const unsigned char *src = a.str + t * (KS * 4096);
#pragma unroll
        for (int q = 0; q < KS; ++q) dma16s(src + (KS * w + q) * 1024, l16, lds + (KS * w + q) * 1024);
        dma4s(a.brec + t * 128 + (w & 1) * 64, l4, lds + KS * 4096 + (w & 1) * 256);
        if constexpr (MODE == 1) {
            constexpr int NV = (NC + 1) / 2;
            const int v = w % NV;
            const int c = min(2 * v + lh, NC - 1);
            int64_t i = t * 32 + lj;
            i = i < a.n_str ? i : a.n_str - 1;   // (rows beyond the matrix: only in flagged tiles, masked there)
            dma4(a.V + i * a.ldv + a.p0 + c, lds + KS * 4096 + kRecBytes + v * 256);
        }
        if constexpr (MODE == 2) {
            constexpr int PW = (NC * 6 + 3) / 4;
            const unsigned char *vs = a.vimg + t * (NC * 6 * 1024);
#pragma unroll
            for (int q = 0; q < PW; ++q) {
                const int pc = min(w * PW + q, NC * 6 - 1);   // (a repeated last piece keeps the waves' load counts equal)
                dma16s(vs + pc * 1024, l16, lds + KS * 4096 + kRecBytes + pc * 1024);
            }
        }
        ++issued;
    };

    // Everything that is loaded once, behind the first tile, and waited for once.
    if (LONG && G > 0) issue();
    int at = -1, at_dot = 0;   // the point that m was last raised for and its product with the row, in units of r2^2 2^-22
    double m0 = -INFINITY;
    if (LONG && a.seed_in) {
        // m starts at the score of the best of the points that the last pass over these rows found in its splits
        constexpr int kOnce = 6;
        FxSeed sd[kOnce];
        auto best = [&](const FxSeed &v) __attribute__((always_inline)) {
            const double score = v.point >= 0 ? fma((double)v.dot, u3d, a.bias[v.point]) : -INFINITY;
            if (score > m0) {
                m0 = score;
                at = v.point;
                at_dot = v.dot;
            }
        };
        const FxSeed *in = a.seed_in + row0 + lj;
#pragma unroll
        for (int k = 0; k < kOnce; ++k) sd[k] = in[(int64_t)min(2 * k + lh, a.seed_splits - 1) * a.partial_stride];
#pragma unroll
        for (int k = 0; k < kOnce; ++k) best(sd[k]);
        for (int k = 2 * kOnce + lh; k < a.seed_splits; k += 2) best(in[(int64_t)k * a.partial_stride]);
    }
    // resident digits: registers for the whole pass
    i4 b[KS][4], bw[HAD ? KS : 1][4];
    double w3 = 0.0, w5 = 0.0, wadd = 0.0;   // units of the Hadamard weights
    {
        const unsigned char *rt = a.res + (row0 >> 5) * (KS * 4096) + l16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int dg = 0; dg < 4; ++dg) b[ks][dg] = *reinterpret_cast<const i4 *>(rt + (ks * 4 + dg) * 1024);
        // (used here, so that the wait for these loads stands before the loop: inside it, it would wait for the ring's)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int dg = 0; dg < 4; ++dg) asm volatile("" : "+v"(b[ks][dg]));
        if constexpr (HAD) {
            const unsigned char *ht = a.had + (row0 >> 5) * (KS * 4096) + l16;
            const double sc = (double)a.had_scale[row0 + lj] * *a.gate.r2;
            w3 = ldexp(sc, -22);
            w5 = ldexp(sc, -38);
            wadd = a.had_add[row0 + lj];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int dg = 0; dg < 4; ++dg) bw[ks][dg] = *reinterpret_cast<const i4 *>(ht + (ks * 4 + dg) * 1024);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int dg = 0; dg < 4; ++dg) asm volatile("" : "+v"(bw[ks][dg]));
            asm volatile("" : "+v"(w3), "+v"(w5), "+v"(wadd));
        }
    }

    // running sum of 2^(score - m) with m = -u3 nhm (s == 0: nothing seen yet, m is free).  Sixteen scores are summed in
    // float, tiles in double: two more instructions per tile, and the sum over a long split keeps no rounding of its own.
    // `known`: m is the score of a point of the row, or was raised to one.
    double s = 0.0;
    int nhm = 0;
    bool known = false;
    if (LONG && a.seed_in) {
        const double m1 = __shfl_xor(m0, 32);
        const int at1 = __shfl_xor(at, 32), dot1 = __shfl_xor(at_dot, 32);
        if (m1 > m0 || (m1 == m0 && lh)) {   // (the same choice in both halves)
            m0 = m1;
            at = at1;
            at_dot = dot1;
        }
        const double q = floor(m0 * a.gate.per_unit(22));
        known = fabs(q) <= 1073741824.0;
        nhm = known ? -(int)q : 0;
        if (!known) at = -1;
        asm volatile("" : "+v"(nhm));   // (waited for here)
    }
    bool far = false;      // m is beyond the integer range: m = mfar
    float mfar = 0.0f;
    constexpr int NO = MODE == 2 ? NC : 1;
    f16v O[NO];
    double ov[MODE == 1 ? NC : 1];
#pragma unroll
    for (int cb = 0; cb < NO; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[cb][r] = 0.0f;
#pragma unroll
    for (int c = 0; c < (MODE == 1 ? NC : 1); ++c) ov[c] = 0.0;

    auto scale_sums = [&](float sc) __attribute__((always_inline)) {
        s *= (double)sc;
        if constexpr (MODE == 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c) ov[c] *= (double)sc;
        }
        if constexpr (MODE == 2) {
#pragma unroll
            for (int cb = 0; cb < NC; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) O[cb][r] *= sc;
        }
    };
    // the pairs (-1, 0) and (0, -1) in bf16, held in vector registers (the dot-product instruction does not read inline
    // constants as a bf16 pair)
    uint32_t ksel0 = 0, ksel1 = 0;
    if constexpr (MODE == 2) {
        asm("v_mov_b32 %0, 0xbf80" : "=v"(ksel0));
        asm("v_mov_b32 %0, 0xbf800000" : "=v"(ksel1));
    }

    // ---- scores of a tile: the digit products ------------------------------------------------------------------
    struct Tile {
        i16v H, L, Q;   // (Q: in MODE 0 and 1, see low)
        i4 av[KS][4];   // digits of the streamed points
        int kind;       // of the tile: 0 whole, 1 flagged, 2 with points without weight
    };
#define FX_MM(ACC, I, J) ACC = __builtin_amdgcn_mfma_i32_32x32x32_i8(T.av[ks][I], b[ks][J], ACC, 0, 0, 0)
    auto digits = [&](const unsigned char *sb, Tile &T, int ks, int first, int last) __attribute__((always_inline)) {
#pragma unroll
        for (int dg = first; dg <= last; ++dg) T.av[ks][dg] = *reinterpret_cast<const i4 *>(sb + l16 + (ks * 4 + dg) * 1024);
    };
    auto biases = [&](const unsigned char *sb, int which) __attribute__((always_inline)) {
        const int *rec = reinterpret_cast<const int *>(sb + KS * 4096) + 32 * which + 4 * lh;
        i16v v;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const i4 q = *reinterpret_cast<const i4 *>(rec + 8 * g4);
#pragma unroll
            for (int z = 0; z < 4; ++z) v[4 * g4 + z] = q[z];
        }
        return v;
    };
    auto contract_high = [&](const unsigned char *sb, Tile &T) __attribute__((always_inline)) {
        T.kind = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int *>(sb + KS * 4096)[96]);
        T.H = biases(sb, 0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            digits(sb, T, ks, 0, 1);
            FX_MM(T.H, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)   // (wraps are undone by what follows: only the difference counts)
            T.H[r] = (int)(((unsigned)T.H[r] << 8) + (unsigned)nhm);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            FX_MM(T.H, 0, 1);
            FX_MM(T.H, 1, 0);
        }
    };
    auto contract_low = [&](const unsigned char *sb, Tile &T) __attribute__((always_inline)) {
        constexpr int HOLD = S::kHold(FULL);
        i16v P;
        if constexpr (HOLD == 1) {
            // the products of least weight first, then one pass over the digits, two accumulators at a time beside H
            if constexpr (FULL) {
                P = biases(sb, 2);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    digits(sb, T, ks, 1, 3);
                    FX_MM(P, 3, 1);
                    FX_MM(P, 2, 2);
                    FX_MM(P, 1, 3);
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) T.L[r] = FULL ? P[r] >> 8 : 0;
            asm volatile("" : "+s"(sb));   // (read again rather than kept)
            i16v Q = biases(sb, 1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                digits(sb, T, ks, 0, 3);
                FX_MM(Q, 2, 0);
                FX_MM(T.L, 0, 3);
                FX_MM(Q, 1, 1);
                FX_MM(T.L, 1, 2);
                FX_MM(Q, 0, 2);
                FX_MM(T.L, 2, 1);
                FX_MM(T.L, 3, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) T.L[r] = (int)(((unsigned)Q[r] << 8) + (unsigned)T.L[r]);
        } else if constexpr (HOLD == 0) {
            // one pass over the digits, three accumulators
            i16v Q = biases(sb, 1);
            P = biases(sb, 2);
#pragma unroll
            for (int r = 0; r < 16; ++r) T.L[r] = 0;
            asm volatile("" : "+s"(sb));   // (read again rather than kept)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                digits(sb, T, ks, 0, 3);
                FX_MM(Q, 2, 0);
                FX_MM(T.L, 0, 3);
                FX_MM(P, 3, 1);
                FX_MM(Q, 1, 1);
                FX_MM(T.L, 1, 2);
                FX_MM(P, 2, 2);
                FX_MM(Q, 0, 2);
                FX_MM(T.L, 2, 1);
                FX_MM(P, 1, 3);
                FX_MM(T.L, 3, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) T.L[r] = (int)(((unsigned)Q[r] << 8) + (unsigned)T.L[r] + (unsigned)(P[r] >> 8));
        } else {
            // sums of one weight are shifted before those of the next one join them: fewer accumulators at a time
            if constexpr (HOLD == 4) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) digits(sb, T, ks, 2, 3);
            }
            if constexpr (FULL) {
                P = biases(sb, 2);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    FX_MM(P, 3, 1);
                    FX_MM(P, 2, 2);
                    FX_MM(P, 1, 3);
                }
            }
            T.L = biases(sb, 1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if constexpr (HOLD == 2) digits(sb, T, ks, 2, 2);
                FX_MM(T.L, 2, 0);
                FX_MM(T.L, 1, 1);
                FX_MM(T.L, 0, 2);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r)
                T.L[r] = FULL ? (int)(((unsigned)T.L[r] << 8) + (unsigned)(P[r] >> 8)) : (int)((unsigned)T.L[r] << 8);
            if constexpr (HOLD == 2) asm volatile("" : "+s"(sb));
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if constexpr (HOLD == 2) digits(sb, T, ks, 2, 3);
                FX_MM(T.L, 0, 3);
                FX_MM(T.L, 1, 2);
                FX_MM(T.L, 2, 1);
                FX_MM(T.L, 3, 0);
            }
        }
    };
    // all of them at once, where nothing is decided in between
    auto contract_all = [&](const unsigned char *sb, Tile &T) __attribute__((always_inline)) {
        constexpr bool HOLD = KS <= 2;
        T.kind = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int *>(sb + KS * 4096)[96]);
        if constexpr (HOLD) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) digits(sb, T, ks, 0, 3);
        }
        T.Q = biases(sb, 1);
        T.H = biases(sb, 0);
        // (all of them asked for before the first product; not where that costs more than it brings: one wave a SIMD waits for them, and
        // at one k-step and one column 16384 x 16384 took 194 us for 190 with this and the two other lines for kOneStep)
        if constexpr (HOLD && !HAD && !kOneStep) __builtin_amdgcn_sched_barrier(0);
        if constexpr (FULL) {
            T.L = biases(sb, 2);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if constexpr (!HOLD) digits(sb, T, ks, 1, 3);
                FX_MM(T.L, 3, 1);
                FX_MM(T.L, 2, 2);
                FX_MM(T.L, 1, 3);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) T.L[r] = T.L[r] >> 8;
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) T.L[r] = 0;
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (!HOLD) digits(sb, T, ks, 0, 2);
            FX_MM(T.H, 0, 0);
            FX_MM(T.Q, 2, 0);
            FX_MM(T.Q, 1, 1);
            FX_MM(T.Q, 0, 2);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) T.H[r] = (int)(((unsigned)T.H[r] << 8) + (unsigned)nhm);
        if constexpr (!HOLD) asm volatile("" : "+s"(sb));   // (read again rather than kept)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (!HOLD) digits(sb, T, ks, 0, 3);
            FX_MM(T.H, 0, 1);
            FX_MM(T.H, 1, 0);
            FX_MM(T.L, 0, 3);
            FX_MM(T.L, 1, 2);
            FX_MM(T.L, 2, 1);
            FX_MM(T.L, 3, 0);
        }
        if constexpr (MODE == 2 && !HAD) {
#pragma unroll
            for (int r = 0; r < 16; ++r) T.L[r] = (int)(((unsigned)T.Q[r] << 8) + (unsigned)T.L[r]);
        }
    };
#undef FX_MM
    // (not before it is used: the vector ALU is not to wait for the last of the products, see settle)
    auto low = [&](const Tile &T, int r) __attribute__((always_inline)) {
        return MODE >= 2 && !HAD ? T.L[r] : (int)(((unsigned)T.Q[r] << 8) + (unsigned)T.L[r]);
    };

    // ---- before the exponentials of tile g: the slow path of a tile, and the lift of the max ------------------
    // The points without weight as this lane's registers see them: register r is bit 8 (r / 4) + r % 4.  (Opaque to the
    // compiler, which would keep sixteen masks in registers over the whole pass.)
    auto none_of_lane = [&](int g) __attribute__((always_inline)) {
        unsigned none = reinterpret_cast<const unsigned *>(ring + (g % NS) * S::kStage + KS * 4096)[97] >> (4 * lh);
        asm volatile("" : "+v"(none));
        return none;
    };
    // their scores: 2^31 units below, 2^8 base-2 units or more (see FxGate)
    auto mask_none = [&](int g, Tile &T) __attribute__((always_inline)) {
        const unsigned none = none_of_lane(g);
#pragma unroll
        for (int r = 0; r < 16; ++r) T.H[r] = none >> (8 * (r >> 2) + (r & 3)) & 1 ? INT32_MIN : T.H[r];
    };
    auto far_tile = [&](int g, const Tile &T, float (&e)[16]) __attribute__((always_inline)) {
        // float64 scores (the record of a flagged tile holds no bias)
        const double *bd = a.bias + ((int64_t)(t_begin + g)) * 32 + 4 * lh;
        unsigned back = 0u - (unsigned)nhm;
        // (the record's biases are in where the tile is not flagged, but for points without weight)
        const unsigned add = T.kind == 1 ? 0xffffffffu : T.kind == 2 ? none_of_lane(g) : 0u;
        auto score = [&](int r) __attribute__((always_inline)) {
            const double v = fma((double)low(T, r), u5d, (double)(int)((unsigned)T.H[r] + back) * u3d);
            return add >> (8 * (r >> 2) + (r & 3)) & 1 ? v + bd[8 * (r >> 2) + (r & 3)] : v;
        };
        float mx = kNegInit;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            mx = fmaxf(mx, (float)score(r));
            asm volatile("" : "+v"(mx));   // (one after the other)
        }
        if constexpr (MODE == 2) mx = fmaxf(mx, __shfl_xor(mx, 32));   // (m is common to the two lane halves)
        double md = far ? (double)mfar : -u3d * (double)nhm;
        if (mx > kNegInit && (!known || (double)mx > md)) {
            const double q = ceil((double)mx / u3d);
            const bool out = !(fabs(q) <= 1073741824.0);
            const double mnew = out ? (double)mx : q * u3d;
            if (known) scale_sums(fast_exp2((float)(md - mnew)));
            known = true;
            md = mnew;
            nhm = out ? 0 : -(int)q;
            far = out;
            mfar = mx;
        }
        bool nan = false;
        asm volatile("" : "+v"(back));   // (the scores are formed anew rather than kept in 32 registers)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const double v = score(r) - md;
            nan = nan || v != v;
            float x = (float)fmax(v, -30000.0);
            asm volatile("" : "+v"(x));
            e[r] = fast_exp2(x);
        }
        // (MODE 2: a lane's outputs are columns, half of them, while the NaN score is in one lane half: common to the two)
        if constexpr (MODE == 2) {
            const int other = __shfl_xor((int)nan, 32);   // (by all lanes, so not behind the ||)
            nan = nan || other != 0;
        }
        if (nan) scale_sums(NAN);
        if constexpr (MODE == 1) {
            // rows beyond the matrix: zero values (every wave writes the same)
            const int left = (int)min((int64_t)32, a.n_str - (int64_t)(t_begin + g) * 32);
            float *vals = reinterpret_cast<float *>(ring + (g % NS) * S::kStage + KS * 4096 + kRecBytes);
            if (lj >= left)
                for (int c = lh; c < NC; c += 2) vals[c * 32 + lj] = 0.0f;
        }
    };
    // m moves to the largest score where one exceeds it by more than `lazy`, 4 base-2 units (a float argument of 4 is
    // rounded by 2^-23); in MODE 2 both lane halves move together, since the second MFMA sums over them.  The factor of the old sums is a
    // rounded power: what it is off by counts with the weight 2^(old m - new m) of those sums, at most 3e-8 of the new one.
    // top: the largest score of the lane, for `skip`.
    // (masked: a tile with points without weight)
    auto settle = [&](int g, Tile &T, int &top, auto masked) __attribute__((always_inline)) {
        if (masked) mask_none(g, T);
        int hx = T.H[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) hx = max(hx, T.H[r]);
        top = hx;
        if (__any(hx > lazy || !(kOneStep ? s > 0.0 : known))) {
            if constexpr (MODE == 2) hx = max(hx, __shfl_xor(hx, 32));
            const int dh = known ? max(hx, 0) : hx == INT32_MIN ? 0 : hx;
            if (LONG && a.seed_out) {
                int which = INT32_MIN;   // (the largest score but for four bits, and its register)
#pragma unroll
                for (int r = 0; r < 16; ++r) which = max(which, (T.H[r] & ~15) | r);
                if (dh != 0 || (!known && hx != INT32_MIN)) {
                    const int i = 2 * (which & 12) + 4 * lh + (which & 3);
                    const int hi = reinterpret_cast<const int *>(ring + (g % NS) * S::kStage + KS * 4096)[i];   // (of its bias)
                    at = (t_begin + g) * 32 + i;
                    at_dot = (int)((unsigned)hx - (unsigned)nhm - ((unsigned)hi << 8));
                }
            }
            known = known || hx != INT32_MIN;
            scale_sums(fast_exp2(fminf((float)-dh * u3, 0.0f)));   // (1 where nothing was seen)
            nhm -= dh;
#pragma unroll
            for (int r = 0; r < 16; ++r) T.H[r] = (int)((unsigned)T.H[r] - (unsigned)dh);
            if (masked) mask_none(g, T);   // (the subtraction has wrapped)
            top = INT32_MAX;
        }
    };
    // ---- exponentials of a tile, score - m = u3 H + u5 L ------------------------------------------------------
    auto exponentials = [&](const Tile &T, float (&e)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = fast_exp2(fmaf((float)low(T, r), u5, (float)T.H[r] * u3));
    };
    // ---- their sum and what they are applied to ----------------------------------------------------------------
    auto finish = [&](int g, const unsigned char *sb, float (&e)[16]) __attribute__((always_inline)) {
        const unsigned char *vals = sb + KS * 4096 + kRecBytes;
        float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (r & 1)
                s1 += e[r];
            else
                s0 += e[r];
        }
        s += (double)(s0 + s1);
        if constexpr (MODE == 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                float o = 0.0f;
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const float4 v = *reinterpret_cast<const float4 *>(vals + c * 128 + (8 * g4 + 4 * lh) * 4);
                    o = fmaf(e[4 * g4], v.x, o);
                    o = fmaf(e[4 * g4 + 1], v.y, o);
                    o = fmaf(e[4 * g4 + 2], v.z, o);
                    o = fmaf(e[4 * g4 + 3], v.w, o);
                }
                ov[c] += (double)o;
            }
        }
        if constexpr (HAD) {
            i16v H, Q, P;
#pragma unroll
            for (int r = 0; r < 16; ++r) H[r] = Q[r] = P[r] = 0;
            const unsigned char *fr = sb + l16;
#define FX_MW(ACC, I, J) ACC = __builtin_amdgcn_mfma_i32_32x32x32_i8(f[I], bw[ks][J], ACC, 0, 0, 0)
            // (all thirteen products: a weight may be a small remainder of large products, and nothing else of it is rounded)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                i4 f[4];
#pragma unroll
                for (int dg = 1; dg < 4; ++dg) f[dg] = *reinterpret_cast<const i4 *>(fr + (ks * 4 + dg) * 1024);
                FX_MW(P, 3, 1);
                FX_MW(P, 2, 2);
                FX_MW(P, 1, 3);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) P[r] = P[r] >> 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                i4 f[4];
#pragma unroll
                for (int dg = 0; dg < 4; ++dg) f[dg] = *reinterpret_cast<const i4 *>(fr + (ks * 4 + dg) * 1024);
                FX_MW(H, 0, 0);
                FX_MW(Q, 2, 0);
                FX_MW(Q, 1, 1);
                FX_MW(Q, 0, 2);
                FX_MW(P, 3, 0);
                FX_MW(P, 2, 1);
                FX_MW(P, 1, 2);
                FX_MW(P, 0, 3);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) H[r] <<= 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                i4 f[2];
#pragma unroll
                for (int dg = 0; dg < 2; ++dg) f[dg] = *reinterpret_cast<const i4 *>(fr + (ks * 4 + dg) * 1024);
                FX_MW(H, 0, 1);
                FX_MW(H, 1, 0);
            }
#undef FX_MW
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int L = (int)(((unsigned)Q[r] << 8) + (unsigned)P[r]);
                e[r] *= (float)fma((double)L, w5, fma((double)H[r], w3, wadd));
            }
        }
        if constexpr (MODE == 2) {
            bf8 ep[2][3];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // three bf16 pieces of eight exponentials; what a piece leaves comes from one bf16 dot product each (the
                // packed pieces with (-1, 0) or (0, -1), accumulated onto the value: exact)
                uint32_t pk[3][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float x0 = e[8 * h + 2 * q], x1 = e[8 * h + 2 * q + 1];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const bf2 hd = {(__bf16)x0, (__bf16)x1};
                        pk[k][q] = __builtin_bit_cast(uint32_t, hd);
                        if (k < 2) {
                            x0 = __builtin_amdgcn_fdot2_f32_bf16(hd, __builtin_bit_cast(bf2, ksel0), x0, false);
                            x1 = __builtin_amdgcn_fdot2_f32_bf16(hd, __builtin_bit_cast(bf2, ksel1), x1, false);
                        }
                    }
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) ep[h][k] = __builtin_bit_cast(bf8, make_uint4(pk[k][0], pk[k][1], pk[k][2], pk[k][3]));
            }
            // A tile's products are summed on the matrix cores from zero, small ones first, and added to the output by the
            // vector ALU: the matrix cores truncate where they align a product to the accumulator, and an accumulator kept
            // there over the whole pass drifts (row sums of a plan at n = 8192 by 2e-7 of their size).  The truncation goes
            // towards minus infinity, so every other tile has its values stored negated: what is left of it alternates.
            const float sign = (t_begin + g) & 1 ? -1.0f : 1.0f;
            auto second = [&](auto odd_c) __attribute__((always_inline)) {
#pragma unroll
                for (int cb = 0; cb < NC; ++cb) {
                    f16v acc = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                    bf8 v[2][3];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const unsigned char *vp = vals + ((cb * 2 + h) * 3) * 1024 + l16;
#pragma unroll
                        for (int k = 0; k < 3; ++k) v[h][k] = *reinterpret_cast<const bf8 *>(vp + k * 1024);
                        // an infinite or NaN value (in piece 0 alone) meets the leading piece of its exponential only:
                        // the later ones may be zero or negative
                        const bf8 vf = decltype(odd_c)::value ? finite_only(v[h][0]) : v[h][0];
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[h][2], ep[h][0], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, ep[h][2], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[h][1], ep[h][1], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[h][1], ep[h][0], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, ep[h][1], acc, 0, 0, 0);
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[h][0], ep[h][0], acc, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 16; ++r) O[cb][r] = fmaf(acc[r], sign, O[cb][r]);
                }
            };
            if (a.vflag[t_begin + g])
                second(std::integral_constant<bool, true>{});
            else
                second(std::integral_constant<bool, false>{});
        }
    };

    [[maybe_unused]] int left = 0;   // (COUNT: tiles that were left at their leading products)
    for (; issued < NS - 1 && issued < G;) issue();
    for (int g = 0; g < G; ++g) {
        const int newer = issued - g - 1;
        if (newer >= 2)
            wait_vm<2 * S::kLoads>();
        else if (newer == 1)
            wait_vm<S::kLoads>();
        else
            wait_vm<0>();
        lds_done_barrier();          // everybody's pieces of this tile have landed, and its predecessor is read
        if (issued < G) issue();     // into the predecessor's slot
        const unsigned char *sb = ring + (g % NS) * S::kStage;
        Tile T;
        if constexpr (LONG)
            contract_high(sb, T);
        else
            contract_all(sb, T);
        float e[16];
        int top;
        const bool near = !__any(far);
        // (Whole tiles, and those with points without weight, have code copies of their own: where the others' scores join
        // theirs, the compiler moves all of them from one set of registers to another in every tile, 3 to 5 % of a pass.  In
        // MODE 2 and 3 the copies would spill, and in MODE 2 points without weight take the float64 epilogue.  HAD has the registers, and
        // its exponentials run beside the products of the weights only from the same piece of code: 16384 x 16384, d = 64, 8 columns,
        // 667 us where they join, 619 here.)
        if constexpr (LONG) {
            const bool direct = T.kind != 1 && near;
            if (direct) {
                settle(g, T, top, T.kind == 2);
                if (!__any(top > skip)) {
                    if constexpr (COUNT) ++left;
                    continue;
                }
            }
            contract_low(sb, T);
            if (__builtin_expect(direct, 1)) {
                exponentials(T, e);
                finish(g, sb, e);
                continue;
            }
            far_tile(g, T, e);
        } else if (__builtin_expect(T.kind == 0 && near, 1)) {
            settle(g, T, top, std::false_type{});
            exponentials(T, e);
            if constexpr (MODE != 2 || HAD) {
                finish(g, sb, e);
                continue;
            }
        } else if (MODE != 2 && T.kind == 2 && near) {
            settle(g, T, top, std::true_type{});
            exponentials(T, e);
            finish(g, sb, e);
            continue;
        } else
            far_tile(g, T, e);
        finish(g, sb, e);
    }

    // merge the two lane halves of every resident row
    // (the merges expect integer maxima)
    const double mym = s == 0.0 ? (double)kNegInit : far ? (double)mfar : -u3d * (double)nhm;
    const double mo = __shfl_xor(mym, 32);
    const double so = __shfl_xor(s, 32);
    const double M = fmax(mym, mo) > (double)kNegInit ? ceil(fmax(mym, mo)) : (double)kNegInit;
    const float f0 = fast_exp2((float)(mym - M)), f1 = fast_exp2((float)(mo - M));
    const int64_t rec_row = (int64_t)by * a.partial_stride + row0 + lj;
    if (LONG && a.seed_out) {
        const int at1 = __shfl_xor(at, 32), dot1 = __shfl_xor(at_dot, 32);
        const bool other = at < 0 || (at1 >= 0 && mo > mym);   // (the half that was raised higher)
        if (lh == 0) a.seed_out[rec_row] = other ? FxSeed{dot1, at1} : FxSeed{at_dot, at};
    }
    if constexpr (COUNT) {
        if (l == 0) {
            atomicAdd(a.count, (unsigned long long)left);
            atomicAdd(a.count + 1, (unsigned long long)G);
        }
    }
    if (lh == 0) a.partial[rec_row] = make_double2(M, s * (double)f0 + so * (double)f1);
    if constexpr (MODE == 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double oo = __shfl_xor(ov[c], 32);
            if (lh == 0) a.opart[rec_row * NC + c] = (float)(ov[c] * (double)f0 + oo * (double)f1);
        }
    }
    if constexpr (MODE == 2) {
        // (m is common to the two halves; each holds half of the columns)
        const float fm = fmaxf(f0, f1);
        float *o = a.opart + rec_row * S::kPC;
#pragma unroll
        for (int cb = 0; cb < NC; ++cb)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                *reinterpret_cast<float4 *>(o + 32 * cb + 8 * g4 + 4 * lh) =
                    make_float4(O[cb][4 * g4] * fm, O[cb][4 * g4 + 1] * fm, O[cb][4 * g4 + 2] * fm, O[cb][4 * g4 + 3] * fm);
    }
}

// what a pass leaves whose scores the other kernel forms
__device__ inline void no_seeds(const FxArgs &a, int bx, int by)
{
    if (a.seed_out && threadIdx.x < kRows) a.seed_out[(int64_t)by * a.partial_stride + (int64_t)bx * kRows + threadIdx.x] = FxSeed{0, -1};
}

// (The dispatcher fills CU after CU, so half-steps are held to as many workgroups per CU as the launch shape counts on.  Applications are
// not: where more fit, a last round that is nearly empty is hidden.  Held to the one that the shape counts on, Hadamard-weighted ones to 8
// columns at n = 40000, m = 2000, d = 20 took 257 us instead of 207.)
template <int KS, int MODE, int NC, bool HAD = false, bool COUNT = false>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(FxShape<KS, MODE, NC, HAD>::kWgPerCu, MODE == 1 || MODE == 2 ? 8 : FxShape<KS, MODE, NC, HAD>::kWgPerCu)))
void k_fx(FxArgs a)
{
    using S = FxShape<KS, MODE, NC, HAD>;
    __shared__ __attribute__((aligned(1024))) unsigned char ring[S::kStages * S::kStage];
    if (!a.gate.on()) {
        no_seeds(a, blockIdx.x, blockIdx.y);
        return;
    }
    if (a.gate.full())
        fx_body<KS, MODE, NC, true, HAD, COUNT>(a, ring, blockIdx.x, blockIdx.y);
    else
        fx_body<KS, MODE, NC, false, HAD, COUNT>(a, ring, blockIdx.x, blockIdx.y);
}

// Both passes of one iteration of the averaged schedule (Eq. 4-5) in one launch: the first rb0 row blocks of the
// grid belong to the f-pass (a0), the others to the g-pass (a1).
template <int KS, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FxShape<KS, MODE, 1>::kWgPerCu, FxShape<KS, MODE, 1>::kWgPerCu)))
void k_fx_pair(FxArgs a0, FxArgs a1, int rb0, int splits0, int splits1)
{
    using S = FxShape<KS, MODE, 1>;
    __shared__ __attribute__((aligned(1024))) unsigned char ring[S::kStages * S::kStage];
    const bool second = (int)blockIdx.x >= rb0;   // uniform over the workgroup
    if ((int)blockIdx.y >= (second ? splits1 : splits0)) return;
    const int bx = (int)blockIdx.x - (second ? rb0 : 0);
    if (!a0.gate.on()) {
        no_seeds(second ? a1 : a0, bx, blockIdx.y);
        return;
    }
    if (a0.gate.full())
        fx_body<KS, MODE, 1, true>(second ? a1 : a0, ring, bx, blockIdx.y);
    else
        fx_body<KS, MODE, 1, false>(second ? a1 : a0, ring, bx, blockIdx.y);
}

// Value images for MODE 2: [tile][32-column block][16 points][piece][64 lanes][8 bf16], lane l holding column l % 32
// and the eight streamed points whose exponentials sit in that lane half (registers 8 h .. 8 h + 7 of the score tile).
// Zero outside the matrix; odd tiles hold the negated values (see finish).  A block of 128 nc threads makes the image of
// one tile.
__global__ __launch_bounds__(512) void k_vimg_fx(const float *V, int64_t ldv, int64_t n_str, int p0, int p, int nc, unsigned char *img,
                                                 int *vflag, FxGate gate)
{
    if (!gate.on()) return;
    const int64_t t = blockIdx.x;
    const int cb = threadIdx.x >> 7;
    const int h = (threadIdx.x >> 6) & 1, l = threadIdx.x & 63, lh = l >> 5;
    const int c = p0 + 32 * cb + (l & 31);
    uint32_t pk[3][4];
    int odd = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        __bf16 x[2][3];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const int r = 8 * h + 2 * q + z;
            const int64_t i = t * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
            const float u = (i < n_str && c < p) ? V[i * ldv + c] : 0.0f, v = t & 1 ? -u : u;
            split3(v, x[z]);
            if (!(fabsf(v) < INFINITY)) {
                odd = 1;
                x[z][1] = x[z][2] = (__bf16)0.0f;
            } else if (fabsf(v) > 3.3895313892515355e38f) {   // (would round to an infinite first piece)
                const float top = copysignf(3.3895313892515355e38f, v);
                x[z][0] = (__bf16)top;
                x[z][1] = (__bf16)(v - top);
                x[z][2] = (__bf16)(v - top - (float)x[z][1]);
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) pk[k][q] = bf16_pair(x[0][k], x[1][k]);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
        *reinterpret_cast<uint4 *>(img + (((t * nc + cb) * 2 + h) * 3 + k) * 1024 + l * 16) = make_uint4(pk[k][0], pk[k][1], pk[k][2], pk[k][3]);
    odd = __syncthreads_or(odd);
    if (threadIdx.x == 0) vflag[t] = odd;
}

// Digit image of the rows of A [n][lda] (layout of the points' images), each row with its own power-of-two scale; a row that
// is not finite gets the scale NaN.  add: the streamed points are stored shifted, y - origin in every coordinate, so
// <row, y> = <row, y - origin> + origin sum(row).  A block of 256 threads makes one tile of 32 rows.
__global__ __launch_bounds__(256) void k_had_digits(const float *A, int64_t lda, int64_t n, int d, int ks, const double *origin,
                                                    unsigned char *img, float *scale, double *add)
{
    __shared__ float pt[32][32 * kFxMaxKs + 1];
    __shared__ int sh_ex[32];
    const int64_t row0 = (int64_t)blockIdx.x * 32;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int r = wv; r < 32; r += 4) {
        const int64_t row = row0 + r;
        uint32_t mx = 0;
        double sum = 0.0;
        for (int k = lane; k < 32 * ks; k += 64) {
            const float v = (row < n && k < d) ? A[row * lda + k] : 0.0f;
            pt[r][k] = v;
            mx = max(mx, __float_as_uint(fabsf(v)));
            sum += (double)v;
        }
        for (int off = 32; off > 0; off >>= 1) {
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
            sum += __shfl_xor(sum, off, 64);
        }
        const float big = __uint_as_float(mx);
        int ex = 0;
        if (big < INFINITY && big > 0.0f) (void)frexp((double)big * (128.0 / 127.49), &ex);
        if (lane == 0) {
            sh_ex[r] = ex;
            scale[row] = big < INFINITY ? (float)ldexp(1.0, ex) : NAN;
            add[row] = *origin * sum;
        }
    }
    __syncthreads();
    for (int e = tid; e < ks * 64; e += 256) {
        const int q = e >> 6, l = e & 63;
        const int k0 = 32 * q + 16 * (l >> 5);
        const double to_fixed = ldexp(1.0, 31 - sh_ex[l & 31]);
        int X[16];
#pragma unroll
        for (int z = 0; z < 16; ++z) {
            const float v = pt[l & 31][k0 + z];
            X[z] = fabsf(v) < INFINITY ? (int)rint((double)v * to_fixed) : 0;
        }
        uint4 o[4];
        fx_digits16(X, o);
#pragma unroll
        for (int dg = 0; dg < 4; ++dg) *reinterpret_cast<uint4 *>(img + ((((int64_t)blockIdx.x * ks + q) * 4 + dg) << 10) + l * 16) = o[dg];
    }
}

// Launch shape: row blocks x splits of the streamed side, minimising a makespan model in units of one tile of one
// workgroup on a full CU: workgroups are dealt to the CUs evenly and run `occ` at a time (one to three); one left over where two
// would run leaves the matrix pipe partly idle and is charged 2, of three one is charged 1.75 and two 2.25 (half-steps at n = m = 10000, d = 64
// with 3, 6 and 9 splits: 103, 71 and 66 us behind the same 13; n = m = 6000 with 5, 10 and 16: 36, 25 and 22).  `startup`: filling the
// ring, loading the resident digits, the first lift of the max and the merge, in tiles.
PassShape fx_shape(const Ctx *c, int64_t n_res, int64_t n_str, int occ)
{
    PassShape s;
    s.rows_per_block = kRows;
    s.row_blocks = (int)ceil_div(n_res, kRows);
    const int n_tiles = (int)ceil_div(n_str, 32);
    int cap = max_splits(c->partial_budget, n_res);
    if (cap > n_tiles) cap = n_tiles;
    if (c->dbg_fx_splits > 0) {
        const int sp = c->dbg_fx_splits < cap ? c->dbg_fx_splits : cap;
        const int tps = (int)ceil_div(n_tiles, sp);
        s.splits = (int)ceil_div(n_tiles, tps);
        s.cols_per_split = (int64_t)tps * 32;
        return s;
    }
    const double startup = 4.0;
    double best = 0.0;
    int best_tps = n_tiles;
    for (int sp = 1; sp <= cap; ++sp) {
        const int tps = (int)ceil_div(n_tiles, sp);
        if ((int)ceil_div(n_tiles, tps) != sp) continue;
        const int64_t wg = ceil_div((int64_t)s.row_blocks * sp, (int64_t)c->num_cu);
        const int rem = (int)(wg % occ);
        const double units = (double)(wg - rem) + (rem == 0 ? 0.0 : rem == 2 ? 2.25 : occ == 3 ? 1.75 : 2.0);
        const double cost = units * ((double)tps + startup) + 0.05 * sp;
        if (best == 0.0 || cost < best * 0.995) {
            best = s.cost = cost;
            best_tps = tps;
        }
    }
    s.splits = (int)ceil_div(n_tiles, best_tps);
    s.cols_per_split = (int64_t)best_tps * 32;
    return s;
}

fs_status pass_args(Ctx *c, const Prepared *P, const Side *res, const Side *str, const PassShape &s, double eps, int mode, void *partial,
                    FxArgs *out)
{
    FxArgs a{};
    a.res = res->dig;
    a.str = str->dig;
    a.brec = str->brec;
    a.bias = str->bias_d;
    a.gate = fx_gate(P, eps);
    a.n_tiles = (int)ceil_div(str->cnt, 32);
    a.tiles_per_split = (int)(s.cols_per_split / 32);
    a.partial = (double2 *)partial;
    a.partial_stride = res->cnt_pad;
    a.n_str = str->cnt;
    a.count = c->fx_count && !capturing(c) ? c->fx_count : nullptr;   // (the counters may be gone before a graph is)
    if ((int64_t)s.row_blocks * kRows > res->cnt_pad || (int64_t)a.n_tiles * 32 > str->cnt_pad ||
        (size_t)s.splits * res->cnt_pad * 16 > P->partial_bytes || P->fx_ks < 1 || P->fx_ks > kFxMaxKs)
        return fail(c, FS_ERR_DEVICE, "internal: fixed-point launch shape exceeds the padded buffers");
    Prepared::Seeds &sd = P->seeds;
    const int t = res == &P->X ? 0 : 1;
    if (mode >= 3 && sd.last[t] >= 0) {
        a.seed_in = reinterpret_cast<const FxSeed *>(sd.buf[t][sd.last[t]]);
        a.seed_splits = sd.splits[t];
    }
    if (mode >= 3 && (size_t)s.splits * res->cnt_pad * sizeof(FxSeed) <= sd.bytes[t]) {
        const int next = sd.last[t] == 0 ? 1 : 0;
        a.seed_out = reinterpret_cast<FxSeed *>(sd.buf[t][next]);
        sd.last[t] = next;
        sd.splits[t] = s.splits;
    }
    *out = a;
    return FS_OK;
}

template <int KS>
void launch_apply(Ctx *c, const FxArgs &a, dim3 grid, int mode, int nc)
{
    if (a.had) {
        if (nc == 1)
            hipLaunchKernelGGL((k_fx<KS, 2, 1, true>), grid, dim3(256), 0, c->stream, a);
        else
            hipLaunchKernelGGL((k_fx<KS, 2, 2, true>), grid, dim3(256), 0, c->stream, a);
        return;
    }
#define FX_LAUNCH(M, N) hipLaunchKernelGGL((k_fx<KS, M, N>), grid, dim3(256), 0, c->stream, a)
    if (mode == 1) {
        switch (nc) {
        case 1: FX_LAUNCH(1, 1); break;
        case 2: FX_LAUNCH(1, 2); break;
        case 3: FX_LAUNCH(1, 3); break;
        default: FX_LAUNCH(1, 4); break;
        }
    } else {
        switch (nc) {
        case 1: FX_LAUNCH(2, 1); break;
        case 2: FX_LAUNCH(2, 2); break;
        case 3: FX_LAUNCH(2, 3); break;
        default: FX_LAUNCH(2, 4); break;
        }
    }
#undef FX_LAUNCH
}

// columns of a pass with `left` columns to go: up to 4 on the vector ALU, else blocks of 32 (at most 128; Hadamard-weighted:
// matrix blocks always, at most 64)
void fx_columns(int64_t left, bool had, int *mode, int *nc)
{
    const int64_t most = had ? 64 : 128;
    *mode = left <= 4 && !had ? 1 : 2;
    *nc = *mode == 1 ? (int)left : (int)ceil_div(left < most ? left : most, 32);
}

// buffer of a pass: [splits][rows][PC] accumulators, value images and their flags, digits, scales and summands of A
struct ApplyBuf {
    size_t vimg, vflag, had, scale, add, total;
    ApplyBuf(int splits, int64_t rows_pad, int64_t n_tiles, int ks, int mode, int nc, bool with_had)
    {
        Arena A;
        (void)A.take((size_t)splits * rows_pad * (mode == 2 ? 32 * nc : nc) * 4);
        vimg = A.take(mode == 2 ? (size_t)n_tiles * nc * 6144 : 0);
        vflag = A.take(mode == 2 ? (size_t)n_tiles * 4 : 0);
        had = A.take(with_had ? (size_t)rows_pad * ks * 128 : 0);
        scale = A.take(with_had ? (size_t)rows_pad * 4 : 0);
        add = A.take(with_had ? (size_t)rows_pad * 8 : 0);
        total = A.off;
    }
};

}  // namespace

// Whether a half-step runs in MODE 3 (`s` is its shape there, `s0` in MODE 0): where a workgroup has at least 24 tiles.  At d <= 64, where
// its three workgroups per CU bring least, they also have to fill their places: the model of the shapes may expect no more than
// 1.05 times the time in MODE 0, or, for `seeds`, the calls that pass over the rows several times, 1.09 (d <= 32) or 1.11: only
// there are tiles left early, if the clouds allow it at all.  (d > 96: see fx_mode.)  MODE 0 over MODE 3 in time, unit cube with ten products /
// with thirteen, where no tile can be left / normal points of spread 1, a unit apart, where many are, at the model's 1.0, 1.08, 1.10 and
// 1.125 (n = m = 14500, 12500, 9000; n = 20000, m = 3000):
//     solves, d = 20     1.08 1.05 1.10    1.02 1.00 1.03    0.96 0.97 0.96    0.93 0.94 0.94
//     d = 64             1.05 1.03 1.44    1.01 1.00 1.31    0.99 0.97 1.17    0.97 0.96 1.08
//     d = 96             1.11 1.01 1.56    1.07 0.98 1.42    1.05 0.96 1.28    1.05 0.96 1.15
//     single, d = 20     1.08 1.04 1.03    1.00 0.98 0.98    0.96 0.96 0.96    0.91 0.97 0.92
//     d = 64             1.04 1.02 1.04    1.01 1.00 1.00    1.01 0.96 0.99    0.99 0.94 0.95
//     d = 96             1.09 1.01 1.02    1.06 0.97 0.98    1.05 0.97 0.97    1.03 0.99 1.00
constexpr int64_t kFxLong = 24 * 32;
constexpr double kFxFilled = 1.025;   // (four k-steps)
static bool fx_long(const PassShape &s, const PassShape &s0, int ks, bool seeds)
{
    const double most = ks == 4 ? kFxFilled : ks == 3 ? INFINITY : !seeds ? 1.05 : ks == 1 ? 1.09 : 1.11;
    return s.cols_per_split >= kFxLong && s.cost <= most * s0.cost;
}

// the shape of a half-step over the rows of side t (0: X)
static const PassShape &fx_half_step(const Ctx *c, const Prepared *P, int t, int mode)
{
    PassShape &s = P->fx_shapes[t][mode ? mode - 2 : 0];
    if (s.row_blocks == 0) s = fx_shape(c, (t ? P->Y : P->X).cnt, (t ? P->X : P->Y).cnt, fx_wg_per_cu(P->fx_ks, mode, 1, false));
    return s;
}
// ... and its mode: 0, 3 or 4.  At four k-steps three workgroups per CU pay where tiles are left early, and cost where none can be and
// they do not fill their places: three for `seeds` and shapes that fill them, two for the others, and for those that have 24 tiles a
// workgroup only with two.  MODE 0 over MODE 3 and over MODE 4 at d = 120, clouds as above: solves at n = m = 15000 (the model's 1.02) 1.10 0.99
// 1.68 and 1.11 1.02 1.35, 10000 (1.026) 1.08 0.96 1.39 and 1.11 1.01 1.28, 12500 (1.084) 1.06 0.93 1.41 and 1.11 1.02 1.34; single
// half-steps at 15000 1.10 0.98 0.99 and 1.10 1.00 1.04.
static int fx_mode(const Ctx *c, const Prepared *P, int t, bool seeds)
{
    const bool two = P->fx_ks > 3;
    if (c->dbg_fx_long) return c->dbg_fx_long == 2 ? 0 : two && !seeds ? 4 : 3;
    const PassShape &s0 = fx_half_step(c, P, t, 0);
    if ((seeds || !two) && fx_long(fx_half_step(c, P, t, 3), s0, P->fx_ks, seeds)) return 3;
    return two && fx_long(fx_half_step(c, P, t, 4), s0, P->fx_ks, seeds) ? 4 : 0;
}
// (Both passes of one launch fill its places together, n = m = 9000, d = 20, us a half-step: 44.8 in MODE 0 and 42.3 in MODE 3, 48.8 and
// 45.1.  At four k-steps that is enough where one side is more than 1.5 times as long as the other, since workgroups of unequal length fill
// each other's gaps, or where the model expects both passes filled; elsewhere two per CU.  MODE 0 over MODE 3 and over MODE 4 at d = 112,
// clouds as above: n = 30000, m = 7000 (the model's 1.036) 1.29 1.11 1.84 and 1.03 0.99 1.45; 28000, 8000 (1.007) 1.17 1.02 1.75 and 1.06
// 1.01 1.48; 13500, 12000 (0.95) 1.13 1.01 1.69 and 1.09 1.02 1.51; 16000, 12500 (1.059) 1.06 0.95 1.66 and 1.09 1.01 1.51; n = m = 12500
// (1.085) 1.04 0.92 1.55 and 1.09 1.01 1.46.  The line is not sharp: 12000, 20000 (1.002) 1.08 0.95 1.72 and 1.10 1.01 1.53, in MODE 3.)
static int fx_pair_mode(const Ctx *c, const Prepared *P)
{
    const bool two = P->fx_ks > 3;
    if (c->dbg_fx_long) return c->dbg_fx_long == 2 ? 0 : 3;
    const int64_t n = P->X.cnt, m = P->Y.cnt;
    const bool unequal = 2 * n > 3 * m || 2 * m > 3 * n;
    for (int mode = 3; mode <= (two ? 4 : 3); ++mode) {
        const PassShape &sx = fx_half_step(c, P, 0, mode), &sy = fx_half_step(c, P, 1, mode);
        if (sx.cols_per_split < kFxLong || sy.cols_per_split < kFxLong) continue;
        if (mode == 4 || !two || unequal || sx.cost + sy.cost <= kFxFilled * (fx_half_step(c, P, 0, 0).cost + fx_half_step(c, P, 1, 0).cost))
            return mode;
    }
    return 0;
}

size_t fx_seed_bytes(const Ctx *c, const Prepared *P, int t, bool pairs)
{
    const int mode = pairs ? fx_pair_mode(c, P) : fx_mode(c, P, t, true);
    return mode == 0 ? 0 : (size_t)fx_half_step(c, P, t, mode).splits * (t ? P->Y : P->X).cnt_pad * sizeof(FxSeed);
}

fs_status fx_lse(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, int *splits, bool launch)
{
    FxArgs a;
    const int t = res == &P->X ? 0 : 1;
    const int mode = fx_mode(c, P, t, P->seeds.bytes[t] != 0);
    const PassShape &s = fx_half_step(c, P, t, mode);
    fs_status st = pass_args(c, P, res, str, s, eps, mode, P->partial, &a);
    if (st != FS_OK) return st;
    *splits = s.splits;
    if (!launch) {
        P->seeds.last[t] = -1;   // (nothing writes the seeds of this pass)
        return FS_OK;
    }
    const dim3 grid((unsigned)s.row_blocks, (unsigned)s.splits);
#define FX_LSE(KS)                                                                          \
    if (mode && a.count)                                                                    \
        hipLaunchKernelGGL((k_fx<KS, 3, 1, false, true>), grid, dim3(256), 0, c->stream, a); \
    else if (KS == 4 && mode == 4)                                                          \
        hipLaunchKernelGGL((k_fx<4, 4, 1>), grid, dim3(256), 0, c->stream, a);              \
    else if (mode)                                                                          \
        hipLaunchKernelGGL((k_fx<KS, 3, 1>), grid, dim3(256), 0, c->stream, a);             \
    else                                                                                    \
        hipLaunchKernelGGL((k_fx<KS, 0, 1>), grid, dim3(256), 0, c->stream, a)
    switch (P->fx_ks) {
    case 1: FX_LSE(1); break;
    case 2: FX_LSE(2); break;
    case 3: FX_LSE(3); break;
    default: FX_LSE(4); break;
    }
#undef FX_LSE
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

fs_status fx_lse_pair(Ctx *c, const Prepared *P, double eps, void *partial_x, void *partial_y, int *splits_x, int *splits_y, bool launch)
{
    FxArgs ax, ay;
    const int mode = fx_pair_mode(c, P);
    const PassShape &sx = fx_half_step(c, P, 0, mode), &sy = fx_half_step(c, P, 1, mode);
    fs_status st;
    if ((st = pass_args(c, P, &P->X, &P->Y, sx, eps, mode, partial_x, &ax)) != FS_OK) return st;
    if ((st = pass_args(c, P, &P->Y, &P->X, sy, eps, mode, partial_y, &ay)) != FS_OK) return st;
    *splits_x = sx.splits;
    *splits_y = sy.splits;
    if (!launch) {
        P->seeds.last[0] = P->seeds.last[1] = -1;
        return FS_OK;
    }
    const dim3 grid((unsigned)(sx.row_blocks + sy.row_blocks), (unsigned)(sx.splits > sy.splits ? sx.splits : sy.splits));
#define FX_PAIR(KS)                                                                                                         \
    if (KS == 4 && mode == 4)                                                                                               \
        hipLaunchKernelGGL((k_fx_pair<4, 4>), grid, dim3(256), 0, c->stream, ax, ay, sx.row_blocks, sx.splits, sy.splits);  \
    else if (mode)                                                                                                          \
        hipLaunchKernelGGL((k_fx_pair<KS, 3>), grid, dim3(256), 0, c->stream, ax, ay, sx.row_blocks, sx.splits, sy.splits); \
    else                                                                                                                    \
        hipLaunchKernelGGL((k_fx_pair<KS, 0>), grid, dim3(256), 0, c->stream, ax, ay, sx.row_blocks, sx.splits, sy.splits)
    switch (P->fx_ks) {
    case 1: FX_PAIR(1); break;
    case 2: FX_PAIR(2); break;
    case 3: FX_PAIR(3); break;
    default: FX_PAIR(4); break;
    }
#undef FX_PAIR
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

// buffer for any application to p columns, plain or Hadamard-weighted (the passes of one call differ in width and shape)
size_t fx_apply_ws(const Ctx *c, int64_t n_res, int64_t n_str, int64_t d, int64_t p)
{
    const int ks = fx_ksteps(d);
    if (ks == 0) return 0;
    size_t most = 0;
    for (int had = 0; had < 2; ++had)
        for (int64_t left : {p, p % (had ? 64 : 128)}) {   // the first pass and the last one (those between are as the first)
            if (left == 0) continue;
            int mode, nc;
            fx_columns(left, had != 0, &mode, &nc);
            const PassShape s = fx_shape(c, n_res, n_str, fx_wg_per_cu(ks, mode, nc, had != 0));
            const ApplyBuf b(s.splits, round_up(n_res, 1024), ceil_div(n_str, 32), ks, mode, nc, had != 0);
            if (b.total > most) most = b.total;
        }
    return most;
}

// one pass of an application: columns p0 .. of V; *pc = row length of the accumulators in P->extra.  hadA != nullptr:
// Hadamard-weighted, with the rows of hadA [res->cnt][lda]; *had_add: see FxArgs.
fs_status fx_apply_pass(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, const float *V, int64_t p, int64_t ldv,
                        int p0, const float *hadA, int64_t lda, int *splits, int *pc, const double **had_add, bool launch)
{
    int mode, nc;
    fx_columns(p - p0, hadA != nullptr, &mode, &nc);
    FxArgs a;
    const PassShape s = fx_shape(c, res->cnt, str->cnt, fx_wg_per_cu(P->fx_ks, mode, nc, hadA != nullptr));
    fs_status st = pass_args(c, P, res, str, s, eps, mode, P->partial, &a);
    if (st != FS_OK) return st;
    const ApplyBuf buf(s.splits, res->cnt_pad, a.n_tiles, P->fx_ks, mode, nc, hadA != nullptr);
    if (!P->extra || buf.total > P->extra_bytes) return fail(c, FS_ERR_DEVICE, "internal: fixed-point application exceeds its buffer");
    unsigned char *x = reinterpret_cast<unsigned char *>(P->extra);
    *pc = mode == 2 ? 32 * nc : nc;
    a.V = V;
    a.ldv = ldv;
    a.p0 = p0;
    a.opart = (float *)P->extra;
    a.vimg = x + buf.vimg;
    a.vflag = reinterpret_cast<const int *>(x + buf.vflag);
    if (mode == 2 && launch)
        hipLaunchKernelGGL(k_vimg_fx, dim3((unsigned)a.n_tiles), dim3(128 * nc), 0, c->stream, V, ldv, str->cnt, p0, (int)p, nc,
                           x + buf.vimg, reinterpret_cast<int *>(x + buf.vflag), a.gate);
    if (hadA) {
        a.had = x + buf.had;
        a.had_scale = reinterpret_cast<const float *>(x + buf.scale);
        double *add = reinterpret_cast<double *>(x + buf.add);
        a.had_add = add;
        *had_add = add;
        hipLaunchKernelGGL(k_had_digits, dim3((unsigned)(res->cnt_pad / 32)), dim3(256), 0, c->stream, hadA, lda, res->cnt, (int)P->d,
                           P->fx_ks, P->scalars + 11, x + buf.had, reinterpret_cast<float *>(x + buf.scale), add);
    }
    *splits = s.splits;
    if (!launch) return FS_OK;
    const dim3 grid((unsigned)s.row_blocks, (unsigned)s.splits);
    switch (P->fx_ks) {
    case 1: launch_apply<1>(c, a, grid, mode, nc); break;
    case 2: launch_apply<2>(c, a, grid, mode, nc); break;
    case 3: launch_apply<3>(c, a, grid, mode, nc); break;
    default: launch_apply<4>(c, a, grid, mode, nc); break;
    }
    FS_HIP(c, hipGetLastError());
    return FS_OK;
}

}  // namespace fs
