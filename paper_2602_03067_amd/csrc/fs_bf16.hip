// bf16 matrix-core path (d >= 16): the score tile 2<x_i, y_j> of Alg. 1 / Alg. 3 is a dense
// contraction over d, computed with v_mfma_f32_32x32x16_bf16 (bf16 in, fp32 accumulate); bias,
// online LSE and potentials stay in fp32/fp64.
//
// Shape of the work.  A resident row block at d = 784..1024 does not fit on chip (256 rows x
// 800 x 2 B = 400 KB), so unlike Alg. 1 the pass is organised as a GEMM with an LSE epilogue:
// a workgroup owns 256 resident rows (j) and a group of streamed tiles (i); for every streamed
// tile of 256 points it runs the full contraction over d in chunks of 32 through a four-stage
// LDS ring filled by direct global->LDS loads (three stages in flight), then folds
// the 256 x 256 scores into the per-row running (max, sum).  Groups of streamed tiles ("splits")
// are merged afterwards.  Concurrent workgroups of one XCD form 8 x 8 super-tiles, so each panel
// chunk fetched into that XCD's L2 is shared by eight workgroups.
//
// MFMA operand roles (32x32x16): A = streamed points (i), B = resident rows (j);
//   A: lane l holds A[i = l%32][k = 8*(l/32) .. +7],  B likewise with j = l%32,
//   D: lane l, register r holds D[i = 8*(r/4) + 4*(l/32) + r%4][j = l%32],
// i.e. the 16 accumulator registers of a lane are 16 streamed points of ONE resident row, so
// the row-wise LSE runs inside the lane; lanes/waves are merged once per workgroup.
#include <type_traits>

#include "fs_internal.h"

namespace fs {
namespace {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int BI = 256;          // streamed points per tile (4 waves x 64)
constexpr int KC = 32;           // contraction chunk per pipeline stage (bf16 elements) = 64 B per row
constexpr int NBIAS = 8;         // ring of bias tiles (one per stage, deeper than the data ring)
constexpr float kLazyMax = 1.152921504606846976e18f;   // 2^60

__device__ inline float fast_exp2(float v) { return __builtin_amdgcn_exp2f(v); }

// all LDS reads of this wave have returned, then the workgroup barrier
__device__ inline void lds_done_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
template <int N> __device__ inline void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// N consecutive 1 KB pieces (N <= 4) by direct global -> LDS loads behind ONE write of the LDS base to m0, the
// pieces addressed by immediate offsets (they advance the memory and the LDS address alike).  A write to m0 waits
// until the wave's earlier direct loads have left for the address unit, so a load with its own m0 write between the
// MFMAs of the contraction loop stalls the wave behind the queue of all eight waves' loads: issuing a stage's loads
// as one run took the pass at n = m = 70000, d = 784 from 7.7 to 6.6 ms.
template <int N>
__device__ inline void dma16_run(const void *g_uniform, unsigned lane_off, unsigned lds_off)
{
    static_assert(N >= 1 && N <= 4, "immediate offsets reach 3 KB");
    if constexpr (N == 1)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(g_uniform), "s"(lds_off)
                     : "memory", "m0");
    else if constexpr (N == 2)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024" ::"v"(
                         lane_off),
                     "s"(g_uniform), "s"(lds_off)
                     : "memory", "m0");
    else if constexpr (N == 3)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024\n\t"
                     "global_load_lds_dwordx4 %0, %1 offset:2048" ::"v"(lane_off),
                     "s"(g_uniform), "s"(lds_off)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024\n\t"
                     "global_load_lds_dwordx4 %0, %1 offset:2048\n\tglobal_load_lds_dwordx4 %0, %1 offset:3072" ::"v"(lane_off),
                     "s"(g_uniform), "s"(lds_off)
                     : "memory", "m0");
}
// (n is uniform over the wave)
__device__ inline void dma16_run_n(int n, const void *g_uniform, unsigned lane_off, unsigned lds_off)
{
    switch (n) {
    case 1: dma16_run<1>(g_uniform, lane_off, lds_off); break;
    case 2: dma16_run<2>(g_uniform, lane_off, lds_off); break;
    case 3: dma16_run<3>(g_uniform, lane_off, lds_off); break;
    case 4: dma16_run<4>(g_uniform, lane_off, lds_off); break;
    default: break;
    }
}

struct BfArgs {
    const uint16_t *res;     // resident side, tiled bf16 copy (see k_prep_bf16)
    const uint16_t *str;     // streamed side, tiled bf16 copy
    const float *bias;       // [str_pad] base-2 bias of the streamed points (-inf on padding)
    int kp;                  // multiple of 32
    float cscale;            // 2 log2(e) / eps
    int n_jtiles, n_itiles, splits, tiles_per_split;
    double2 *partial;
    int64_t partial_stride;
    // plan application only
    const unsigned char *vimg;   // [n_itiles] value images (see k_vimg_bf16)
    float *opart;                // [splits][partial_stride][PC]
    // plan slab (see Epi)
    const float *rowmax;         // Plan: [resident rows] the fixed, integer-valued stabiliser of each row
    unsigned char *eslab;        // Plan: E of this slab's resident rows, tiled like the point copies with the streamed points as coordinates
    int e_chunks;                // Plan: chunks of 32 streamed points per row group of the slab; Product: chunks of both operands
    int ch_per_split;            // Product: chunks of a split of the contraction
    int row_off;                 // Plan: first row of the slab
    int out_rows;                // Product: rows of the slab, opart is [splits][out_rows][opart_ld]
    int64_t opart_ld;
};

// What a tile's 256 x 256 contraction is used for:
//   Lse      running (max, sum) of every resident row
//   Plan     the exponentials themselves, exp2(score - rowmax), rounded to bf16 and stored as the left operand of a second
//            product, with their row sums.  No running max: bf16 has the exponent range of a float, and a row whose entries
//            leave it (its sum tells) is done again by Direct.
//   Product  the second product out[row][c] = sum_i E[row][i] V[i][c]: the same contraction over the stored exponentials
//            (streamed role: rows) and the transposed values (resident role: columns), its accumulators stored as they are
//   Direct   (with PC > 0) the application over all streamed points in one workgroup, which writes its rows of the result
enum class Epi { Lse, Plan, Product, Direct };

// where Direct writes: rows of resident tiles whose flag is set
struct DirectArgs {
    const int *flags;            // [0]: any; [1 + tile of kApplyBJ rows]
    int64_t cnt;
    double inv_eps;
    const float *w;
    double log_uniform;
    const double *pot, *norm;
    int p;
    float *out;
    int64_t ldo;
    float *mass_out;
    const float *V;              // [n_str][ldv]: the value images are made in LDS
    int64_t ldv, n_str;
    int col_blocks;
};

// Workgroup shapes (WJ = waves along the resident side, each owning 128 resident rows; four waves
// along the streamed side, each owning 64 of the tile's 256 streamed points):
//   WJ = 2: 512 threads, 256 x 256 tile, ring of 4 stages x 32 KB, one workgroup per CU;
//   WJ = 1: 256 threads, 256 x 128 tile, ring of 3 stages x 24 KB, two workgroups per CU, which
//           run out of phase: one's tile epilogue (vector ALU only) and barrier waits are covered by
//           the other's MFMAs, at the price of 1.5x the operand traffic per flop.  Measured slower
//           (8.8 against 7.9 ms at n = m = 70000, d = 784): the operand traffic costs more than the
//           overlap brings.  The LSE pass is built with WJ = 2 only; the template keeps the parameter.
//
// LDS layout of a stage: row r (0..255 streamed, then the resident rows) occupies 64 bytes = four
// 16-byte pieces; piece p is stored at position p ^ ((r >> 2) & 3): sixteen consecutive rows then read
// one MFMA fragment from sixteen different 16-byte bank groups of a 256-byte line (measured fragment-read
// rate 179 B/clk/CU, against 120 with a rotation by (r >> 1) & 3 and 63 without one).
// The derived bf16 copies in HBM already have this layout in 1 KB tiles (16 rows x 32 coordinates),
// so every direct load is a linear 1 KB copy: measured 52 B/clk/CU from L2 against 26 B/clk/CU for
// 64-byte row segments, and a 256 x 256 tile needs 32 B/clk/CU at full MFMA rate.
//
// Schedule of one stage g in every wave (F0/F1 = fragment registers of the two 16-wide k-steps):
//     4 MFMA on F0(g) | read F1(g), issue the loads of stage g + NS - 1 | 4 MFMA on F0(g) | 4 MFMA on F1(g) |
//     wait "stage g+1 landed" + barrier | read F0(g+1) | 4 MFMA on F1(g)
// A wave's loads of a stage (its 1 KB pieces, consecutive in memory and in LDS) go out as ONE run behind a
// single write of m0; the biases of a streamed tile come with the tile's first stage.  The barrier and the
// LDS latency of the next fragments hide behind the last MFMAs.
// Ceiling: with random operands the matrix cores sustain ~1.83 PFLOP/s here (a loop of nothing but
// this MFMA: 2.42 PFLOP/s on constant operands, 1.83 on uniform random ones), i.e. the chip is
// power-limited well below the 2.5 PFLOP/s peak that the roofline fraction is quoted against; the
// shipped pass runs at 1.84 GHz with the matrix pipe 67 % busy.
//
// PC > 0 is the plan application (Alg. 2 / Alg. 4) in this mode: a fused matmul - softmax - matmul.
// A wave then owns JTW = 2 blocks of 32 resident rows (64 x 64 scores per tile, 256 x 128 per
// workgroup), which leaves registers for the output accumulators O[resident row][PC value columns].
// After the contraction over d the exponentials exp2(score - max) of a tile are rounded to bf16 IN
// the accumulator layout, which is exactly the B operand of a second MFMA whose contraction runs
// over the streamed points:   O^T[c][j] += sum_i Vt[c][i] E[i][j].   The value rows of the tile
// arrive as a bf16 image Vt[c][i] (rows padded to 520 bytes: conflict-free 8-byte fragment reads)
// by direct loads issued at the start of the tile's contraction.  The running max of a resident
// row is common to the two lane halves here (the second MFMA sums over them).
constexpr int kVRow = 520;                       // bytes per value column in the LDS image (256 points + pad)
constexpr int kVImgBytes(int pc) { return (pc * kVRow + 1023) / 1024 * 1024; }

template <int WJ, int NS, int JTW, int PC, bool HALF = false, Epi EPI = Epi::Lse>
__device__ __forceinline__ void lse_bf16_body(const BfArgs &a, const int block, const DirectArgs *direct = nullptr, const int p0 = 0)
{
    constexpr bool APPLY = PC > 0;
    constexpr int BJ = 32 * JTW * WJ;            // resident rows per workgroup
    constexpr int ROWS = BI + BJ;
    constexpr int STAGE_BYTES = ROWS * KC * 2;   // 32 KB / 24 KB
    constexpr int NW = 4 * WJ;                   // waves
    constexpr int PPW = (ROWS / 16) / NW;        // 1 KB pieces of a stage per wave
    constexpr int D = NS - 1;                    // stages in flight
    constexpr int NCB = APPLY ? PC / 32 : 1;     // 32-column blocks of the value matrix
    constexpr int VIMG = APPLY ? kVImgBytes(PC) : 16;
    constexpr int NVP = VIMG / 1024;             // 1 KB pieces of a value image
    static_assert((ROWS / 16) % NW == 0 && PPW <= 4 && D >= 2 && D <= 3, "pipeline shape");
    static_assert(JTW == 4 || JTW == 2, "MFMA schedules below");
    static_assert(!APPLY || (PC % 32 == 0 && BJ * PC * 4 + BJ * 64 <= NS * STAGE_BYTES), "merge buffers fit the ring");
    __shared__ __attribute__((aligned(1024))) unsigned char ring[NS * STAGE_BYTES];
    __shared__ __attribute__((aligned(256))) float bias_ring[NBIAS][BI];                 // 8,192 B
    __shared__ __attribute__((aligned(1024))) unsigned char vimg[VIMG];

    // ---- which (resident tile, split) this workgroup owns.  Workgroups go to XCDs round-robin;
    // each XCD gets a contiguous, equally long run of the work list, which is ordered in patches of
    // 8 resident tiles x 8 splits (clipped at the edges), so that the workgroups running on an
    // XCD at any time share their panels through that XCD's L2.
    const int b = block;
    const int total = a.n_jtiles * a.splits;
    const int per = (total + 7) >> 3;
    const int lb = b >> 3;
    const int idx = (b & 7) * per + lb;
    if (lb >= per || idx >= total) return;
    int jtile, split;
    {
        const int NJ = a.n_jtiles, full = a.splits >> 3, gsz = NJ * 8;
        int gs, rem, h;
        if (idx < full * gsz) {
            gs = idx / gsz;
            rem = idx - gs * gsz;
            h = 8;
        } else {
            gs = full;
            rem = idx - full * gsz;
            h = a.splits - 8 * full;
        }
        const int pj = rem / (8 * h);
        const int r = rem - pj * 8 * h;
        const int wp = min(8, NJ - 8 * pj);
        jtile = 8 * pj + r % wp;
        split = 8 * gs + r / wp;
    }

    const int tid = threadIdx.x;
    // (the wave number as a scalar: stage, piece and address arithmetic of the loads below then runs on
    // the scalar unit instead of taking vector-ALU issue slots from the MFMA loop)
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int wi = w & 3, wj = w >> 2;
    const int lh = l >> 5, lr = l & 31;
    constexpr bool PRODUCT = EPI == Epi::Product;
    // Product: one tile per workgroup, `split` counts (row tile, split of the contraction)
    const int ksplit = PRODUCT ? split / a.n_itiles : 0;
    const int ch0 = PRODUCT ? ksplit * a.ch_per_split : 0;
    const int all_chunks = PRODUCT ? a.e_chunks : a.kp / KC;                     // chunks of a row group in memory
    const int n_chunks = PRODUCT ? min(a.ch_per_split, all_chunks - ch0) : all_chunks;
    const int64_t row0 = (int64_t)jtile * BJ + (EPI == Epi::Plan ? a.row_off : 0);
    const int t_begin = PRODUCT ? split % a.n_itiles : split * a.tiles_per_split;
    const int t_end = PRODUCT ? t_begin + 1 : min(a.n_itiles, t_begin + a.tiles_per_split);
    const int G = (t_end - t_begin) * n_chunks;   // pipeline stages of this workgroup

    const unsigned ring_off = (unsigned)(size_t)ring;
    const unsigned bias_off = (unsigned)(size_t)&bias_ring[0][0];
    const unsigned vimg_off = (unsigned)(size_t)vimg;

    // The bf16 copies are stored as 1 KB tiles (16 rows x 32 coordinates, already swizzled); the sixteen
    // tiles of a group of 256 rows at one chunk are contiguous (16 KB) and the chunks of a group follow
    // each other: a stage is ROWS/16 linear 1 KB copies, PPW consecutive ones per wave (pieces w PPW + q;
    // 0..15 streamed rows, then the resident rows), so a wave's loads of a stage, and of the next, walk
    // through memory linearly.
    const unsigned char *res_tiles = reinterpret_cast<const unsigned char *>(a.res) +
                                     ((((int64_t)(row0 >> 8) * all_chunks + ch0) * 16 + ((row0 >> 4) & 15)) << 10);
    const unsigned char *str_tiles = reinterpret_cast<const unsigned char *>(a.str);
    const unsigned l16 = l * 16, l4 = l * 4;

    int pg = 0, pch = 0, pt = t_begin;   // next stage this wave issues: number, chunk, tile
    // This wave's share of the next stage: PPW consecutive pieces starting at piece w PPW, i.e. one run of the
    // streamed group and / or one of the resident group; with the first stage of a tile also the wave's quarter of the
    // tile's biases (with two waves per streamed quarter both write the same 256 bytes: harmless).
    auto issue_stage = [&]() {
        if (!PRODUCT && pch == 0) dma4s(a.bias + (int64_t)pt * BI + wi * 64, l4, bias_off + ((pt - t_begin) & (NBIAS - 1)) * (BI * 4) + wi * 256);
        const int s0 = w * PPW;
        const int n_str = s0 >= 16 ? 0 : (16 - s0 < PPW ? 16 - s0 : PPW);
        const unsigned lds = ring_off + (pg % NS) * STAGE_BYTES;
        if (n_str > 0)
            dma16_run_n(n_str, str_tiles + ((((int64_t)pt * all_chunks + ch0 + pch) * 16 + s0) << 10), l16, lds + s0 * 1024);
        if (n_str < PPW)
            dma16_run_n(PPW - n_str, res_tiles + (((int64_t)pch * 16 + (s0 + n_str - 16)) << 10), l16, lds + (s0 + n_str) * 1024);
        ++pg;
        if (++pch == n_chunks) {
            pch = 0;
            ++pt;
        }
    };

    float mrun[JTW], srun[JTW];
    f16v O[APPLY ? JTW : 1][NCB];
#pragma unroll
    for (int jt = 0; jt < JTW; ++jt) {
        mrun[jt] = EPI == Epi::Plan ? a.rowmax[row0 + 32 * JTW * wj + 32 * jt + lr] : kNegInit;
        srun[jt] = 0.0f;
        if constexpr (EPI == Epi::Plan) asm volatile("" : "+v"(mrun[jt]));   // (loaded before the ring's loads start)
    }
    if constexpr (APPLY) {
#pragma unroll
        for (int jt = 0; jt < JTW; ++jt)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) O[jt][cb][r] = 0.0f;
    }

    // fragment addressing inside a stage
    const int sw = (lr >> 2) & 3;
    const int offA = (64 * wi + lr) * 64, offB = (BI + 32 * JTW * wj + lr) * 64;
    const int pk0 = ((0 + lh) ^ sw) * 16, pk1 = ((2 + lh) ^ sw) * 16;
    bf8 a0[2], b0[JTW], a1[2], b1[JTW];
    auto read_frags = [&](bf8(&af)[2], bf8(&bf)[JTW], int stage, int pk) {
        const unsigned char *sb = ring + (stage % NS) * STAGE_BYTES + pk;
#pragma unroll
        for (int it = 0; it < 2; ++it) af[it] = *reinterpret_cast<const bf8 *>(sb + offA + it * 32 * 64);
#pragma unroll
        for (int jt = 0; jt < JTW; ++jt) bf[jt] = *reinterpret_cast<const bf8 *>(sb + offB + jt * 32 * 64);
    };
    // this wave's loads of stage `upto` and older have landed, given that it has issued stages up to `issued`
    // (loads of a value image issued in between only make these waits stricter)
    auto wait_landed = [&](int upto, int issued) {
        const int newer = issued - upto;   // whole stages issued after `upto`
        // (a stage has PPW loads of this wave, the first stage of a tile one more: counting PPW per newer stage
        // can only wait for more than necessary)
        if (newer >= 2)
            wait_vm<2 * PPW>();
        else if (newer == 1)
            wait_vm<PPW>();
        else
            wait_vm<0>();
    };
    int vstamp = 0;   // pg when this wave issued its pieces of the current tile's value image
    auto issue_vimg = [&](int t) {
        if constexpr (EPI == Epi::Direct) {
            for (int e = tid; e < BI * PC; e += 256 * WJ) {
                const int i = e / PC, cc = e - i * PC;
                const int64_t row = (int64_t)t * BI + i;
                const float v = (row < direct->n_str && p0 + cc < direct->p) ? direct->V[row * direct->ldv + p0 + cc] : 0.0f;
                *reinterpret_cast<__bf16 *>(vimg + cc * kVRow + 2 * i) = (__bf16)v;
            }
            vstamp = pg;
        } else if constexpr (APPLY) {
            const unsigned char *src = reinterpret_cast<const unsigned char *>(a.vimg) + (int64_t)t * VIMG;
            // consecutive pieces per wave, in runs of up to four behind one LDS base each
            constexpr int VPW = (NVP + NW - 1) / NW;
            const int p0 = w * VPW;
            const int cnt = p0 >= NVP ? 0 : (NVP - p0 < VPW ? NVP - p0 : VPW);
#pragma unroll
            for (int r0 = 0; r0 < VPW; r0 += 4) {
                const int n = cnt - r0 < 4 ? cnt - r0 : 4;
                if (n > 0) dma16_run_n(n, src + (p0 + r0) * 1024, l16, vimg_off + (p0 + r0) * 1024);
            }
            vstamp = pg;
        }
    };

    // ---- prologue: D stages in flight, stage 0 landed, its first fragments on the way ----
    while (pg < D && pg < G) issue_stage();
    wait_landed(0, pg - 1);
    lds_done_barrier();
    read_frags(a0, b0, 0, pk0);

    int g = 0;
    for (int t = t_begin; t < t_end; ++t) {
        f16v acc[2][JTW];
        if constexpr (APPLY) {
#pragma unroll
            for (int it = 0; it < 2; ++it)
#pragma unroll
                for (int jt = 0; jt < JTW; ++jt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[it][jt][r] = 0.0f;
        }

        if constexpr (!APPLY) {
            // One stage of the LSE pass.  The first chunk of a tile has a code copy of its own, in which the first
            // eight MFMAs start from a zero accumulator operand: no registers to clear per tile.
            //     4 MFMA on F0(g) | read F1(g), issue stage g+3 | 4 MFMA on F0(g) | 4 MFMA on F1(g) |
            //     wait "stage g+1 landed" + barrier | read F0(g+1) | 4 MFMA on F1(g)
            // Stage g + D goes to the ring slot of stage g - 1, which nobody reads any more: every
            // wave had its reads of that stage back before it passed the barrier of stage g - 1.
            auto stage = [&](auto first_c, auto half_c) {
                constexpr bool FIRST = decltype(first_c)::value;
                constexpr bool skip_second = decltype(half_c)::value;
                const f16v zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#define FS_MFMA0(IT, JT) acc[IT][JT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[IT], b0[JT], FIRST ? zero : acc[IT][JT], 0, 0, 0)
#define FS_MFMA1(IT, JT) acc[IT][JT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[IT], b1[JT], acc[IT][JT], 0, 0, 0)
                // (only F0(g) is pending here, so the wait the compiler puts before the first MFMA is
                // exactly "F0 has arrived"; F1 is requested behind the first MFMA group)
#pragma unroll
                for (int jt = 0; jt < JTW; ++jt) FS_MFMA0(0, jt);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (!skip_second) read_frags(a1, b1, g, pk1);
                if (g + D < G) issue_stage();
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int jt = 0; jt < JTW; ++jt) FS_MFMA0(1, jt);
                // (the second 16 coordinates of a tile's last chunk are zero padding when d ends in its first half:
                // 784 = 49 x 16 saves 2 % of the MFMAs this way)
                if constexpr (!skip_second) {
#pragma unroll
                    for (int jt = 0; jt < JTW; ++jt) FS_MFMA1(0, jt);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (g + 1 < G) {
                    wait_landed(g + 1, pg - 1);   // this wave's pieces of stage g+1 have landed ...
                    lds_done_barrier();           // ... and after the barrier everybody's; F0 may be refilled
                    read_frags(a0, b0, g + 1, pk0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (!skip_second) {
#pragma unroll
                    for (int jt = 0; jt < JTW; ++jt) FS_MFMA1(1, jt);
                }
#undef FS_MFMA0
#undef FS_MFMA1
                ++g;
            };
            using yes = std::integral_constant<bool, true>;
            using no = std::integral_constant<bool, false>;
            // (HALF: the launcher has checked that d ends in the first 16 coordinates of the last chunk and that a
            // tile has at least two chunks; the three code copies follow each other without a branch between them)
            stage(yes{}, no{});
            if constexpr (HALF) {
                for (int ch = 1; ch + 1 < n_chunks; ++ch) stage(no{}, no{});
                stage(no{}, yes{});
            } else {
                for (int ch = 1; ch < n_chunks; ++ch) stage(no{}, no{});
            }
        }
        for (int ch = 0; APPLY && ch < n_chunks; ++ch, ++g) {
            const bool issue = g + D < G;
#define FS_MFMA(IT, JT, AF, BF) acc[IT][JT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(AF[IT], BF[JT], acc[IT][JT], 0, 0, 0)
#define FS_PIECE(Q)                          \
    __builtin_amdgcn_sched_barrier(0);       \
    if (Q == 0 && issue) issue_stage();      \
    __builtin_amdgcn_sched_barrier(0)
            // (plan application: 64 x 64 scores per wave)
            //     2 MFMA on F0(g) | read F1(g), issue stage g+3 | 2 MFMA on F0(g) | 2 MFMA on F1(g) |
            //     wait "stage g+1 landed" + barrier | read F0(g+1) | 2 MFMA on F1(g)
            static_assert(!APPLY || JTW == 2, "schedule of the application");
            FS_MFMA(0, 0, a0, b0);
            FS_MFMA(0, 1, a0, b0);
            __builtin_amdgcn_sched_barrier(0);
            read_frags(a1, b1, g, pk1);
            FS_PIECE(0);
            FS_MFMA(1, 0, a0, b0);
            FS_MFMA(1, 1, a0, b0);
            FS_MFMA(0, 0, a1, b1);
            FS_MFMA(0, 1, a1, b1);
            __builtin_amdgcn_sched_barrier(0);
            if (g + 1 < G) {
                // this wave's pieces of stage g+1 have landed ...
                wait_landed(g + 1, pg - 1);
                // ... and after the barrier everybody's; F0 may be refilled
                lds_done_barrier();
                read_frags(a0, b0, g + 1, pk0);
            }
            if constexpr (APPLY) {
                // every wave is past the previous tile's use of the value image now
                if (ch == 0) {
                    if (g + 1 >= G) lds_done_barrier();
                    issue_vimg(t);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            FS_MFMA(1, 0, a1, b1);
            FS_MFMA(1, 1, a1, b1);
#undef FS_MFMA
#undef FS_PIECE
        }

        // ---- epilogue: fold 2 x 16 streamed points per resident row into (max, sum) ----------
        // lazy stabiliser: exponents against the current integer running max; the slow branch
        // (lift the max, rescale by an exact power of two) runs only when a sum leaves [0, 2^60)
        if constexpr (PRODUCT) {
            // accumulator register r of block it: row 64 wi + 32 it + 8 (r / 4) + 4 lh + r % 4 of the tile; lane: column
#pragma unroll
            for (int jt = 0; jt < JTW; ++jt) {
                const int64_t c = row0 + 32 * JTW * wj + 32 * jt + lr;
#pragma unroll
                for (int it = 0; it < 2; ++it)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int64_t row = (int64_t)t * BI + 64 * wi + 32 * it + 8 * (r >> 2) + 4 * lh + (r & 3);
                        a.opart[((int64_t)ksplit * a.out_rows + row) * a.opart_ld + c] = acc[it][jt][r];
                    }
            }
            continue;
        }
        const int bslot = (t - t_begin) & (NBIAS - 1);   // the first stage of this tile carried its biases
        float bias[2][16];
#pragma unroll
        for (int it = 0; it < 2; ++it)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                float4 bv = *reinterpret_cast<const float4 *>(&bias_ring[bslot][64 * wi + 32 * it + 8 * g4 + 4 * lh]);
                bias[it][4 * g4 + 0] = bv.x;
                bias[it][4 * g4 + 1] = bv.y;
                bias[it][4 * g4 + 2] = bv.z;
                bias[it][4 * g4 + 3] = bv.w;
            }
        if constexpr (EPI == Epi::Plan) {
            // A lane half holds streamed points 8 g4 + 4 lh .. + 3 of resident row rl, half a 16-byte piece of the slab's
            // tile.  Swapping the upper lanes of an even g4 with the lower ones of the next gives every lane a whole
            // piece: g4 in the lower half, g4 + 1 in the upper one.
#pragma unroll
            for (int jt = 0; jt < JTW; ++jt) {
                const int rl = 32 * JTW * wj + 32 * jt + lr;
                const int64_t group = (row0 - a.row_off + rl) >> 8, rb = (row0 + rl) >> 4 & 15;
                float part = 0.0f;
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    unsigned char *dst = a.eslab + (((group * a.e_chunks + t * (BI / KC) + 2 * wi + it) * 16 + rb) << 10) + (rl & 15) * 64;
#pragma unroll
                    for (int g2 = 0; g2 < 2; ++g2) {
                        uint32_t pk[2][2];
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            float ev[4];
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const int e = 4 * (2 * g2 + h) + q;
                                ev[q] = fast_exp2(fmaf(acc[it][jt][e], a.cscale, bias[it][e]) - mrun[jt]);
                                part += ev[q];
                            }
                            pk[h][0] = bf16_pair((__bf16)ev[0], (__bf16)ev[1]);
                            pk[h][1] = bf16_pair((__bf16)ev[2], (__bf16)ev[3]);
                        }
                        const auto s0 = __builtin_amdgcn_permlane32_swap(pk[0][0], pk[1][0], false, false);
                        const auto s1 = __builtin_amdgcn_permlane32_swap(pk[0][1], pk[1][1], false, false);
                        *reinterpret_cast<uint4 *>(dst + (((2 * g2 + lh) ^ ((rl >> 2) & 3)) << 4)) = make_uint4(s0[0], s1[0], s0[1], s1[1]);
                    }
                }
                srun[jt] += part;
            }
        } else if constexpr (!APPLY) {
            float csum[JTW];
            bool bad = false;
#pragma unroll
            for (int jt = 0; jt < JTW; ++jt) {
                const float m = mrun[jt];
                float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    s0 += fast_exp2(fmaf(acc[0][jt][r], a.cscale, bias[0][r]) - m);
                    s1 += fast_exp2(fmaf(acc[1][jt][r], a.cscale, bias[1][r]) - m);
                }
                csum[jt] = s0 + s1;
                bad = bad || !(csum[jt] < kLazyMax);
            }
            if (__any(bad)) {
#pragma unroll
                for (int jt = 0; jt < JTW; ++jt) {
                    float mx = kNegInit;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        mx = fmaxf(mx, fmaf(acc[0][jt][r], a.cscale, bias[0][r]));
                        mx = fmaxf(mx, fmaf(acc[1][jt][r], a.cscale, bias[1][r]));
                    }
                    float mnew = fmaxf(mrun[jt], ceilf(mx));
                    float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        s0 += fast_exp2(fmaf(acc[0][jt][r], a.cscale, bias[0][r]) - mnew);
                        s1 += fast_exp2(fmaf(acc[1][jt][r], a.cscale, bias[1][r]) - mnew);
                    }
                    csum[jt] = s0 + s1;
                    srun[jt] *= fast_exp2(mrun[jt] - mnew);
                    mrun[jt] = mnew;
                }
            }
#pragma unroll
            for (int jt = 0; jt < JTW; ++jt) srun[jt] += csum[jt];
        } else {
            // scores in place of the accumulators
#pragma unroll
            for (int it = 0; it < 2; ++it)
#pragma unroll
                for (int jt = 0; jt < JTW; ++jt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[it][jt][r] = fmaf(acc[it][jt][r], a.cscale, bias[it][r]);
            // the stabiliser must keep every exponential representable in bf16 next to the row's
            // largest one and the fp32 sums finite: lift it when a score exceeds it by more than 60
            bool lift = false;
            float mx[JTW];
#pragma unroll
            for (int jt = 0; jt < JTW; ++jt) {
                float m = kNegInit;
#pragma unroll
                for (int r = 0; r < 16; ++r) m = fmaxf(m, fmaxf(acc[0][jt][r], acc[1][jt][r]));
                m = fmaxf(m, __shfl_xor(m, 32, 64));   // common to the two lane halves of the row
                mx[jt] = m;
                lift = lift || (m > mrun[jt] + 60.0f);
            }
            if (__any(lift)) {
#pragma unroll
                for (int jt = 0; jt < JTW; ++jt) {
                    const float mnew = fmaxf(mrun[jt], ceilf(mx[jt]));
                    const float scale = fast_exp2(mrun[jt] - mnew);   // exact power of two (or 0)
                    srun[jt] *= scale;
                    mrun[jt] = mnew;
                    // accumulator column n = lr is this lane's resident row: one factor per lane
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                        for (int r = 0; r < 16; ++r) O[jt][cb][r] *= scale;
                }
            }
            // this wave's pieces of the value image have landed, then everybody's
            {
                const int newer = pg - vstamp;
                if (newer >= 2)
                    wait_vm<2 * PPW>();
                else if (newer == 1)
                    wait_vm<PPW>();
                else
                    wait_vm<0>();
            }
            lds_done_barrier();
#pragma unroll
            for (int it = 0; it < 2; ++it)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    // A fragments: Vt[c = 32 cb + lr][the eight streamed points of this lane half]
                    bf8 vf[NCB];
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) {
                        const unsigned char *vp = vimg + (32 * cb + lr) * kVRow + 2 * (64 * wi + 32 * it + 16 * s + 4 * lh);
                        const uint2 lo = *reinterpret_cast<const uint2 *>(vp);
                        const uint2 hi = *reinterpret_cast<const uint2 *>(vp + 16);
                        const uint4 u = make_uint4(lo.x, lo.y, hi.x, hi.y);
                        vf[cb] = *reinterpret_cast<const bf8 *>(&u);
                    }
#pragma unroll
                    for (int jt = 0; jt < JTW; ++jt) {
                        bf8 e;
                        float part = 0.0f;
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            const float ev = fast_exp2(acc[it][jt][8 * s + q] - mrun[jt]);
                            part += ev;
                            e[q] = (__bf16)ev;
                        }
                        srun[jt] += part;
#pragma unroll
                        for (int cb = 0; cb < NCB; ++cb)
                            O[jt][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[cb], e, O[jt][cb], 0, 0, 0);
                    }
                }
        }
    }

    if constexpr (PRODUCT) return;
    // ---- merge the 2 lane halves x 4 streamed-side waves of every resident row -------------
    lds_done_barrier();   // the ring is free: reuse it for the merge
    float2 *red = reinterpret_cast<float2 *>(ring);   // [BJ][8]: 4 streamed-side waves x 2 lane halves per row
#pragma unroll
    for (int jt = 0; jt < JTW; ++jt)
        red[(32 * JTW * wj + 32 * jt + lr) * 8 + 2 * wi + lh] = make_float2(mrun[jt], srun[jt]);
    __syncthreads();
    if constexpr (APPLY) {
        // output accumulators: scaled to the row's common max and added wave by wave (fixed order)
        float *obuf = reinterpret_cast<float *>(ring + BJ * 64);   // [BJ][PC]
        for (int ww = 0; ww < 4; ++ww) {
            if (wi == ww) {
#pragma unroll
                for (int jt = 0; jt < JTW; ++jt) {
                    const int j = 32 * JTW * wj + 32 * jt + lr;
                    float M = kNegInit;
#pragma unroll
                    for (int k = 0; k < 8; ++k) M = fmaxf(M, red[j * 8 + k].x);
                    const float sc = fast_exp2(mrun[jt] - M);
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int cc = 32 * cb + 8 * (r >> 2) + 4 * lh + (r & 3);
                            const float v = O[jt][cb][r] * sc;
                            obuf[j * PC + cc] = ww == 0 ? v : obuf[j * PC + cc] + v;
                        }
                }
            }
            __syncthreads();
        }
        if constexpr (EPI == Epi::Direct) {
            // (as launch_apply_finalize does it from the records of the splits)
            double *fac = reinterpret_cast<double *>(&bias_ring[0][0]);
            static_assert(BJ * 8 <= sizeof(bias_ring), "row factors fit the bias ring");
            if (tid < BJ) {
                float M = kNegInit;
                double S = 0.0;
#pragma unroll
                for (int k = 0; k < 8; ++k) M = fmaxf(M, red[tid * 8 + k].x);
#pragma unroll
                for (int k = 0; k < 8; ++k) S += (double)(red[tid * 8 + k].y * fast_exp2(red[tid * 8 + k].x - M));
                const int64_t i = row0 + tid;
                if (i < direct->cnt) {
                    const double lw = direct->w ? log((double)direct->w[i]) : direct->log_uniform;
                    fac[tid] = exp2(((direct->pot[i] - direct->norm[i]) * direct->inv_eps + lw) * kLog2e + (double)M);
                    if (direct->mass_out && p0 == 0) direct->mass_out[i] = (float)(fac[tid] * S);
                }
            }
            __syncthreads();
            for (int e = tid; e < BJ * PC; e += 256 * WJ) {
                const int j = e / PC, cc = e - j * PC;
                if (row0 + j < direct->cnt && p0 + cc < direct->p)
                    direct->out[(row0 + j) * direct->ldo + p0 + cc] = (float)(fac[j] * (double)obuf[e]);
            }
            return;
        }
        for (int e = tid; e < BJ * PC; e += 256 * WJ) {
            const int j = e / PC, cc = e - j * PC;
            a.opart[((int64_t)split * a.partial_stride + row0 + j) * PC + cc] = obuf[e];
        }
    }
    if (tid < BJ) {
        float M = kNegInit;
#pragma unroll
        for (int k = 0; k < 8; ++k) M = fmaxf(M, red[tid * 8 + k].x);
        double S = 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float2 q = red[tid * 8 + k];
            S += (double)(q.y * fast_exp2(q.x - M));
        }
        a.partial[(int64_t)split * a.partial_stride + row0 + tid] = make_double2((double)M, S);
    }
}

template <int WJ, int NS, int JTW, int PC, bool HALF = false, Epi EPI = Epi::Lse>
__global__ __launch_bounds__(256 * WJ, WJ == 2 ? 1 : 2) void k_lse_bf16(BfArgs a)
{
    lse_bf16_body<WJ, NS, JTW, PC, HALF, EPI>(a, blockIdx.x);
}

// Both LSE passes of one iteration of the averaged schedule (Eq. 4-5) in one launch: the first `blocks0`
// workgroups (a multiple of 8, so that the dealing to XCDs is the same as in a launch of its own) run the
// f-pass, the others the g-pass.
template <int WJ, int NS, int JTW>
__global__ __launch_bounds__(256 * WJ, WJ == 2 ? 1 : 2) void k_lse_bf16_pair(BfArgs a0, BfArgs a1, int blocks0)
{
    const bool second = (int)blockIdx.x >= blocks0;   // uniform over the workgroup
    lse_bf16_body<WJ, NS, JTW, 0>(second ? a1 : a0, (int)blockIdx.x - (second ? blocks0 : 0));
}

// Rows of the plan whose entries left the exponent range of a stored slab (see k_plan_finalize): workgroup (row tile, first of
// every gridDim.y column blocks), all of which leave at once where the row tile has no such row.  (Mostly that is all of them,
// one at a time per CU with this much LDS: a workgroup for each of 313 x 9 pairs took 12 us to leave.)
template <int PC>
__global__ __launch_bounds__(512, 1) void k_apply_direct(BfArgs a, DirectArgs o)
{
    const int jtile = blockIdx.x;
    if (!o.flags[1 + jtile]) return;
    const int per = (a.n_jtiles + 7) >> 3;   // (the inverse of the body's dealing, for one split)
    for (int cb = blockIdx.y; cb < o.col_blocks; cb += gridDim.y) {
        lse_bf16_body<2, 4, 2, PC, false, Epi::Direct>(a, (jtile % per) * 8 + jtile / per, &o, cb * PC);
        __syncthreads();   // the rows are written from LDS
    }
}

// Value image of every streamed tile for the plan application: bf16 Vt[c][i], c < pc value columns
// starting at p0, i < 256 points of tile t, rows of kVRow bytes, one image per img_bytes; zero
// outside the matrix.  (The pad bytes are copied to LDS with the rest and never read.)
__global__ __launch_bounds__(BI) void k_vimg_bf16(const float *V, int64_t ldv, int64_t n_str, int p0, int p, int pc,
                                                   int img_bytes, unsigned char *img)
{
    const int i = threadIdx.x;
    const int64_t row = (int64_t)blockIdx.x * BI + i;
    unsigned char *dst = img + (int64_t)blockIdx.x * img_bytes;
    for (int cc = 0; cc < pc; ++cc) {
        const float v = (row < n_str && p0 + cc < p) ? V[row * ldv + p0 + cc] : 0.0f;
        *reinterpret_cast<__bf16 *>(dst + cc * kVRow + 2 * i) = (__bf16)v;
    }
}

// Transposed values for the second product: bf16 V^T, tiled like the point copies with the value columns as rows and the
// streamed points as coordinates; zero outside the matrix.  A block: 64 columns x 32 points (one chunk); thread (column,
// piece of eight points).
__device__ __forceinline__ void transpose_values(const float *V, int64_t ldv, int64_t n_str, int p, int chunks, unsigned char *img)
{
    const int c = blockIdx.y * 64 + (threadIdx.x & 63), piece = threadIdx.x >> 6;
    const int64_t ch = blockIdx.x;
    uint32_t pk[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        __bf16 v[2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const int64_t i = ch * KC + piece * 8 + 2 * q + z;
            v[z] = (__bf16)((i < n_str && c < p) ? V[i * ldv + c] : 0.0f);
        }
        pk[q] = bf16_pair(v[0], v[1]);
    }
    const int64_t rb = c >> 4;
    *reinterpret_cast<uint4 *>(img + ((((rb >> 4) * chunks + ch) * 16 + (rb & 15)) << 10) + (c & 15) * 64 +
                               ((piece ^ ((c >> 2) & 3)) << 4)) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
}

// The stabiliser of a row of the plan slab: minus the base-2 exponent t its own potential contributes, rounded, so that
// exp2(score - rowmax) is 2^30 times the plan's entry without the row's weight, to a factor below sqrt(2).  Kept where a
// float holds it exactly; a row beyond that (a potential that masks it, for one) has sums that say so, see k_plan_finalize.
// Padding rows: no entry.  Also clears the flags of the rows to do again.
constexpr double kPlanShift = 30.0, kPlanLimit = 16777216.0;
struct RowmaxArgs {
    const double *pot, *norm;
    double inv_eps;
    int64_t cnt, cnt_pad;
    float *rowmax;
    int *flags, n_flags;
};
__device__ __forceinline__ void plan_rowmax(const RowmaxArgs &a, const int64_t i)
{
    if (i < a.n_flags) a.flags[i] = 0;
    if (i >= a.cnt_pad) return;
    double r = 3.0e38;
    if (i < a.cnt) {
        r = -rint((a.pot[i] - a.norm[i]) * a.inv_eps * kLog2e) - kPlanShift;
        r = r > kPlanLimit ? kPlanLimit : r < -kPlanLimit ? -kPlanLimit : r;   // (NaN stays)
    }
    a.rowmax[i] = (float)r;
}

// both in one launch: rows of blocks from `vt_rows` make the stabilisers
__global__ __launch_bounds__(256) void k_plan_prep(const float *V, int64_t ldv, int64_t n_str, int p, int chunks, unsigned char *img,
                                                   int vt_rows, RowmaxArgs rm)
{
    if ((int)blockIdx.y < vt_rows) {
        transpose_values(V, ldv, n_str, p, chunks, img);
        return;
    }
    const int64_t block = (int64_t)(blockIdx.y - vt_rows) * gridDim.x + blockIdx.x, blocks = (int64_t)(gridDim.y - vt_rows) * gridDim.x;
    for (int64_t i = block * 256 + threadIdx.x; i < rm.cnt_pad; i += blocks * 256) plan_rowmax(rm, i);
}

// out_i = w_i exp(fhat_i/eps) 2^rowmax_i (sum over the splits of the product), columns col0 .. col0 + cols; a block per row.
//
// Which rows that is good for is read off the row's sum of stored exponentials (mass_out and flags are given with the first
// columns only).  Within 2^-40 .. 2^60, that is a row mass of 2^-70 .. 2^30 times its weight, the entries that were rounded to
// zero are below 2^-126 each, 2^-62 of the sum for 2^24 points.  A row below that whose factor is below 2^-400 is zero
// in float, whatever the values: potentials of -inf or -1e30 that mask a row.  A sum that is not a number comes from such a
// score, and the row is NaN here as anywhere.  All other rows are flagged and done by k_apply_direct.
__global__ __launch_bounds__(256) void k_plan_finalize(const float *opart, int64_t ld, int splits, int slab_rows, int row_off, int64_t cnt,
                                                       double inv_eps, const float *w, double log_uniform, const double *pot,
                                                       const double *norm, const float *rowmax, int col0, int cols, float *out, int64_t ldo,
                                                       const double2 *partial, int64_t stride, int plan_splits, float *mass_out, int *flags)
{
    const int64_t i = row_off + (int64_t)blockIdx.x;
    if (i >= cnt) return;
    double S = 0.0;   // (asked for before the products: its latency is that of a block)
    if (flags && threadIdx.x < 64)
        for (int k = threadIdx.x; k < plan_splits; k += 64) S += partial[(int64_t)k * stride + i].y;
    const double lw = w ? log((double)w[i]) : log_uniform;
    const double e0 = ((pot[i] - norm[i]) * inv_eps + lw) * kLog2e + (double)rowmax[i];
    const double fac = exp2(e0);
    const float *o = opart + (int64_t)blockIdx.x * ld;
    for (int c = threadIdx.x; c < cols; c += 256) {
        double acc = 0.0;
        for (int k = 0; k < splits; ++k) acc += (double)o[(int64_t)k * slab_rows * ld + c];
        out[i * ldo + col0 + c] = (float)(fac * acc);
    }
    if (flags && threadIdx.x < 64) {
        if (plan_splits > 1)
            for (int off = 32; off > 0; off >>= 1) S += __shfl_xor(S, off);
        if (threadIdx.x == 0) {
            if (mass_out) mass_out[i] = (float)(fac * S);
            const bool kept = (S >= 0x1p-40 && S <= 0x1p60) || S != S || (S <= 0x1p60 && e0 < -400.0);
            if (!kept) flags[0] = flags[1 + i / 128] = 1;
        }
    }
}

// Number of splits of the streamed side that minimises  rounds x tiles-per-workgroup
// (rounds = ceil(workgroups / workgroups the chip holds at a time)), i.e. the time including the
// idle tail of the last round; prefer fewer, longer workgroups on near-ties.
int choose_splits(const Ctx *c, int n_jtiles, int n_itiles, int cap, int per_cu)
{
    int best_s = 1;
    double best_cost = 1e300;
    const int smax = n_itiles < cap ? n_itiles : cap;
    for (int sp = 1; sp <= smax; ++sp) {
        int tps = (int)ceil_div(n_itiles, sp);
        int seff = (int)ceil_div(n_itiles, tps);
        if (seff != sp) continue;
        double rounds = (double)ceil_div((int64_t)n_jtiles * seff, (int64_t)c->num_cu * per_cu);
        double cost = rounds * (tps + 0.25);   // 0.25: pipeline fill and merge of a workgroup
        if (cost < best_cost * 0.99) {
            best_cost = cost;
            best_s = sp;
        }
    }
    return best_s;
}

constexpr int kApplyPC = 64;    // value columns per application pass
constexpr int kApplyPCWide = 96;   // ... when there are more than 64 (every pass repeats the score contraction)
constexpr int kApplyBJ = 128;   // resident rows per workgroup of the application kernel

// ---- application through a stored slab of the plan -------------------------------------------------------------------
// The fused kernel takes 96 value columns per pass and repeats the contraction over d in every pass.  With many columns it
// is cheaper to form the exponentials once, store them in bf16 (which is what the fused kernel multiplies with as well) and
// run the second product as a matrix product of its own: slabs of resident rows, at most kSlabBytes of exponentials each
// (what the last-level cache holds; 128 MB measured 8 % slower, 512 MB 1 % faster for twice the memory).
// Measured at n = 40009, m = 30011, d = 784, 784 columns: 20.7 ms in nine fused passes, 4.4 ms here; of a slab of 4096 rows
// the exponentials take 212 us (0.93 PFLOP/s with the store of 247 MB), 768 columns of the product 161 us (1.18 PFLOP/s) and
// the last 16 columns 54 us, which is the time to read the slab once more.
constexpr size_t kSlabBytes = size_t(256) << 20;
// The whole workspace of this route (slab, accumulators, transposed values): beyond it the fused kernel runs, which needs a
// fraction of it.
constexpr size_t kSlabTotalBytes = size_t(1) << 30;

struct SlabPlan {
    int rows = 0;            // resident rows of a slab (multiple of 256)
    int e_chunks = 0;        // chunks of 32 streamed points
    int wide_tiles = 0;      // 256-column tiles of the product
    int rest = 0;            // columns beyond them, taken by a 128-column tile (0: none)
    int ks_wide = 0, ks_rest = 0;   // splits of the product's contraction
    int col_blocks = 0;             // column blocks of k_apply_direct
    size_t eslab = 0, vt = 0, rowmax = 0, flags = 0, opart = 0, total = 0;
};

int product_splits(const Ctx *c, int tiles, int chunks)
{
    // about one workgroup per CU, each with at least 32 chunks of the contraction
    int ks = c->num_cu / (tiles < 1 ? 1 : tiles);
    const int most = chunks / 32 < 1 ? 1 : chunks / 32;
    if (ks > most) ks = most;
    if (ks < 1) ks = 1;
    const int per = (int)ceil_div(chunks, ks);
    return (int)ceil_div(chunks, per);
}

SlabPlan slab_plan(const Ctx *c, int64_t n_res, int64_t n_str, int64_t p)
{
    SlabPlan s;
    s.e_chunks = (int)(round_up(n_str, BI) / KC);
    s.wide_tiles = (int)(p / 256);
    s.rest = (int)(p % 256);
    if (s.rest > 128) {
        ++s.wide_tiles;
        s.rest = 0;
    }
    // a row's exponentials and its accumulators for one split of the contraction (more splits are taken only where there are
    // so few rows that a tile per CU does not come together: 64 MB of accumulators at most)
    const size_t per_row = (size_t)s.e_chunks * KC * 2 + (size_t)(s.wide_tiles ? s.wide_tiles * 256 : 128) * 4;
    const int64_t most = (int64_t)(kSlabBytes / per_row) / 256 * 256;
    const int64_t all = round_up(n_res, 256);
    // (slabs of equal size)
    const int64_t cnt = most < 256 ? 0 : ceil_div(all, most);
    s.rows = cnt ? (int)round_up(ceil_div(all, cnt), 256) : 0;
    const int rt = s.rows / 256;
    s.ks_wide = s.wide_tiles ? product_splits(c, rt * s.wide_tiles, s.e_chunks) : 0;
    s.ks_rest = s.rest ? product_splits(c, rt, s.e_chunks) : 0;
    s.col_blocks = (int)ceil_div(p, kApplyPCWide);
    Arena A;
    s.eslab = A.take((size_t)s.rows * s.e_chunks * KC * 2);
    s.vt = A.take((size_t)round_up(p, 256) * s.e_chunks * KC * 2);
    s.rowmax = A.take((size_t)round_up(n_res, 1024) * 4);
    s.flags = A.take((size_t)(1 + ceil_div(n_res, kApplyBJ)) * 4);
    const size_t ow = (size_t)s.ks_wide * s.rows * s.wide_tiles * 256 * 4, orr = (size_t)s.ks_rest * s.rows * 128 * 4;
    s.opart = A.take(ow > orr ? ow : orr);
    s.total = A.off;
    return s;
}

// Which of the two: columns of contraction per pair, the fused kernel's at 0.8 of the rate of the two plain products, the
// store and the load of an exponential counted as kSlabTraffic columns.  At n = 20000, m = 15000 (us, fused / stored):
// d = 64, 128 columns 405 / 433; d = 128, 128 columns 536 / 425; d = 192, 192 columns 623 / 520; d = 96, 200 columns
// 655 / 533; d = 256, 256 columns 1020 / 554; d = 784, 100 columns 1357 / 772.
constexpr double kSlabTraffic = 230.0;
bool use_slab(const Ctx *c, int64_t n_res, int64_t n_str, int64_t d, int64_t p)
{
    if (p <= kApplyPCWide) return false;
    const SlabPlan plan = slab_plan(c, n_res, n_str, p);
    if (plan.rows < 256 || plan.total > kSlabTotalBytes) return false;
    const double fused = (double)ceil_div(p, kApplyPCWide) * (double)(round_up(d, KC) + kApplyPCWide);
    const int64_t rest = p % 256;
    const double cols = (double)(p / 256 * 256 + (rest == 0 ? 0 : rest > 128 ? 256 : 128));
    return (double)round_up(d, KC) + cols + kSlabTraffic < 1.25 * fused;
}

}  // namespace

// arguments of an LSE pass (res resident, str streamed) writing its records to `partial`; *blocks = its grid
static fs_status lse_pass_args(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, void *partial, BfArgs *out,
                               int *blocks)
{
    // (a 256 x 128 workgroup tile, two workgroups per CU, was measured slower and is not built)
    const int bj = 256, per_cu = 1;
    BfArgs a{};
    a.res = res->pts_b;
    a.str = str->pts_b;
    a.bias = str->bias_f;
    a.kp = P->kp;
    a.cscale = (float)(2.0 * kLog2e / eps);
    a.n_jtiles = (int)ceil_div(res->cnt, bj);
    a.n_itiles = (int)ceil_div(str->cnt, BI);
    a.splits = choose_splits(c, a.n_jtiles, a.n_itiles, max_splits(c->partial_budget, res->cnt), per_cu);
    a.tiles_per_split = (int)ceil_div(a.n_itiles, a.splits);
    const int total = a.n_jtiles * a.splits;
    a.partial = (double2 *)partial;
    a.partial_stride = res->cnt_pad;
    if ((int64_t)a.n_jtiles * bj > res->cnt_pad || (int64_t)a.n_itiles * BI > str->cnt_pad ||
        (size_t)a.splits * res->cnt_pad * 16 > P->partial_bytes || (a.kp & 31) != 0 || a.kp < 32)
        return fail(c, FS_ERR_DEVICE, "internal: bf16 launch shape exceeds the padded buffers");
    *out = a;
    *blocks = (total + 7) / 8 * 8;
    return FS_OK;
}

fs_status bf16_lse(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, Splits *splits_out)
{
    BfArgs a;
    int blocks = 0;
    fs_status st = lse_pass_args(c, P, res, str, eps, P->partial, &a, &blocks);
    if (st != FS_OK) return st;
    // the coordinates end in the first 16 of a tile's last chunk (d = 784 = 49 x 16): the kernel copy that leaves
    // out that chunk's second, all-zero k-step (2 % of the MFMAs at d = 784)
    const bool half = (P->d % 32) >= 1 && (P->d % 32) <= 16 && a.kp >= 64;
    prof_begin(c, (double)res->cnt * (double)str->cnt);
    if (half)
        hipLaunchKernelGGL((k_lse_bf16<2, 4, 4, 0, true>), dim3((unsigned)blocks), dim3(512), 0, c->stream, a);
    else
        hipLaunchKernelGGL((k_lse_bf16<2, 4, 4, 0>), dim3((unsigned)blocks), dim3(512), 0, c->stream, a);
    prof_end(c);
    FS_HIP(c, hipGetLastError());
    *splits_out = a.splits;
    return FS_OK;
}

// The f-pass (records to partial_x) and the g-pass (records to partial_y) of one iteration of the averaged
// schedule (Eq. 4-5) in ONE launch.
fs_status bf16_lse_pair(Ctx *c, const Prepared *P, double eps, void *partial_x, void *partial_y, Splits *splits_x, Splits *splits_y)
{
    BfArgs ax, ay;
    int bx = 0, by = 0;
    fs_status st;
    if ((st = lse_pass_args(c, P, &P->X, &P->Y, eps, partial_x, &ax, &bx)) != FS_OK) return st;
    if ((st = lse_pass_args(c, P, &P->Y, &P->X, eps, partial_y, &ay, &by)) != FS_OK) return st;
    if (bx + by <= 4 * c->num_cu) {
        prof_begin(c, 2.0 * (double)P->X.cnt * (double)P->Y.cnt);
        hipLaunchKernelGGL((k_lse_bf16_pair<2, 4, 4>), dim3((unsigned)(bx + by)), dim3(512), 0, c->stream, ax, ay, bx);
        prof_end(c);
    } else {
        // many rounds of workgroups: one launch saves nothing there, and two passes of different shape in one
        // grid share the L2 of an XCD worse than one after the other (n = 50000, m = 20000, d = 1024: 4 % slower)
        prof_begin(c, (double)P->X.cnt * (double)P->Y.cnt);
        hipLaunchKernelGGL((k_lse_bf16<2, 4, 4, 0>), dim3((unsigned)bx), dim3(512), 0, c->stream, ax);
        prof_end(c);
        prof_begin(c, (double)P->X.cnt * (double)P->Y.cnt);
        hipLaunchKernelGGL((k_lse_bf16<2, 4, 4, 0>), dim3((unsigned)by), dim3(512), 0, c->stream, ay);
        prof_end(c);
    }
    FS_HIP(c, hipGetLastError());
    *splits_x = ax.splits;
    *splits_y = ay.splits;
    return FS_OK;
}

static fs_status slab_apply(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, const float *V, int64_t p, int64_t ldv,
                            float *out, int64_t ldo, float *mass_out)
{
    const SlabPlan sp = slab_plan(c, res->cnt, str->cnt, p);
    char *x = P->extra;
    if (!x || sp.total > P->extra_bytes || sp.rows < 256) return fail(c, FS_ERR_DEVICE, "internal: plan slab exceeds its buffer");
    float *rowmax = reinterpret_cast<float *>(x + sp.rowmax), *opart = reinterpret_cast<float *>(x + sp.opart);
    unsigned char *vt = reinterpret_cast<unsigned char *>(x + sp.vt);
    int *flags = reinterpret_cast<int *>(x + sp.flags);
    const int n_jtiles = (int)ceil_div(res->cnt, kApplyBJ);
    // (fewer flags than padded rows)
    const RowmaxArgs rm{res->pot, res->norm, 1.0 / eps, res->cnt, res->cnt_pad, rowmax, flags, 1 + n_jtiles};
    const int vt_rows = (sp.wide_tiles * 256 + (sp.rest ? 128 : 0)) / 64;
    int64_t rm_rows = ceil_div(res->cnt_pad, (int64_t)sp.e_chunks * 256);   // (a row per thread, up to 1024 rows of blocks)
    if (rm_rows > 1024) rm_rows = 1024;
    hipLaunchKernelGGL(k_plan_prep, dim3((unsigned)sp.e_chunks, (unsigned)(vt_rows + rm_rows)), dim3(256), 0, c->stream, V, ldv, str->cnt,
                       (int)p, sp.e_chunks, vt, vt_rows, rm);
    const int n_itiles = (int)ceil_div(str->cnt, BI);
    const int64_t all = round_up(res->cnt, 256);
    for (int64_t off = 0; off < all; off += sp.rows) {
        const int rows = (int)(all - off < sp.rows ? all - off : sp.rows), rt = rows / 256;
        // the exponentials of the slab
        BfArgs a{};
        a.res = res->pts_b;
        a.str = str->pts_b;
        a.bias = str->bias_f;
        a.kp = P->kp;
        a.cscale = (float)(2.0 * kLog2e / eps);
        a.n_jtiles = rt;
        a.n_itiles = n_itiles;
        a.splits = choose_splits(c, rt, n_itiles, max_splits(c->partial_budget, res->cnt), 1);
        a.tiles_per_split = (int)ceil_div(n_itiles, a.splits);
        a.partial = (double2 *)P->partial;
        a.partial_stride = res->cnt_pad;
        a.rowmax = rowmax;
        a.eslab = reinterpret_cast<unsigned char *>(x + sp.eslab);
        a.e_chunks = sp.e_chunks;
        a.row_off = (int)off;
        if (off + rows > res->cnt_pad || (int64_t)n_itiles * BI > str->cnt_pad || n_itiles * (BI / KC) != sp.e_chunks ||
            (size_t)a.splits * res->cnt_pad * 16 > P->partial_bytes || (a.kp & 31) != 0 || a.kp < 32)
            return fail(c, FS_ERR_DEVICE, "internal: plan slab launch shape exceeds the padded buffers");
        const bool half = (P->d % 32) >= 1 && (P->d % 32) <= 16 && a.kp >= 64;   // (as in bf16_lse)
        const dim3 grid((unsigned)round_up(rt * a.splits, 8));
        if (half)
            hipLaunchKernelGGL((k_lse_bf16<2, 4, 4, 0, true, Epi::Plan>), grid, dim3(512), 0, c->stream, a);
        else
            hipLaunchKernelGGL((k_lse_bf16<2, 4, 4, 0, false, Epi::Plan>), grid, dim3(512), 0, c->stream, a);
        // times the values: the 256-column tiles, then the rest
        for (int part = 0; part < 2; ++part) {
            const int tiles = part ? (sp.rest ? 1 : 0) : sp.wide_tiles, ks = part ? sp.ks_rest : sp.ks_wide;
            if (!tiles) continue;
            const int col0 = part ? sp.wide_tiles * 256 : 0;
            const int cols = (int)(part ? sp.rest : (p < (int64_t)tiles * 256 ? p : (int64_t)tiles * 256));
            BfArgs b{};
            b.str = reinterpret_cast<const uint16_t *>(x + sp.eslab);
            b.res = reinterpret_cast<const uint16_t *>(vt + (size_t)sp.wide_tiles * part * 256 * sp.e_chunks * KC * 2);
            b.n_jtiles = tiles;
            b.n_itiles = rt;
            b.splits = rt * ks;
            b.e_chunks = sp.e_chunks;
            b.ch_per_split = (int)ceil_div(sp.e_chunks, ks);
            b.out_rows = rows;
            b.opart = opart;
            b.opart_ld = part ? 128 : tiles * 256;
            const dim3 g2((unsigned)round_up(tiles * b.splits, 8));
            if (part)
                hipLaunchKernelGGL((k_lse_bf16<2, 4, 2, 0, false, Epi::Product>), g2, dim3(512), 0, c->stream, b);
            else
                hipLaunchKernelGGL((k_lse_bf16<2, 4, 4, 0, false, Epi::Product>), g2, dim3(512), 0, c->stream, b);
            hipLaunchKernelGGL(k_plan_finalize, dim3((unsigned)rows), dim3(256), 0, c->stream, opart, b.opart_ld, ks, rows, (int)off, res->cnt,
                               1.0 / eps, res->w, res->log_uniform, res->pot, res->norm, rowmax, col0, cols, out, ldo,
                               (const double2 *)P->partial, res->cnt_pad, a.splits, mass_out, (part == 0 || !sp.wide_tiles) ? flags : nullptr);
        }
        FS_HIP(c, hipGetLastError());
    }
    // rows that the stored slab is not good for (a launch that leaves at once where there are none)
    {
        constexpr int pc = kApplyPCWide;
        BfArgs a{};
        a.res = res->pts_b;
        a.str = str->pts_b;
        a.bias = str->bias_f;
        a.kp = P->kp;
        a.cscale = (float)(2.0 * kLog2e / eps);
        a.n_jtiles = n_jtiles;
        a.n_itiles = n_itiles;
        a.splits = 1;
        a.tiles_per_split = n_itiles;
        a.partial_stride = res->cnt_pad;
        const DirectArgs o{flags, res->cnt, 1.0 / eps, res->w, res->log_uniform, res->pot, res->norm, (int)p, out, ldo, mass_out,
                           V, ldv, str->cnt, sp.col_blocks};
        const int per_tile = n_jtiles >= 512 ? 1 : 512 / n_jtiles;

        if ((int64_t)n_jtiles * kApplyBJ > res->cnt_pad) return fail(c, FS_ERR_DEVICE, "internal: bf16 apply launch shape exceeds the padded buffers");
        hipLaunchKernelGGL((k_apply_direct<pc>), dim3((unsigned)n_jtiles, (unsigned)(sp.col_blocks < per_tile ? sp.col_blocks : per_tile)),
                           dim3(512), 0, c->stream, a, o);
        FS_HIP(c, hipGetLastError());
    }
    return FS_OK;
}

// workspace of bf16_apply: [splits][rows][kApplyPC] float accumulators, then the value images (fused kernel), or what the
// stored slab takes; *least: what the call can do with
size_t bf16_apply_ws(const Ctx *c, int64_t n_res, int64_t n_str, int64_t d, int64_t p, size_t *least)
{
    const int n_jtiles = (int)ceil_div(n_res, kApplyBJ), n_itiles = (int)ceil_div(n_str, BI);
    const int splits = choose_splits(c, n_jtiles, n_itiles, max_splits(c->partial_budget, n_res), 1);
    const size_t opart = (size_t)splits * (size_t)round_up(n_res, 1024) * kApplyPCWide * 4;
    *least = ((opart + 1023) & ~size_t(1023)) + (size_t)n_itiles * kVImgBytes(kApplyPCWide);
    return use_slab(c, n_res, n_str, d, p) ? slab_plan(c, n_res, n_str, p).total : *least;
}

fs_status bf16_apply(Ctx *c, const Prepared *P, const Side *res, const Side *str, double eps, const float *V, int64_t p,
                     int64_t ldv, float *out, int64_t ldo, float *mass_out)
{
    if (use_slab(c, res->cnt, str->cnt, P->d, p) && slab_plan(c, res->cnt, str->cnt, p).total <= P->extra_bytes)
        return slab_apply(c, P, res, str, eps, V, p, ldv, out, ldo, mass_out);
    BfArgs a{};
    a.res = res->pts_b;
    a.str = str->pts_b;
    a.bias = str->bias_f;
    a.kp = P->kp;
    a.cscale = (float)(2.0 * kLog2e / eps);
    a.n_jtiles = (int)ceil_div(res->cnt, kApplyBJ);
    a.n_itiles = (int)ceil_div(str->cnt, BI);
    a.splits = choose_splits(c, a.n_jtiles, a.n_itiles, max_splits(c->partial_budget, res->cnt), 1);
    a.tiles_per_split = (int)ceil_div(a.n_itiles, a.splits);
    a.partial = (double2 *)P->partial;
    a.partial_stride = res->cnt_pad;
    // 96 columns per pass when there are more than 64 (the registers allow three 32-column accumulator blocks), 64 else
    const int pc = p > kApplyPC ? kApplyPCWide : kApplyPC;
    const size_t opart_bytes = ((size_t)a.splits * res->cnt_pad * pc * 4 + 1023) & ~size_t(1023);
    const size_t vimg_bytes = (size_t)a.n_itiles * kVImgBytes(pc);
    a.opart = reinterpret_cast<float *>(P->extra);
    unsigned char *vimg = reinterpret_cast<unsigned char *>(P->extra) + opart_bytes;
    a.vimg = vimg;
    // host-side shape checks: every access of the kernels stays inside the padded buffers
    if ((int64_t)a.n_jtiles * kApplyBJ > res->cnt_pad || (int64_t)a.n_itiles * BI > str->cnt_pad ||
        (size_t)a.splits * res->cnt_pad * 16 > P->partial_bytes || (a.kp & 31) != 0 || a.kp < 32 ||
        opart_bytes + vimg_bytes > P->extra_bytes || !P->extra)
        return fail(c, FS_ERR_DEVICE, "internal: bf16 apply launch shape exceeds the padded buffers");
    const int total = a.n_jtiles * a.splits;
    const int per = (total + 7) / 8;
    for (int p0 = 0; p0 < p; p0 += pc) {
        hipLaunchKernelGGL(k_vimg_bf16, dim3((unsigned)a.n_itiles), dim3(BI), 0, c->stream, V, ldv, str->cnt, p0, (int)p, pc,
                           kVImgBytes(pc), vimg);
        if (pc == kApplyPCWide)
            hipLaunchKernelGGL((k_lse_bf16<2, 4, 2, kApplyPCWide>), dim3((unsigned)(per * 8)), dim3(512), 0, c->stream, a);
        else
            hipLaunchKernelGGL((k_lse_bf16<2, 4, 2, kApplyPC>), dim3((unsigned)(per * 8)), dim3(512), 0, c->stream, a);
        FS_HIP(c, hipGetLastError());
        fs_status st = launch_apply_finalize(c, P, res, res->norm, a.splits, eps, a.opart, pc, p0, (int)p, out, ldo, mass_out);
        if (st != FS_OK) return st;
    }
    return FS_OK;
}

}  // namespace fs
