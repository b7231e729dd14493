// Tiled kernel: one workgroup of W wavefronts per conditional, the augmented
// block held in registers as 16x16 tiles, the Cholesky blocked by tile
// columns with its trailing updates on FP64 matrix cores and its triangular
// solves by substitution.
//
// Block layout (same augmented block as the unblocked kernel): rows 0..k-1
// neighbours, row k the point itself, row k+1 the observations, rows k+2..
// 16T-1 identity padding.  Factoring rows 0..k gives L_kk^2 = c_i and, in row
// k+1, the two forward solves of Algorithm 1 (POTRF + 2 TRSV, fused).
//
// Register tiles.  v_mfma_f64_16x16x4f64 leaves D[4r + l/16][l%16] in
// accumulator register r of lane l, and every tile M of the block is kept in
// that layout ("N-layout"): lane (g, n) = (l/16, l%16), register r holds
// M[4r + g][n].  The transposed form ("T-layout", register r of lane (g, j)
// holding M[j][4r + g]) is the one panel tiles take in LDS, because as
// either MFMA operand a T-layout tile X enters a product directly:
//   SYRK   A_RC -= X_R X_C^T   operands -X_R and X_C, register s of each,
//                              accumulating straight into the N-layout tile.
//
// Per tile column t:
//   1. the owner of the diagonal tile factors it in its registers, four
//      columns at a time (one row per lane, 64-bit DPP row broadcasts, then a
//      rank-4 update on the matrix core), and publishes the substitution
//      weights -L[j][c] / L[c][c] and the inverse pivots;
//   2. the owners of the tiles below solve X L_tt^T = A in registers by
//      forward substitution over the 16 columns (column c of an N-layout
//      tile lives in lane c of every 16-lane row, so each step is one DPP
//      broadcast FMA per register), and publish X to LDS in T-layout;
//   3. the owners of the trailing tiles subtract X_R X_C^T (4 MFMAs per
//      tile), in the order of their slots: column t + 1, the next diagonal
//      tile with it, comes last, and the other waves wait for its
//      factorisation.
// Gradient: back substitution with L^T by columns of tiles: the sums of
// L_Rt^T x_R over the tiles below diagonal tile t on the vector units (every
// wave its own tiles), then x_t by substitution (one wave).  No step
// multiplies by an explicit inverse, so every solve is backward stable, as in
// the unblocked kernel.
#pragma once

#include <type_traits>

#include "device_common.h"
#include "kernel_lds.h"

namespace vecchia {

typedef double dvec4 __attribute__((ext_vector_type(4)));

#ifndef VECCHIA_KEEP_DBETA
#define VECCHIA_KEEP_DBETA 1
#endif

__host__ __device__ constexpr int tile_count(int T) { return T * (T + 1) / 2; }
__host__ __device__ constexpr int tiles_per_wave(int T, int W) { return (tile_count(T) + W - 1) / W; }

// LDS layout of the tiled kernel, in doubles.  The great-circle codes add
// cos(latitude) of every row, the power exponential a table of the logarithm.
//
// CUR[t % NPAR] receives the substitution weights of diagonal tile t
// (row-major, row stride 17) and, after that block, its 16 inverse pivots.
// With several waves the buffer alternates by the parity of t: the one tile
// t + 1 is published into served column t - 1, whose readers all passed a
// workgroup barrier since.  One array of T slots (DS doubles each) serves both
// the panel and, with the gradient, the factored diagonal tiles: while column
// t is processed, slot R > t holds the panel tile X_R (T-layout, lane-major),
// and slot t' <= t holds factor t' in the CUR format, copied there once every
// reader of X_t' has passed a barrier.
//
// A workgroup that evaluates G parameter vectors of one conditional in
// lockstep keeps G copies of everything that depends on the parameters (CUR,
// SLOT, YP, UB, SCAL, RED); the gathered coordinates, observations and the
// exponential table are shared.  G = 1 is the one-vector layout.  With one
// wavefront per vector (INPLACE, also for G = 1) there is no CUR: the
// wavefront publishes factor t + 1 into slot t + 1 once its trailing updates
// have read X_(t+1) there.
template <int T, int W, bool GRAD, bool GCD = false, int G = 1, bool POWEXP = false>
struct TileLds {
    static constexpr int KP = 16 * T;
    static constexpr int DS = 288;                        // a 16 x 17 tile, then 16 inverse pivots
    static constexpr bool INPLACE = W == 1;
    static constexpr int NPAR = (W > 1 && T > 1) ? 2 : 1;
    static constexpr int CUR = 0;                         // [G][NPAR][DS]  diagonal tile / its factor
    static constexpr int SLOT = CUR + (INPLACE ? 0 : G * NPAR * DS);  // [G][T][DS] panel tiles / factors
    static constexpr int XY = SLOT + G * T * DS;          // [KP][2]        coordinates
    static constexpr int ZV = XY + 2 * KP;                // [KP]           observations
    static constexpr int YP = ZV + KP;                    // [G][KP]        factor row k+1
    static constexpr int UB = YP + G * KP;                // [G][KP][2]     back-substitution solutions (u, b), gradient
    static constexpr int SCAL = UB + (GRAD ? G * 2 * KP : 0);  // [G][16]   scalars: [0] L_kk, [1] 1 / L_kk
    static constexpr int RED = SCAL + G * 16;             // [G][2][4W]     reductions (two values, W waves x 4 rows)
    static constexpr int CL = RED + G * 8 * W;            // [KP]           cos(latitude) (great-circle codes only)
    static constexpr int EXPT = CL + (GCD ? KP : 0);      //                staged tables (stage_tables)
    static constexpr int TOTAL = EXPT + staged_doubles(POWEXP);
    static constexpr size_t BYTES = (size_t)TOTAL * sizeof(double);
    // per-parameter-vector strides
    static constexpr int CUR_G = NPAR * DS, SLOT_G = T * DS, YP_G = KP, QUB_G = 2 * KP, SCAL_G = 16, RED_G = 8 * W;
};

// TileLds<T, W, grad, gcd, G, powexp>::TOTAL, for the occupancy estimate.
__host__ __device__ constexpr int tile_lds_doubles(int T, int W, bool grad, bool gcd, int G = 1, bool powexp = false) {
    return (W == 1 ? 0 : G * ((W > 1 && T > 1) ? 2 : 1) * 288) + G * T * 288 +
           16 * T * (3 + G * (1 + (grad ? 2 : 0)) + (gcd ? 1 : 0)) + G * (16 + 8 * W) + staged_doubles(powexp);
}
static_assert(TileLds<8, 4, true, false>::TOTAL == tile_lds_doubles(8, 4, true, false), "LDS estimate out of date");
static_assert(TileLds<3, 1, false, true>::TOTAL == tile_lds_doubles(3, 1, false, true), "LDS estimate out of date");
static_assert(TileLds<4, 1, true, true, 4, true>::TOTAL == tile_lds_doubles(4, 1, true, true, 4, true),
              "LDS estimate out of date");
static_assert(TileLds<5, 2, false, false, 2>::TOTAL == tile_lds_doubles(5, 2, false, false, 2), "LDS estimate out of date");

// Parameter vectors a workgroup evaluates in lockstep, per shape: four for
// the one-wavefront shapes (up to five tile rows: six rows make 21 tiles,
// past the 20 one wavefront holds), where the four wavefronts share the
// gathered neighbours and the pair distances; other shapes keep one vector
// (G = 1).
// Only these group sizes are compiled.
__host__ __device__ constexpr int lockstep_group(int T, int W) { return (T <= 5 && W == 1) ? 4 : 1; }

// Shapes measured faster with one more workgroup per CU than the register
// estimate below allows, at the price of a small spill:
//   T = 8, W = 4 (m from 110 to 125): value + gradient 67.0 ms at four
//     workgroups (9-11 VGPRs spilled) against 79.3 ms at three for the
//     10^6-point, m = 120 field; a fifth workgroup (102 VGPRs) spilled more
//     and took 91 ms;
//   T = 10, W = 4 (m from 142 to 157): 32.5 ms at three workgroups against
//     41.7 ms at two (34.1 ms at four) for 250,000 uniform points, m = 150,
//     nu = 3/2, value + gradient;
//   T = 4, W = 2 (m from 47 to 62; LDS leaves room only without the
//     gradient): 2.82 ms at nine workgroups against 2.89 ms at eight for the
//     same points at m = 60, value only.
//   T = 8, W = 4, great circle: power exponential value + gradient 3.67 ms at four
//     workgroups (two registers spilled) against 4.28 ms at three (129 VGPRs),
//     Matern 3/2 3.09 against 3.63 ms, for 40,000 points, m = 124;
//   T = 11, W = 4, great circle (m of 159 and 160): Matern 3/2 value + gradient
//     3.91 ms at three workgroups against 4.65 ms at two, power exponential
//     4.48 against 5.52 ms, for 20,000 points.
// (Times and spills of the first two from before the covariances and the
// contraction became leaner: T = 8 now fits at 125 VGPRs and T = 10 at 166,
// without scratch.)
// T = 7 and 9 with W = 4, T = 2 to 4 with W = 1 and T = 3, 5, 6 with W = 2
// measured no faster one workgroup up.  Other shapes keep the estimate.
__host__ __device__ constexpr bool tile_measured_raise(int T, int W, bool gcd) {
    return (T == 8 && W == 4) || (T == 10 && W == 4 && !gcd) || (T == 4 && W == 2 && !gcd) || (T == 11 && W == 4 && gcd);
}

// Occupancy target (wavefronts per SIMD) the register allocation aims at.
// Workgroups per CU are limited by LDS and by registers: each lane holds 8
// VGPRs per tile (16 when the beta-derivative tiles are kept) plus about 72
// for the diagonal factorisation, the covariance code and addressing (the
// compiler reports 143 VGPRs for T = 8, W = 4 with the gradient, nine tiles).
// A lockstep workgroup (G parameter vectors) has G W wavefronts.
__host__ __device__ constexpr int tile_waves_per_simd(int T, int W, bool keep_d, bool grad, bool gcd, int G,
                                                      bool powexp) {
    const int lds = tile_lds_doubles(T, W, grad, gcd, G, powexp) * 8;
    const int blocks_lds = 163840 / lds;
    const int need = 8 * tiles_per_wave(T, W) * (keep_d ? 2 : 1) + 72 + (gcd ? 16 : 0);
    const int wps_regs = 512 / need;                 // wavefronts per SIMD the registers allow
    const int blocks_regs = (wps_regs * 4) / (W * G);  // workgroups per CU the registers allow
    int blocks = blocks_lds < blocks_regs ? blocks_lds : blocks_regs;
    if (blocks < 1) blocks = 1;
    if (G == 1 && !keep_d && tile_measured_raise(T, W, gcd) && blocks + 1 <= blocks_lds) blocks += 1;
    int wps = (blocks * W * G + 3) / 4;
    if (wps < 1) wps = 1;
    if (wps > 8) wps = 8;
    return wps;
}

// Whether the gradient keeps the beta-derivative tiles in registers (one
// covariance evaluation per entry) or recomputes them after the solves.  For
// the Matern codes on Euclidean distances an evaluation is about 36 issue
// slots, and the tiles are kept only when the extra registers cost no
// occupancy.  The great-circle codes spend about 100 to 130 (two sines, a root
// and a series, for the power exponential a logarithm and an exponential):
// there one-wavefront shapes keep the tiles whenever two wavefronts per SIMD
// still fit (measured, power exponential, 100,000 points, m = 60: 2.17 ms
// keeping at two wavefronts per SIMD, 2.56 recomputing at three; with four
// wavefronts per conditional, m = 120, 50,000 points, keeping lost: 5.74
// against 4.64 ms).  The one-wavefront shape of three tile rows always keeps
// them, which on Euclidean distances concerns the power exponential (m = 44,
// 40,000 points: 0.381 ms keeping with 24 registers spilled, 0.454 recomputing).
// Lockstep workgroups follow the one-vector decision: the two ways round the
// derivative contract their arithmetic differently, and the lockstep results
// must be the one-vector bits.
__host__ __device__ constexpr bool keep_dbeta(int T, int W, bool gcd, bool powexp) {
    const int kept = tile_waves_per_simd(T, W, true, true, gcd, 1, powexp);
    return VECCHIA_KEEP_DBETA && (kept >= tile_waves_per_simd(T, W, false, true, gcd, 1, powexp) ||
                                  (gcd && W == 1 && kept >= 2) || (T == 3 && W == 1));
}

// Tile enumeration: column C descending, row R ascending inside a column, so
// the tiles still active after step t form a prefix and a round-robin owner
// assignment balances every step.  Slot s of wavefront w holds tile w + W s;
// its (R, C) is byte s of the wavefront's row of the map, R in the high four
// bits.  Slots past the last tile read as (0, 15), a column no step reaches.
template <int T, int W>
struct TileMap {
    static constexpr int WORDS = (tiles_per_wave(T, W) + 3) / 4;
    uint32_t word[W][WORDS];
    constexpr TileMap() : word{} {
        for (int w = 0; w < W; ++w)
            for (int q = 0; q < WORDS; ++q) word[w][q] = 0x0F0F0F0Fu;
        int idx = 0;
        for (int c = T - 1; c >= 0; --c)
            for (int r = c; r < T; ++r, ++idx) {
                const int sh = 8 * ((idx / W) % 4);
                uint32_t &x = word[idx % W][idx / W / 4];
                x = (x & ~(0xFFu << sh)) | ((uint32_t)(r * 16 + c) << sh);
            }
    }
};
template <int T, int W>
__device__ constexpr TileMap<T, W> kTileMap = TileMap<T, W>();

__device__ inline int tile_index(int T, int R, int C) {
    // tiles of columns T-1 .. C+1 come first
    const int before = (T - 1 - C) * (T - C) / 2;
    return before + (R - C);
}

template <int SRC>
__device__ __forceinline__ double bcast_row(double v) {
    // every lane of each 16-lane row receives lane SRC of that row (64-bit DPP row_newbcast)
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + SRC, 0xF, 0xF, false);
}

// acc -= v(lane SRC of this lane's row) * w, one fused 64-bit DPP FMA with a
// negated operand.  With NOP, two wait states precede it: a DPP source
// written by the instruction just before needs them, and the compiler does
// not look inside inline assembly for that hazard.
template <int SRC, bool NOP>
__device__ __forceinline__ void fms_bcast_row(double &acc, double v, double w) {
    if constexpr (NOP)
        asm volatile("s_nop 1\n\tv_fmac_f64_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                     : "+v"(acc)
                     : "v"(v), "v"(w), "i"(SRC));
    else
        asm volatile("v_fmac_f64_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                     : "+v"(acc)
                     : "v"(v), "v"(w), "i"(SRC));
}

// acc += acc(lane SRC of this lane's row) * w: the accumulator is also the
// broadcast source (one register, no copy).
template <int SRC, bool NOP>
__device__ __forceinline__ void fma_bcast_row_self(double &acc, double w) {
    if constexpr (NOP)
        asm volatile("s_nop 1\n\tv_fmac_f64_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
                     : "+v"(acc)
                     : "v"(w), "i"(SRC));
    else
        asm volatile("v_fmac_f64_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
                     : "+v"(acc)
                     : "v"(w), "i"(SRC));
}

// compile-time loop: f(std::integral_constant<int, I>) for I = B .. E-1
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// f(B), f(B + S), .. up to but excluding E: with UNROLL as compile-time
// constants, else as ints in a loop that stays rolled.
template <bool UNROLL, int B, int E, int S, class F>
__device__ __forceinline__ void for_columns(F &&f) {
    if constexpr (!UNROLL) {
#pragma unroll 1
        for (int t = B; t != E; t += S) f(t);
    } else if constexpr (B != E) {
        f(std::integral_constant<int, B>{});
        for_columns<true, B + S, E, S>(f);
    }
}

// 1/sqrt(x) for x > 0: the hardware estimate y (relative error near 2^-24)
// and one third-order correction y (1 + e/2 + 3e^2/8), e = 1 - x y^2.  The
// residual e is formed without rounding loss (x y split into h + hl), so
// the result is within about half an ulp; five dependent steps where two
// Newton steps take six.
__device__ __forceinline__ double rsqrt_refined(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double h = x * y;
    const double hl = fma(x, y, -h);  // x y = h + hl exactly
    const double e = fma(-hl, y, fma(-h, y, 1.0));
    const double p = fma(e, 0.375, 0.5);
    return fma(y * e, p, y);
}

// 64-bit DPP move of both halves of a double (any DPP control).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the 16 lanes of each row by DPP (pairs, quads, half rows, rows);
// every lane of the row ends with the same bits.
__device__ __forceinline__ double row_sum16(double v) {
    v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);  // row_half_mirror
    v += dpp_f64<0x140>(v);  // row_mirror
    return v;
}

// The value of v in one lane, uniform over the wavefront.
__device__ __forceinline__ double read_lane(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Entry (a, b) of the augmented block for rows or columns past k, given the
// covariance entry v (nugget included): the observation row k+1 holds z of
// the other index, the padding beyond it is the identity.  The diagonal of
// row k+1 is never used as a result; 2^600 keeps its pivot positive (it
// exceeds the squared norm of the row by far for any finite data), so the
// factorisation needs no special case for it.
__device__ __forceinline__ double augment_value(int a, int b, int k, double v, const double *__restrict__ Z) {
    const int hi = a > b ? a : b, lo = a > b ? b : a;
    if (hi == k + 1) v = (lo == k + 1) ? 0x1p600 : Z[lo];
    if (hi > k + 1) v = (a == b) ? 1.0 : 0.0;
    return v;
}

// Writes an N-layout tile to a panel slot in T-layout, lane-major: the reader
// lane (g', j) finds M[j][4r' + g'] at slot[(16 g' + j) 4 + r'].  Element
// (4r + g, n) of this lane goes to reader lane (n % 4, 4r + g), register n / 4.
__device__ __forceinline__ void store_panel_tlayout(const dvec4 &v, double *slot) {
    const int l = threadIdx.x % kWave, g = l / 16, n = l % 16;
#pragma unroll
    for (int r = 0; r < 4; ++r) slot[(16 * (n % 4) + 4 * r + g) * 4 + n / 4] = v[r];
}

// The values of x in the four 16-lane row groups, each copied to every row
// group: o[r] in lane (g, j) is x of lane (r, j).
__device__ __forceinline__ void row_groups(double x, double (&o)[4]) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const unsigned int lo = (unsigned int)__double2loint(x), hi = (unsigned int)__double2hiint(x);
    // 32-lane halves, then the two 16-lane rows of each half
    const u32x2 l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const u32x2 h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    const u32x2 l01 = __builtin_amdgcn_permlane16_swap(l[0], l[0], false, false);
    const u32x2 h01 = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
    const u32x2 l23 = __builtin_amdgcn_permlane16_swap(l[1], l[1], false, false);
    const u32x2 h23 = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
    o[0] = __hiloint2double((int)h01[0], (int)l01[0]);
    o[1] = __hiloint2double((int)h01[1], (int)l01[1]);
    o[2] = __hiloint2double((int)h23[0], (int)l23[0]);
    o[3] = __hiloint2double((int)h23[1], (int)l23[1]);
}

// Sums of x and of y over the four row groups: row groups 0 and 1 end with
// the sum of x, row groups 2 and 3 with the sum of y.
__device__ __forceinline__ double sum_row_groups2(double x, double y) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    u32x2 l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
    u32x2 h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
    x = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(x), false, false);
    h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(x), false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}

// acc - a b over one 16 x 4 by 4 x 16 product (the matrix core negates its
// first operand).
__device__ __forceinline__ dvec4 mfma_sub(double a, double b, const dvec4 &acc) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 1);
}

// Factors diagonal tile t, held by the calling wave in N-layout registers
// (the whole symmetric tile), four columns at a time, and publishes to D the
// substitution weights W[j][c] = -L[j][c] / L[c][c] of the strictly lower part
// (row-major, stride 17, zeros elsewhere) and the inverse pivots D[272 + c].
// Records L_kk, its inverse and the part of factor row k+1 that falls in this
// tile.
//
// Column block b (columns 4b .. 4b + 3): by symmetry rows 4b .. 4b + 3 of the
// tile, register b, are its columns, so row-group copies of that register
// give every lane j row j of the block.  The four columns are factored one
// row per lane (DPP row broadcasts), the four row groups alike; each row
// group g then selects column 4b + g, which is register b of the factor in
// T-layout and both operands of the rank-4 update of the tile on the matrix
// core.  Rows above the block hold rounding residue that nothing reads.
// (One row per lane over all 16 columns, 120 broadcast FMAs and 16 row
// registers, took 663 vector instructions per tile; this takes about 300 and
// a dependency chain half as long.)
//
// Every row is factored: the padding rows have pivot 1 and the observation
// row's diagonal is 2^600 (augment_value), so their pivots are positive and
// nothing past row k reaches rows up to k.  A pivot that is not positive and
// finite turns L_kk, and with it the conditional's value, into NaN, which the
// caller reports.
__device__ __forceinline__ void factor_diag(dvec4 A, int t, int k, double *D, double *scal, double *yp) {
    int l = threadIdx.x % kWave;
    asm volatile("" : "+v"(l));  // keep the lane masks below inside the tile loop (no hoisting)
    const int g = l / 16, j = l % 16;
    const bool g1 = (g & 1) != 0, g2 = (g & 2) != 0;
    const int base = 16 * t;
    const bool has_k = (k >> 4) == t, has_y = ((k + 1) >> 4) == t;  // rows k and k + 1 lie in this tile
    const int jk = k - base, jy = k + 1 - base;
    // this wave is the critical path of the workgroup: let it win instruction
    // issue over the other waves sharing its SIMD while it factors
    __builtin_amdgcn_s_setprio(3);
    static_for<0, 4>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        double R[4], inv[4];
        row_groups(A[b], R);
        static_for<0, 4>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            inv[q] = rsqrt_refined(bcast_row<4 * b + q>(R[q]));
            // column 4b + q of L: L[j][.] below the diagonal, piv inv in its own lane
            const double lq = R[q] * inv[q];
            R[q] = lq;
            static_for<q + 1, 4>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                fms_bcast_row<4 * b + c, c == q + 1>(R[c], lq, lq);
            });
        });
        // column 4b + g of row j, and its inverse pivot
        const double L4 = g2 ? (g1 ? R[3] : R[2]) : (g1 ? R[1] : R[0]);
        const double i4 = g2 ? (g1 ? inv[3] : inv[2]) : (g1 ? inv[1] : inv[0]);
        if constexpr (b < 3) A = mfma_sub(L4, L4, A);
        const int c = 4 * b + g;
        D[j * 17 + c] = (j > c) ? -(L4 * i4) : 0.0;
        if (j == 0) D[272 + c] = i4;
        if (has_k && j == jk && c == jk) {
            scal[0] = L4;
            scal[1] = i4;
        }
        if (has_y && j == jy && c < jy) yp[base + c] = L4;
    });
    __builtin_amdgcn_s_setprio(0);
}

// Forward substitution X L^T = A for the N-layout tile x held in registers
// (row a of the tile in register a / 4 of row group a % 4, column n in lane
// n): with the weights W in D (factor_diag), column c is final at step c up to
// its pivot, and column n > c gains A[.][c] W[n][c].  Column c of every row
// group sits in lane c of that row, so each step is one DPP broadcast FMA per
// register; the inverse pivots scale the columns at the end.  Backward stable
// like any triangular substitution (no explicit inverse).  The weights of four
// steps are loaded while the previous four steps run; the last column has
// nothing to update.
__device__ __forceinline__ void panel_solve(dvec4 &x, const double *D) {
    const int n = threadIdx.x % 16;
    const double *Wrow = D + n * 17;
    double w[4], wn[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = Wrow[q];
    const double dn = D[272 + n];
    double xs[4] = {x[0], x[1], x[2], x[3]};
    static_for<0, 4>([&](auto gc) {
        constexpr int G = decltype(gc)::value;
        if constexpr (G < 3) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * G + 4 + q < 15) wn[q] = Wrow[4 * G + 4 + q];
        }
        static_for<0, 4>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            constexpr int c = 4 * G + q;
            if constexpr (c < 15) {
                // the first DPP read of a register follows its write by at least three instructions,
                // except at the very first step
                fma_bcast_row_self<c, c == 0>(xs[0], w[q]);
                fma_bcast_row_self<c, false>(xs[1], w[q]);
                fma_bcast_row_self<c, false>(xs[2], w[q]);
                fma_bcast_row_self<c, false>(xs[3], w[q]);
            }
        });
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = wn[q];
    });
    x = dvec4{xs[0] * dn, xs[1] * dn, xs[2] * dn, xs[3] * dn};
}

// One conditional (modes as lds_conditional: qloc == NULL for the
// likelihood term of point i, else the prediction at qloc from row i of nbr).
//
// With G > 1 (W = 1) the workgroup evaluates the conditional of point i for G
// parameter vectors at once (likelihood mode only): wavefront q takes vector
// q, passes its parameters in P and receives its result.  The wavefronts
// share the gather and the pair distances (each evaluates a G-th of them and
// exchanges them through LDS) and otherwise factor and solve their own
// vector, synchronising only with themselves.  Every vector's arithmetic is
// the one the single-vector form performs, in the same order, so the results
// are bitwise the same.  (Factoring the G diagonal tiles of a column in one
// wavefront, one tile per 16-lane row group, returned NaN now and then for
// the vectors held in row groups 1 and 3, in the first workgroups of small
// launches; each vector's wavefront factors its own tile instead.)
template <int T, int W, int KC, bool GRAD, int G = 1>
__device__ __forceinline__ CondOut tile_conditional(const double *__restrict__ locs, const double *__restrict__ z,
                                    const int32_t *__restrict__ nbr, int64_t i, int64_t n, int32_t m,
                                    const double *qloc, const Params &P, double *smem) {
    static_assert(G == 1 || G == 2 || G == 4, "one, two or four parameter vectors per workgroup");
    constexpr bool GCD = kc_gcd(KC);
    using Ls = TileLds<T, W, GRAD, GCD, G, kc_family(KC) == 3>;
    constexpr int NT = G * W * kWave;
    constexpr int NTG = W * kWave;  // threads per parameter vector
    constexpr int NTW = tiles_per_wave(T, W);
    constexpr int NTILES = tile_count(T);
    constexpr int KP = Ls::KP;
    constexpr int DS = Ls::DS;
    constexpr bool UNROLL = W == 1;
    const int tid = threadIdx.x;
    const int wg = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int w = W == 1 ? 0 : (G > 1 ? wg % W : wg);  // wavefront within the vector's group
    const int wq = G > 1 ? wg / W : 0;                 // the group's parameter vector
    const int tg = tid % NTG;            // thread within the group
    double *const CURq = smem + Ls::CUR + wq * Ls::CUR_G;
    double *const SLOTq = smem + Ls::SLOT + wq * Ls::SLOT_G;
    double *const YPq = smem + Ls::YP + wq * Ls::YP_G;
    double *const SCALq = smem + Ls::SCAL + wq * Ls::SCAL_G;
    // synchronisation of the wavefronts that share a vector's tiles: the whole
    // workgroup, except with one wavefront per vector, where each wavefront
    // works on its own vector alone (in lockstep groups, between the shared
    // phases: the gather, and the distance exchanges)
    auto group_sync = [&]() {
        if constexpr (W == 1)
            wave_lds_sync();
        else
            __syncthreads();
    };
    const int l = tid % kWave;
    const int g = l / 16, j = l % 16;
    const int64_t lim = qloc ? n : i;
    const int k = (int)(lim < m ? lim : m);
    double *XY = smem + Ls::XY;
    double *Z = smem + Ls::ZV;
    double *CLv = smem + Ls::CL;

    // my tiles (TileMap); with one wavefront per vector all of this is known
    // at compile time
    uint32_t tmap[TileMap<T, W>::WORDS];
#pragma unroll
    for (int q = 0; q < TileMap<T, W>::WORDS; ++q)
        tmap[q] = W == 1 ? kTileMap<T, W>.word[0][q] : (uint32_t)__builtin_amdgcn_readfirstlane((int)kTileMap<T, W>.word[w][q]);
#define SR(s) ((int)((tmap[(s) / 4] >> (8 * ((s) % 4) + 4)) & 15u))
#define SC(s) ((int)((tmap[(s) / 4] >> (8 * ((s) % 4))) & 15u))
#define SVALID(s) (W * ((s) + 1) <= NTILES || w + W * (s) < NTILES)

    // gather (Algorithm 1: s_{J_i}, y_{J_i}); indices are checked before use.
    // An index out of range or a non-finite input turns the row's observation
    // into NaN, which the forward solve carries into the conditional's value
    // (that is how it is reported); its coordinates become 0, since the
    // covariance code below assumes finite ones.
    for (int t = tid; t < KP; t += NT) {
        double x = 0.0, y = 0.0, zz = 0.0;
        if (t <= k) {
            int64_t jj = i;
            bool ok = true;
            if (t < k) {
                const int32_t jn = nbr[i * (int64_t)m + t];
                ok = (jn >= 0) && ((int64_t)jn < lim);
                jj = ok ? (int64_t)jn : 0;
            }
            if (t == k && qloc) {  // prediction point, observation taken as 0
                x = qloc[0];
                y = qloc[1];
            } else {
                const double2 p = *reinterpret_cast<const double2 *>(locs + 2 * jj);
                x = p.x;
                y = p.y;
                zz = z[jj];
            }
            ok = ok && isfinite(x) && isfinite(y) && isfinite(zz);
            x = ok ? x : 0.0;
            y = ok ? y : 0.0;
            zz = ok ? zz : __builtin_nan("");
        }
        XY[2 * t] = x;
        XY[2 * t + 1] = y;
        Z[t] = zz;
        if constexpr (GCD) CLv[t] = cos_deg(y);
    }
    stage_tables<KC>(tid, smem + Ls::EXPT);
    __syncthreads();

    // covariance generation straight into the N-layout register tiles: lane
    // (g, n) register r of tile (R, C) is entry (16R + 4r + g, 16C + n).
    // Only tiles that reach past row k (the observation row and the identity
    // padding) and diagonal tiles (the nugget) need per-entry cases; the
    // branches on them are uniform over the wavefront.  With the gradient,
    // dC/dbeta is kept in dtile from the same exponential when registers allow.
    constexpr bool KEEP_D = GRAD && keep_dbeta(T, W, GCD, kc_family(KC) == 3);
    const LdsTab ET = lds_table(smem + Ls::EXPT);
    const CovConst CC = cov_const<W == 1>();
    const double diag = P.sigma2 + P.tau2;
    dvec4 tile[NTW];
    dvec4 dtile[KEEP_D ? NTW : 1];
    // With one wavefront per vector (INPLACE) every group needs the same
    // distances: each group's wavefront evaluates those of every G-th (tile,
    // register) pair, 64 lanes at a time, into the panel slots past slot 0,
    // which hold nothing yet (and nothing any more when the gradient's
    // contraction needs the distances again).
    constexpr bool SHARE_D = Ls::INPLACE && G > 1 && T >= 2;
    constexpr int DCH = SHARE_D ? ((T - 1) * DS) / kWave : 1;  // 64-double chunks per vector past slot 0
    static_assert(!SHARE_D || G * DCH >= 4 * NTW, "the shared distances fit in the panel slots");
    auto dslot = [&](int p) __attribute__((always_inline)) -> double * {
        return smem + Ls::SLOT + (p / DCH) * Ls::SLOT_G + DS + (p % DCH) * kWave;
    };
    if constexpr (SHARE_D) {
#pragma unroll
        for (int s = 0; s < NTW; ++s) {
            const int b = 16 * SC(s) + j;
            const double xb = XY[2 * b], yb = XY[2 * b + 1], cb = GCD ? CLv[b] : 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if ((4 * s + r) % G != wq) continue;  // wave-uniform
                const int a = 16 * SR(s) + 4 * r + g;
                dslot(4 * s + r)[l] = pair_dist_pow<KC>(XY[2 * a], XY[2 * a + 1], GCD ? CLv[a] : 0.0, xb, yb, cb, P,
                                                        ET, CC);
            }
        }
        __syncthreads();
    }
    auto fill = [&](auto sc) __attribute__((always_inline)) {
        const int s = sc;
        tile[s] = dvec4{0.0, 0.0, 0.0, 0.0};
        if constexpr (KEEP_D) dtile[s] = dvec4{0.0, 0.0, 0.0, 0.0};
        const int R_ = SR(s), C_ = SC(s);
        if (!SVALID(s)) return;
        const int b = 16 * C_ + j;
        const double xb = XY[2 * b], yb = XY[2 * b + 1], cb = GCD ? CLv[b] : 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = 16 * R_ + 4 * r + g;
            double da;
            if constexpr (SHARE_D)
                da = dslot(4 * s + r)[l];
            else {
                const double2 pa = *reinterpret_cast<const double2 *>(XY + 2 * a);
                da = pair_dist_pow<KC>(pa.x, pa.y, GCD ? CLv[a] : 0.0, xb, yb, cb, P, ET, CC);
            }
            const double rs = scaled_dist(da, P.inv_beta, CC);
            const double e = exp_neg_staged(rs, ET, CC);
            tile[s][r] = cov_value<KC>(rs, e, P);
            if constexpr (KEEP_D) dtile[s][r] = dbeta_raw<KC>(rs, e);
        }
        if (R_ == C_) {
            asm volatile("");  // a branch: the selects cost more than it
#pragma unroll
            for (int r = 0; r < 4; ++r) tile[s][r] = (4 * r + g == j) ? diag : tile[s][r];
        }
        if (16 * R_ + 15 > k) {
#pragma unroll
            for (int r = 0; r < 4; ++r) tile[s][r] = augment_value(16 * R_ + 4 * r + g, b, k, tile[s][r], Z);
        }
    };
    // Great-circle codes as a template loop: with the branches of far pairs the
    // optimiser gives up a loop of this length, and the tiles, indexed at run
    // time, go to scratch memory.
    if constexpr (GCD) {
        static_for<0, NTW>(fill);
    } else {
#pragma unroll
        for (int s = 0; s < NTW; ++s) fill(s);
    }
    // every wavefront has read the shared distances before any writes a
    // panel tile over them
    if constexpr (SHARE_D) __syncthreads();

    // blocked right-looking Cholesky
    const int ty = (k + 1) / 16, jy = (k + 1) % 16;  // the observation row's tile row, and its row there
    auto column = [&](auto tc) __attribute__((always_inline)) {
        const int t = tc;
        // the lane's offset inside a tile slot, opaque to the compiler in every
        // step: otherwise it hoists one address register per slot out of the
        // loop, which at this register budget spill to scratch
        int lo = l * 4;
        asm volatile("" : "+v"(lo));
        const int par = Ls::INPLACE ? t * DS : (Ls::NPAR == 2 ? (t & 1) : 0) * DS;
        double *D = (Ls::INPLACE ? SLOTq : CURq) + par;
        const bool diag_owner = w == tile_index(T, t, t) % W;
        // 1. diagonal tile t (fully updated, in its owner's registers)
        if (diag_owner) {
            dvec4 dt = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < NTW; ++s)
                if (SR(s) == t && SC(s) == t) {
                    if constexpr (!UNROLL) asm volatile("");  // a branch, not eight selects per slot
                    dt = tile[s];
                }
            factor_diag(dt, t, k, D, SCALq, YPq);
        }
        group_sync();
        // 2. tiles below: X = A L_t^-T by substitution, kept in registers
        // (N-layout, the factor tile itself) and published in T-layout
#pragma unroll
        for (int s = 0; s < NTW; ++s) {
            if (SC(s) == t && SR(s) > t) {
                panel_solve(tile[s], D);
                store_panel_tlayout(tile[s], SLOTq + SR(s) * DS);
            }
        }
        group_sync();
        // 3. trailing update of the tiles right of column t
#pragma unroll
        for (int s = 0; s < NTW; ++s) {
            if (SC(s) > t && SVALID(s)) {
                const dvec4 xr = *reinterpret_cast<const dvec4 *>(SLOTq + SR(s) * DS + lo);
                const dvec4 xc = *reinterpret_cast<const dvec4 *>(SLOTq + SC(s) * DS + lo);
#pragma unroll
                for (int q = 0; q < 4; ++q) tile[s] = mfma_sub(xr[q], xc[q], tile[s]);
            }
        }
        // the part of the observation row that lies in this column: row jy of
        // X_ty, entry c in T-layout at lane (c % 4, jy), register c / 4
        if (w == W - 1 && t < ty) {
            if (l < 16) YPq[16 * t + l] = SLOTq[ty * DS + (16 * (l % 4) + jy) * 4 + l / 4];
        }
        // the factor goes to slot t for the back substitution: the panel tile
        // X_t it replaces was last read by the trailing update of column
        // t - 1, and the buffer it leaves is written again by column t + 2
        if constexpr (GRAD && !Ls::INPLACE) {
            if (diag_owner) {
                double *St = SLOTq + t * DS;
                for (int e = l; e < DS; e += kWave) St[e] = D[e];
            }
        }
    };
    // one wavefront per vector knows its tiles at compile time: with the
    // columns unrolled no tile is tested or copied
    for_columns<UNROLL, 0, T, 1>(column);
    group_sync();

    CondOut o;
    const double Lkk = SCALq[0], invk = SCALq[1];
    const double wv = YPq[k];
    o.g0 = o.g1 = o.g2 = 0.0;

    if constexpr (GRAD) {
        const double rr = wv * invk;
        const double half = 0.5 * fma(rr, rr, -(invk * invk));
        // back substitution with L^T for both right-hand sides at once, by
        // columns of tiles from the last: x_t = L_tt^-T (q_t - sum_{R > t}
        // L_Rt^T x_R).  The right-hand sides are q_u = rr y' (y' the
        // observation row of the factor), half L_kk at k, and q_b = L_kk e_k.
        // The sums are taken on the vector units (lane (g, n), register r of
        // an N-layout tile is L[4r + g][n], so a lane's four rows meet the
        // four solution values of its row group: 8 FMAs per tile for both
        // right-hand sides, where a matrix-core product spends 4 x 64 cycles
        // on 2 of 16 columns), then over the row groups.  Every wavefront
        // adds up its tiles R > t + 1 while x_(t+1) is being solved; after
        // the one barrier of a column the owner of tile (t + 1, t) adds that
        // tile and the wavefronts' sums in order and substitutes (row groups
        // 0, 1 and 2, 3 hold the two right-hand sides, lane n entry n).
        double *UB = smem + Ls::UB + wq * Ls::QUB_G;
        double *PART = CURq;  // [2][W][16][2] sums by parity of t; the factors in CUR are in their slots by now
        static_assert(W == 1 || Ls::NPAR * DS >= 64 * W, "the column sums fit in the diagonal-tile buffers");
        auto back_column = [&](auto tc) __attribute__((always_inline)) {
            const int t = tc;
            const double *St = SLOTq + t * DS;  // weights and inverse pivots of tile t
            double su = 0.0, sb = 0.0;
            int uo = 2 * g;  // the lane's rows within a block of the solution, opaque per step (no hoisting)
            asm volatile("" : "+v"(uo));
            auto add_tile = [&](const dvec4 &L, int R) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double2 x = *reinterpret_cast<const double2 *>(UB + 32 * R + 8 * r + uo);
                    su = fma(L[r], x.x, su);
                    sb = fma(L[r], x.y, sb);
                }
            };
            double *Pt = PART + (t & 1) * 32 * W;
            if constexpr (W > 1) {
#pragma unroll
                for (int s = 0; s < NTW; ++s)
                    if (SC(s) == t && SR(s) > t + 1) add_tile(tile[s], SR(s));
                const double sum = sum_row_groups2(su, sb);
                if ((g & 1) == 0) Pt[32 * w + 2 * j + (g >> 1)] = sum;
                group_sync();
                su = sb = 0.0;
            }
            // the solver: the owner of tile (t + 1, t), of tile (t, t) in the last column
            if (w == tile_index(T, t < T - 1 ? t + 1 : t, t) % W) {
#pragma unroll
                for (int s = 0; s < NTW; ++s)
                    if (SC(s) == t && (W > 1 ? SR(s) == t + 1 : SR(s) > t)) add_tile(tile[s], SR(s));
                double sum = sum_row_groups2(su, sb);
                if constexpr (W > 1) {
#pragma unroll
                    for (int v = 0; v < W; ++v) sum += Pt[32 * v + 2 * j + (g >> 1)];
                }
                const int row = 16 * t + j;
                const double qu = (row < k) ? rr * YPq[row] : (row == k ? half * Lkk : 0.0);
                const double q0 = (g >> 1) ? (row == k ? Lkk : 0.0) : qu;
                // x_n = q_n / L_nn, then from the last column x_n += W[c][n] x_c (n < c; the
                // weights W[c][n] = -L[c][n] / L[n][n] are zero for n >= c), four steps loaded ahead
                double qv = (q0 - sum) * St[272 + j];
                double wg[4], wn[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) wg[q] = St[(15 - q) * 17 + j];
                static_for<0, 4>([&](auto gc) {
                    constexpr int S = decltype(gc)::value;  // steps 4S .. 4S + 3 from the last column
                    if constexpr (S < 3) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (11 - 4 * S - q > 0) wn[q] = St[(11 - 4 * S - q) * 17 + j];
                    }
                    static_for<0, 4>([&](auto qc) {
                        constexpr int q = decltype(qc)::value;
                        constexpr int c = 15 - 4 * S - q;
                        if constexpr (c > 0) fma_bcast_row_self<c, true>(qv, wg[q]);
                    });
#pragma unroll
                    for (int q = 0; q < 4; ++q) wg[q] = wn[q];
                });
                if ((g & 1) == 0) UB[2 * row + (g >> 1)] = qv;
            }
            if constexpr (W == 1) group_sync();
        };
        for_columns<UNROLL, T - 1, -1, -1>(back_column);
        group_sync();
        // dl/dtau2 = u^T b; dl/dbeta = sum_{a > b} D_ab (u_a b_b + u_b b_a)
        double ub = 0.0;
        for (int t = tg; t <= k; t += NTG) ub += UB[2 * t] * UB[2 * t + 1];
        double gb = 0.0;
        if constexpr (KEEP_D) {
            // u and b vanish past row k, so entries there add exact zeros; in a
            // diagonal tile the symmetric pairs are both visited and weighted
            // by one half, and D_aa (zero in exact arithmetic, about 2^-500
            // sigma2 / beta^2 with dist_pos) is set to zero.
#pragma unroll
            for (int s = 0; s < NTW; ++s) {
                const int R_ = SR(s), C_ = SC(s);
                if (!SVALID(s) || 16 * R_ > k) continue;
                const double2 ubb = *reinterpret_cast<const double2 *>(UB + 2 * (16 * C_ + j));
                dvec4 db4 = dtile[s];
                double wt = 1.0;
                if (R_ == C_) {  // wave-uniform: only diagonal tiles hold a == b
                    wt = 0.5;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (4 * r + g == j) db4[r] = 0.0;
                }
                double acc = 0.0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double2 uba = *reinterpret_cast<const double2 *>(UB + 2 * (16 * R_ + 4 * r + g));
                    acc = fma(db4[r], fma(uba.x, ubb.y, ubb.x * uba.y), acc);
                }
                gb = fma(wt, acc, gb);
            }
        } else {
            // D again from the distances, over the N (N - 1) / 2 pairs of the
            // N = k + 1 points alone: item p is the pair (b, (b + o) mod N)
            // with b = p mod N and o = 1 + p / N, the items dealt out to the
            // lanes in order (the 16 x 16 tiles hold 1.2 to 2 times as many
            // entries, both halves of the diagonal tiles and the padding
            // among them).  Positions are kept as byte offsets of the 16-byte
            // entries of XY and UB.
            const uint32_t N = (uint32_t)k + 1, NP = N * (uint32_t)k / 2;
            const uint32_t N16 = 16 * N;
            const uint32_t sb16 = 16 * (NTG % N), so16 = 16 * ((NTG / N) % N);
            uint32_t b16 = 16 * ((uint32_t)tg % N), o16 = 16 + 16 * (((uint32_t)tg / N) % N);
            const char *XYb = reinterpret_cast<const char *>(XY), *UBb = reinterpret_cast<const char *>(UB);
            // the next item: b += NTG mod N, o += NTG / N, one more when b passes N
            uint32_t a16 = b16 + o16;
            a16 = min(a16, a16 - N16);
            uint32_t sa16 = sb16 + so16;
            sa16 = min(sa16, sa16 - N16);
            auto next_item = [&]() __attribute__((always_inline)) {
                b16 += sb16;
                a16 += sa16 + (b16 >= N16 ? 16u : 0u);
                b16 = min(b16, b16 - N16);
                a16 = min(a16, a16 - N16);
            };
            auto pair_dist = [&](uint32_t pa, uint32_t pb) __attribute__((always_inline)) {
                const double2 xa = *reinterpret_cast<const double2 *>(XYb + pa);
                const double2 xb = *reinterpret_cast<const double2 *>(XYb + pb);
                return pair_dist_pow<KC>(xa.x, xa.y, GCD ? CLv[pa / 16] : 0.0, xb.x, xb.y, GCD ? CLv[pb / 16] : 0.0, P,
                                         ET, CC);
            };
            if constexpr (SHARE_D) {
                // the distances shared as in the fill, once every wavefront is
                // past its back substitution (the last reader of its slots):
                // wavefront q evaluates those of every G-th run of 64 items
                static_assert(G * DCH >= (KP - 1) * (KP - 2) / 2 / kWave + 1, "the shared distances fit");
                const uint32_t b0 = b16, a0 = a16;
                __syncthreads();
                for (uint32_t p = tg, c = 0; p - tg < NP; p += NTG, ++c) {
                    if ((int)(c % G) == wq && p < NP) dslot((int)c)[l] = pair_dist(a16, b16);
                    next_item();
                }
                __syncthreads();
                b16 = b0;
                a16 = a0;
            }
            auto add_item = [&](uint32_t pa, uint32_t pb, int c) __attribute__((always_inline)) {
                double da;
                if constexpr (SHARE_D) da = dslot(c)[l];
                else da = pair_dist(pa, pb);
                const double rs = scaled_dist(da, P.inv_beta, CC);
                const double dr = dbeta_raw<KC>(rs, exp_neg_staged(rs, ET, CC));
                const double2 ua = *reinterpret_cast<const double2 *>(UBb + pa);
                const double2 vb = *reinterpret_cast<const double2 *>(UBb + pb);
                gb = fma(dr, fma(ua.x, vb.y, vb.x * ua.y), gb);
            };
            const uint32_t whole = NP / NTG;  // rounds in which every lane has an item
            for (uint32_t c = 0; c < whole; ++c) {
                add_item(a16, b16, (int)c);
                next_item();
            }
            if (whole * NTG + tg < NP) add_item(a16, b16, (int)whole);
        }
        // the totals over the lanes (fixed order), then over the wavefronts
        ub = row_sum16(ub);
        gb = row_sum16(gb);
        const double both = sum_row_groups2(ub, gb);  // row groups 0, 1: ub; 2, 3: gb
        if constexpr (W == 1) {
            ub = read_lane(both, 0);
            gb = read_lane(both, 32);
        } else {
            double *red = smem + Ls::RED + wq * Ls::RED_G;
            if ((l & 31) == 0) red[2 * w + l / 32] = both;
            __syncthreads();
            ub = gb = 0.0;
            if (w == 0) {
#pragma unroll
                for (int v = 0; v < W; ++v) {
                    ub += red[2 * v];
                    gb += red[2 * v + 1];
                }
            }
        }
        if (w == 0) {
            o.g2 = ub;
            o.g0 = (0.5 * fma(wv, wv, -1.0) - P.tau2 * ub) / P.sigma2;
            o.g1 = gb * dbeta_scale<KC>(P);
        }
    }
    // the vector's first wavefront reports
    if (w == 0) {
        o.ell = -0.5 * (kLog2Pi + 2.0 * log_pos(Lkk) + wv * wv);
        o.var = Lkk * Lkk;
        o.mean = Z[k] - wv * Lkk;
        o.bad = !isfinite(o.ell) || !isfinite(o.g0) || !isfinite(o.g1) || !isfinite(o.g2);
    } else {
        o.ell = o.var = o.mean = 0.0;
        o.bad = false;
    }
    return o;
#undef SR
#undef SC
#undef SVALID
}

}  // namespace vecchia
