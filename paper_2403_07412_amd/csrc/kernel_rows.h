// Rows kernel: four conditionals per wavefront, one per 16-lane row group, for
// blocks of up to four tile rows (conditioning sets of up to 62 points).
//
// The augmented block is the tiled kernel's (rows 0..k-1 neighbours, row k the
// point, row k+1 the observations, identity beyond), held one row per lane:
// lane j of the group keeps rows j, 16 + j, .., register c of tile (R, C) the
// entry (16R + j, 16C + c).  Column c of the factor is one DPP row broadcast
// per use, so every group factors and solves its own conditional with the same
// instructions and nothing is shared or synchronised between conditionals.
//
// Why: the kernels are bound by vector issue (four cycles of a SIMD for any
// vector instruction, 64 for an FP64 matrix product, never both at once), and
// an FMA with a broadcast operand does as much work per cycle as the matrix
// product.  The tiled kernel's wavefront factors one diagonal tile at a time,
// all four row groups repeating it (380 issue slots); here the same slots
// factor four (m = 30, value: 636 vector instructions per conditional for
// about 1800).  The registers set the limit: 32 per tile and lane.
//
// Gradient: back substitution needs columns of the factor in lanes; each tile
// is transposed through LDS.  dC/dbeta stays in registers from the fill, or is
// evaluated again over the pairs.
#pragma once

#include "device_common.h"
#include "kernel_tile.h"

namespace vecchia {

// Whether dC/dbeta stays in registers from the fill: up to two tile rows; three
// rows of tiles alone take 192 of the 256 registers, and the derivative is
// evaluated again over the pairs.
__host__ __device__ constexpr bool rows_keep_dbeta(int T) { return T <= 2; }

// Whether finished rows of tiles leave the registers: four tile rows with the
// gradient are ten tiles of 32 registers.  Once diagonal tile C is factored the
// tiles (C, 0..C) are needed only by the back substitution; they are
// transposed there and then and kept in the wavefront's scratch memory, as far
// as the factorisation would otherwise hold more than six tiles, its most
// without the gradient: tiles (2, 1) and (2, 2) stay, beside the four of the
// last row.  The four tiles in scratch memory are 8 KB per conditional each
// way, mostly past the L2 (400,000 points, m = 62: 4.15 ms with all six there,
// 3.44 with none moved).
__host__ __device__ constexpr bool rows_stash(int T, bool grad) { return grad && T == 4; }
__host__ __device__ constexpr bool rows_stash_tile(int T, int R, int C) { return R < T - 2 || (R == T - 2 && C == 0); }

// What the four row groups of a wavefront hold.
//   kRowsItems4  four items;
//   kRowsShare   one point under four parameter vectors.  Each group evaluates
//                the distances of every fourth column, or round of the
//                contraction, and the others take them through the LDS
//                crossbar, which is idle: a Matern evaluation is 14
//                instructions of distance and 16 to 19 of covariance;
//   kRowsSolo    one item, for launches that leave most of the GPU idle
//                (rows_solo).  The covariances and their derivatives are
//                shared as the distances are above, a quarter of the
//                evaluations in a chain that a wavefront works through by
//                itself; the groups repeat the factorisation.  (Two items, in
//                two groups each, gained nothing between the two.)
// An item's arithmetic and its order are the same in all of them, so its
// results are the same bits.
enum RowsMode { kRowsItems4, kRowsShare, kRowsSolo };
__host__ __device__ constexpr int rows_groups(RowsMode mode) { return mode == kRowsSolo ? 4 : 1; }

// Whether kRowsSolo keeps the block in LDS for the back substitution: with the
// gradient from three tile rows on, where the other modes transpose tile after
// tile or stash them, and evaluate dC/dbeta again.  One matrix per wavefront
// takes the factor in its lower half and dC/dbeta in the upper, as they come.
__host__ __device__ constexpr bool rows_matrix(int T, bool grad, RowsMode mode) {
    return mode == kRowsSolo && grad && !rows_keep_dbeta(T);
}

// LDS of one wavefront, in doubles: everything is per item (whose row groups
// write alike).
template <int T, bool GRAD, bool GCD, RowsMode MODE>
struct RowsLds {
    static constexpr int KP = 16 * T;
    static constexpr int NG = 4 / rows_groups(MODE);
    static constexpr bool MATRIX = rows_matrix(T, GRAD, MODE);
    static constexpr int TS = 16 * 17;                      // one tile, row stride 17
    static constexpr int LD = KP + 2;                       // row stride of the matrix
    static constexpr int XY = 0;                            // [NG][KP][2] coordinates
    static constexpr int ZV = XY + NG * 2 * KP;             // [NG][KP]    observations
    static constexpr int CL = ZV + NG * KP;                 // [NG][KP]    cos(latitude) (great-circle codes only)
    static constexpr int YP = CL + (GCD ? NG * KP : 0);     // [NG][KP]    zeros, later factor row k+1
    static constexpr int SCAL = YP + NG * KP;               // [NG][2]     L_kk, y_k
    static constexpr int BUF = SCAL + 2 * NG;               // [NG][TS]    tile being transposed (gradient), or the matrix
    static constexpr int UB = BUF + (MATRIX ? KP * LD : 0); // [NG][KP][2] solutions (u, b), once no tile is left
    static constexpr int TOTAL = MATRIX ? UB + 2 * KP : BUF + (GRAD ? NG * TS : 0);
    static_assert(2 * KP <= TS, "the solutions fit in the tile buffer");
};

// v moved up N lanes within each row; the first N lanes get 0.
template <int N>
__device__ __forceinline__ double shift_up(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)__double2loint(v), 0x110 + N, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)__double2hiint(v), 0x110 + N, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// v of lane j of the G-th row group from the one whose lane j is lane first / 4.
template <int G>
__device__ __forceinline__ double from_group(double v, int first) {
    const int lo = __builtin_amdgcn_ds_bpermute(first + 64 * G, (int)__double2loint(v));
    const int hi = __builtin_amdgcn_ds_bpermute(first + 64 * G, (int)__double2hiint(v));
    return __hiloint2double(hi, lo);
}

// One conditional per row group (modes as lds_conditional); `active` is false
// in groups without an item, which compute on an empty set.  Results are
// valid in every lane of the group.
template <int T, int KC, bool GRAD, RowsMode MODE>
__device__ __forceinline__ CondOut rows_conditional(const double *__restrict__ locs, const double *__restrict__ z,
                                                    const int32_t *__restrict__ nbr, int64_t i, int64_t n, int32_t m,
                                                    const double *qloc, const Params &P, bool active,
                                                    LdsTab ET, double *smem) {
    constexpr bool GCD = kc_gcd(KC), SHARE = MODE == kRowsShare;
    constexpr int GPI = rows_groups(MODE);  // row groups per item
    constexpr bool SPLIT = GPI > 1;
    using Ls = RowsLds<T, GRAD, GCD, MODE>;
    constexpr int KP = Ls::KP;
    constexpr int NT = T * (T + 1) / 2;
    constexpr bool KEEP = GRAD && rows_keep_dbeta(T);
    constexpr bool MATRIX = Ls::MATRIX;
    constexpr bool STASH = rows_stash(T, GRAD) && !MATRIX;
    constexpr int LD = Ls::LD;
    const int l = threadIdx.x % kWave;
    const int g = l / 16, j = l % 16;
    const int64_t lim = qloc ? n : i;
    const int k = active ? (int)(lim < m ? lim : m) : 0;
    // the least and the largest set of the wavefront (scalars)
    int kmin = __builtin_amdgcn_readlane(k, 0), kmax = kmin;
#pragma unroll
    for (int q = 1; q < 4; ++q) {
        const int kq = __builtin_amdgcn_readlane(k, 16 * q);
        kmin = min(kmin, kq);
        kmax = max(kmax, kq);
    }
    const int gl = g / GPI, sub = g % GPI;  // the item within the wavefront, the group within the item
    double *XY = smem + Ls::XY + gl * 2 * KP;
    double *Z = smem + Ls::ZV + gl * KP;
    double *CLv = smem + Ls::CL + gl * KP;
    double *YP = smem + Ls::YP + gl * KP;
    double *SC = smem + Ls::SCAL + 2 * gl;
    double *BUF = smem + Ls::BUF + gl * Ls::TS;
    double *M = smem + Ls::BUF;  // MATRIX: L[a][b] at M[a LD + b], dC/dbeta of points a > b at M[b LD + a]

    // gather, as in the tiled kernel: a bad index or a non-finite input makes
    // the row's observation NaN
    double px[T], py[T], pc[T];
#pragma unroll
    for (int R = 0; R < T; ++R) {
        const int r = 16 * R + j;
        double x = 0.0, y = 0.0, zz = 0.0;
        if (active && r <= k) {
            int64_t jj = i;
            bool ok = true;
            if (r < k) {
                const int32_t jn = nbr[i * (int64_t)m + r];
                ok = (jn >= 0) && ((int64_t)jn < lim);
                jj = ok ? (int64_t)jn : 0;
            }
            if (r == k && qloc) {
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
        px[R] = x;
        py[R] = y;
        XY[2 * r] = x;
        XY[2 * r + 1] = y;
        Z[r] = zz;
        YP[r] = 0.0;
        if constexpr (GCD) {
            pc[R] = cos_deg(y);
            CLv[r] = pc[R];
        }
    }
    wave_lds_sync();

    // Left-looking by tile columns: the covariances of a column, the products
    // with the columns before it, then its own factorisation.  Without the
    // gradient a row of tiles is dead once its diagonal tile is factored, so
    // at most (T - C) (C + 1) tiles are live: six of the ten at T = 4.
    //
    // Columns past the largest set of the wavefront take no part
    // in any result and are left out of the factorisation.  A diagonal tile
    // needs its lower half only: column c takes lanes j >= c and column 16 - c
    // the other c, so one pass evaluates both (lane j < c the entry
    // (j + 16 - c, 16 - c)) and a lane shift moves the second into place; with
    // zeros shifted in, dC/dbeta of the tile is its strictly lower half.
    const CovConst CC = cov_const<true>();
    const int j4 = 4 * (j + 16 * (SPLIT ? g - sub : 0));  // lane j of the first group that shares with this one
    double A[NT][16], D[KEEP ? NT : 1][16];
    auto tix = [](int R, int C) constexpr { return R * (R + 1) / 2 + C; };
    const double diag = P.sigma2 + P.tau2;
    // 1 / beta for columns c and 16 - c of a diagonal tile with dC/dbeta: lane 0 has
    // the diagonal of column 16 - c, whose distance of 2^-500 is not small under
    // every beta
    const double inv_beta_two = j > 0 ? P.inv_beta : 0.0;
    // tile (R, C) by columns, as the back substitution takes it: register r of
    // lane n is L[r][n]
    auto transpose = [&](const double (&src)[16], double (&dst)[16]) __attribute__((always_inline)) {
        wave_lds_sync();
#pragma unroll
        for (int c = 0; c < 16; ++c) BUF[j * 17 + c] = src[c];
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[r] = BUF[r * 17 + j];
    };
    // diagonal tile C the same way, ready for substitution: register r > n of
    // lane n is -L[r][n] / L[n][n], register 0 is 1 / L[n][n] (0 past row k),
    // the rest are 0
    auto diag_weights = [&](const double *tile, int stride, int C, double (&dst)[16]) __attribute__((always_inline)) {
        const double dn = tile[j * stride + j];
        double inv = __builtin_amdgcn_rcp(dn);
        inv = fma(fma(-dn, inv, 1.0), inv, inv);
        inv = fma(fma(-dn, inv, 1.0), inv, inv);
        inv = (16 * C + j <= k) ? inv : 0.0;
#pragma unroll
        for (int r = 1; r < 16; ++r) {
            const double v = tile[r * stride + j];
            dst[r] = (r > j) ? -(v * inv) : 0.0;
        }
        dst[0] = inv;
    };
    auto transpose_diag = [&](const double (&src)[16], int C, double (&dst)[16]) __attribute__((always_inline)) {
        wave_lds_sync();
#pragma unroll
        for (int c = 0; c < 16; ++c) BUF[j * 17 + c] = src[c];
        wave_lds_sync();
        diag_weights(BUF, 17, C, dst);
    };
    // the part of factor row k + 1 that lies in tile row R, from its lane
    auto keep_observation_row = [&](auto Rc) __attribute__((always_inline)) {
        constexpr int R = decltype(Rc)::value;
        if (16 * R + j == k + 1) {
            static_for<0, 16 * (R + 1)>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                YP[c] = A[tix(R, c / 16)][c % 16];
            });
        }
    };
    typedef __attribute__((address_space(5))) double *ScratchPtr;
    double stash_mem[STASH ? 16 * ((T - 2) * (T - 1) / 2 + 1) : 1];
    ScratchPtr stash = (ScratchPtr)stash_mem;
    if constexpr (STASH) asm volatile("" : "+v"(stash));  // kept in memory: the compiler cannot see through it
    double Lk = 1.0, yk = 0.0;
    static_for<0, T>([&](auto Cc) {
        constexpr int C = decltype(Cc)::value;
        const double2 *XYt = reinterpret_cast<const double2 *>(XY) + 16 * C;
        if (16 * C <= kmax) {
            // the diagonal tile, columns c and 16 - c together
            auto diag_dist = [&](auto c) __attribute__((always_inline)) {  // of columns c and 16 - c, 0 <= c < 8
                const bool low = j >= c;  // this lane evaluates column c
                const int ra = low ? j : j + 16 - c, cl = low ? c : 16 - c;
                const double2 pa = XYt[ra], pb = XYt[cl];
                double ca = 0.0, cb = 0.0;
                if constexpr (GCD) {
                    ca = CLv[16 * C + ra];
                    cb = CLv[16 * C + cl];
                }
                return pair_dist_pow<KC>(pa.x, pa.y, ca, pb.x, pb.y, cb, P, ET, CC);
            };
            auto column_dist = [&](auto Rc, auto c) __attribute__((always_inline)) {  // of tile (R, C), column c
                constexpr int R = decltype(Rc)::value;
                const double2 pb = XYt[c];
                return pair_dist_pow<KC>(px[R], py[R], GCD ? pc[R] : 0.0, pb.x, pb.y, GCD ? CLv[16 * C + c] : 0.0, P,
                                         ET, CC);
            };
            double shared = 0.0, shared_v = 0.0, shared_d = 0.0;
            // covariance and derivative at distance da
            auto evaluate = [&](double da, double inv_beta, double &v, double &d) __attribute__((always_inline)) {
                const double rs = scaled_dist(da, inv_beta, CC);
                const double e = exp_neg_staged(rs, ET, CC);
                v = cov_value<KC>(rs, e, P);
                if constexpr (KEEP || MATRIX) d = dbeta_raw<KC>(rs, e);
            };
            // of column c of the tile whose column's distance is dist(c): this
            // group's share of the columns from c, or the column itself;
            // put(c) takes the lane's derivative to the matrix
            auto column = [&](auto cc, auto &&dist, auto &&put, double inv_beta, double &v, double &d)
                __attribute__((always_inline)) {
                constexpr int c = decltype(cc)::value;
                if constexpr (SPLIT) {
                    if constexpr (c % GPI == 0) {
                        evaluate(dist(c + sub), inv_beta, shared_v, shared_d);
                        if constexpr (MATRIX) put(c + sub, shared_d);
                    }
                    v = from_group<c % GPI>(shared_v, j4);
                    if constexpr (KEEP) d = from_group<c % GPI>(shared_d, j4);
                } else if constexpr (SHARE) {
                    if constexpr (c % 4 == 0) shared = dist(c + g);
                    evaluate(from_group<c % 4>(shared, j4), inv_beta, v, d);
                } else {
                    evaluate(dist(cc), inv_beta, v, d);
                }
            };
            auto diag_put = [&](int c, double d) __attribute__((always_inline)) {
                const bool low = j >= c;
                const int row = low ? j : j + 16 - c, col = low ? c : 16 - c;
                if (row > col) M[(16 * C + col) * LD + 16 * C + row] = d;
            };
            static_for<0, 9>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                constexpr bool two = c > 0 && c < 8;
                if (16 * C + c <= kmax) {
                    double v, d;
                    const double inv_beta = KEEP && (two || (SPLIT && c < 8)) ? inv_beta_two : P.inv_beta;
                    if constexpr (c < 8 && (two || SHARE || SPLIT)) column(cc, diag_dist, diag_put, inv_beta, v, d);
                    else evaluate(column_dist(Cc, cc), inv_beta, v, d);
                    if constexpr (MATRIX && c == 8) diag_put(c, d);
                    A[tix(C, C)][c] = (j == c) ? diag : v;
                    if constexpr (two) {
                        const double w = shift_up<16 - c>(v);
                        A[tix(C, C)][16 - c] = (j == 16 - c) ? diag : w;
                    }
                    if constexpr (KEEP) {
                        D[tix(C, C)][c] = (j > c) ? d : 0.0;
                        // lane 16 - c receives its own column's diagonal from lane 0, exactly 0
                        if constexpr (two) D[tix(C, C)][16 - c] = shift_up<16 - c>(d);
                    }
                } else {
                    A[tix(C, C)][c] = 0.0;
                    if constexpr (two) A[tix(C, C)][16 - c] = 0.0;
                    if constexpr (KEEP) {
                        D[tix(C, C)][c] = 0.0;
                        if constexpr (two) D[tix(C, C)][16 - c] = 0.0;
                    }
                }
            });
            static_for<C + 1, T>([&](auto Rc) {
                constexpr int R = decltype(Rc)::value;
                static_for<0, 16>([&](auto cc) {
                    constexpr int c = decltype(cc)::value;
                    double v, d;
                    column(
                        cc, [&](auto x) __attribute__((always_inline)) { return column_dist(Rc, x); },
                        [&](int x, double dx) __attribute__((always_inline)) { M[(16 * C + x) * LD + 16 * R + j] = dx; },
                        P.inv_beta, v, d);
                    A[tix(R, C)][c] = v;
                    if constexpr (KEEP) D[tix(R, C)][c] = d;
                });
            });
        } else {
            static_for<C, T>([&](auto Rc) {
                constexpr int R = decltype(Rc)::value;
#pragma unroll
                for (int c = 0; c < 16; ++c) {
                    A[tix(R, C)][c] = 0.0;
                    if constexpr (KEEP) D[tix(R, C)][c] = 0.0;
                }
            });
        }
        // rows past k: the observations in row k+1, zeros beyond
        static_for<C, T>([&](auto Rc) {
            constexpr int R = decltype(Rc)::value;
            if (16 * R + 15 > kmin) {
                const int row = 16 * R + j;
                const double *src = (row == k + 1) ? Z : YP;
                if (row > k) {
#pragma unroll
                    for (int c = 0; c < 16; ++c) A[tix(R, C)][c] = src[16 * C + c];
                }
            }
        });
        // the columns before: entry (., d) loses L[.][c] L[16C + d][c]
        static_for<0, C>([&](auto Ec) {
            constexpr int E = decltype(Ec)::value;
            if (16 * C <= kmax) {
                static_for<0, 16>([&](auto cc) {
                    constexpr int c = decltype(cc)::value;
                    static_for<0, 16>([&](auto dc) {
                        constexpr int d = decltype(dc)::value;
                        static_for<C, T>([&](auto Rc) {
                            constexpr int R = decltype(Rc)::value;
                            fms_bcast_row<d, c == 0 && d == 0 && R == C>(A[tix(R, C)][d], A[tix(C, E)][c],
                                                                        A[tix(R, E)][c]);
                        });
                    });
                });
            }
        });
        // Cholesky of the column, every tile below the diagonal one in step
        static_for<0, 16>([&](auto cc) {
            constexpr int c = decltype(cc)::value;
            constexpr int col = 16 * C + c;
            if (col <= kmax) {
                double piv = bcast_row<c>(A[tix(C, C)][c]);
                if (col > kmin) {  // smaller sets have no such column
                    asm volatile("");
                    piv = (col > k) ? 1.0 : piv;
                }
                const double inv = rsqrt_refined(piv);
                static_for<C, T>([&](auto Rc) { A[tix(decltype(Rc)::value, C)][c] *= inv; });
                const double lq = A[tix(C, C)][c];
                if (col >= kmin) {  // column k of some group: L_kk and the last entry of the observation row
                    asm volatile("");
                    Lk = (col == k) ? lq : Lk;
                    if constexpr (c < 15) yk = (col == k) ? lq : yk;
                    else if constexpr (C + 1 < T) yk = (col == k) ? A[tix(C + 1, C)][c] : yk;
                }
                static_for<c + 1, 16>([&](auto dc) {
                    constexpr int d = decltype(dc)::value;
                    static_for<C, T>([&](auto Rc) {
                        constexpr int R = decltype(Rc)::value;
                        fms_bcast_row<d, R == C && d == c + 1>(A[tix(R, C)][d], lq, A[tix(R, C)][c]);
                    });
                });
            }
        });
        if constexpr (MATRIX) {
            static_for<C, T>([&](auto Rc) {
                constexpr int R = decltype(Rc)::value;
                double *row = M + (16 * R + j) * LD + 16 * C;
                if constexpr (R > C) {
#pragma unroll
                    for (int c = 0; c < 16; c += 2)
                        *reinterpret_cast<double2 *>(row + c) = make_double2(A[tix(R, C)][c], A[tix(R, C)][c + 1]);
                } else {  // the derivative lies above the diagonal
#pragma unroll
                    for (int c = 0; c < 16; ++c)
                        if (j >= c) row[c] = A[tix(R, C)][c];
                }
            });
        }
        if constexpr (STASH && C + 1 < T) {
            if (16 * C + 15 >= kmin) keep_observation_row(std::integral_constant<int, C>{});
            static_for<0, C + 1>([&](auto Ec) {
                constexpr int E = decltype(Ec)::value;
                if constexpr (rows_stash_tile(T, C, E)) {
                    double Lt[16];
                    if constexpr (E == C) transpose_diag(A[tix(C, C)], C, Lt);
                    else transpose(A[tix(C, E)], Lt);
#pragma unroll
                    for (int r = 0; r < 16; ++r) stash[16 * tix(C, E) + r] = Lt[r];
                }
            });
        }
    });
    // L_kk sits in the lane of row k, y_k in the lane of row k + 1
    if (j == k % 16) SC[0] = Lk;
    if (j == (k + 1) % 16) SC[1] = yk;
    if constexpr (GRAD && !MATRIX) static_for<STASH ? T - 1 : 0, T>(keep_observation_row);
    wave_lds_sync();
    CondOut o;
    const double Lkk = SC[0], wv = SC[1];
    o.g0 = o.g1 = o.g2 = 0.0;

    if constexpr (GRAD) {
        const double invk = 1.0 / Lkk;
        const double rr = wv * invk;
        const double half = 0.5 * fma(rr, rr, -(invk * invk));
        // back substitution with L^T for both right-hand sides (the tiled
        // kernel's): lane n holds entry n of each block
        double xu[T], xb[T];
        const double *Y = MATRIX ? M + (k + 1) * LD : YP;  // the observation row of the factor
        for_columns<true, T - 1, -1, -1>([&](auto Cc) __attribute__((always_inline)) {
            constexpr int C = decltype(Cc)::value;
            const int row = 16 * C + j;
            double qu = (row < k) ? rr * Y[row] : (row == k ? half * Lkk : 0.0);
            double qb = (row == k) ? Lkk : 0.0;
            double Lt[16];
            static_for<C + 1, T>([&](auto Rc) {
                constexpr int R = decltype(Rc)::value;
                if (16 * R <= kmax) {
                    if constexpr (STASH && rows_stash_tile(T, R, C)) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) Lt[r] = stash[16 * tix(R, C) + r];
                    } else if constexpr (MATRIX) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) Lt[r] = M[(16 * R + r) * LD + 16 * C + j];
                    } else {
                        transpose(A[tix(R, C)], Lt);
                    }
                    static_for<0, 16>([&](auto rc) {
                        constexpr int r = decltype(rc)::value;
                        fms_bcast_row<r, r == 0>(qu, xu[R], Lt[r]);
                        fms_bcast_row<r, r == 0>(qb, xb[R], Lt[r]);
                    });
                }
            });
            if constexpr (STASH && rows_stash_tile(T, C, C)) {
#pragma unroll
                for (int r = 0; r < 16; ++r) Lt[r] = stash[16 * tix(C, C) + r];
            } else if constexpr (MATRIX) {
                diag_weights(M + 16 * C * (LD + 1), LD, C, Lt);
            } else {
                transpose_diag(A[tix(C, C)], C, Lt);
            }
            qu *= Lt[0];
            qb *= Lt[0];
            for_columns<true, 15, 0, -1>([&](auto rc) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                fma_bcast_row_self<r, true>(qu, Lt[r]);
                fma_bcast_row_self<r, true>(qb, Lt[r]);
            });
            xu[C] = qu;
            xb[C] = qb;
        });
        // dl/dtau2 = u^T b; dl/dbeta = sum over a > b of D_ab (u_a b_b + u_b b_a):
        // per row a the sums of D_ab b_b and D_ab u_b over the columns (u and
        // b vanish past row k)
        double ub = 0.0, gb = 0.0;
        static_for<0, T>([&](auto Rc) { ub = fma(xu[decltype(Rc)::value], xb[decltype(Rc)::value], ub); });
        if constexpr (KEEP) {
            static_for<0, T>([&](auto Rc) {
                constexpr int R = decltype(Rc)::value;
                double su = 0.0, sb = 0.0;
                static_for<0, R + 1>([&](auto Cc) {
                    constexpr int C = decltype(Cc)::value;
                    static_for<0, 16>([&](auto cc) {
                        constexpr int c = decltype(cc)::value;
                        fms_bcast_row<c, c == 0>(su, xu[C], D[tix(R, C)][c]);
                        fms_bcast_row<c, c == 0>(sb, xb[C], D[tix(R, C)][c]);
                    });
                });
                gb -= fma(xu[R], sb, xb[R] * su);
            });
        } else {
            // D again over the N (N - 1) / 2 pairs of the N = k + 1 points, as
            // in the tiled kernel, 16 to a round
            double *UB = smem + Ls::UB + gl * 2 * KP;
            static_for<0, T>([&](auto Rc) {
                constexpr int R = decltype(Rc)::value;
                UB[2 * (16 * R + j)] = xu[R];
                UB[2 * (16 * R + j) + 1] = xb[R];
            });
            wave_lds_sync();
            const uint32_t N = (uint32_t)k + 1, NP = N * (uint32_t)k / 2;
            const char *XYb = reinterpret_cast<const char *>(XY), *UBb = reinterpret_cast<const char *>(UB);
            // the pairs `first`, `first` + `step`, ..: byte offsets of the two points
            struct Walk {
                uint32_t N16, sb, sa, b, a;
                __device__ __forceinline__ Walk(uint32_t N, uint32_t first, uint32_t step) : N16(16 * N) {
                    sb = 16 * (step % N);
                    sa = sb + 16 * ((step / N) % N);
                    sa = min(sa, sa - N16);
                    b = 16 * (first % N);
                    a = b + 16 + 16 * ((first / N) % N);
                    a = min(a, a - N16);
                }
                __device__ __forceinline__ void next() {
                    b += sb;
                    a += sa + (b >= N16 ? 16u : 0u);
                    b = min(b, b - N16);
                    a = min(a, a - N16);
                }
            };
            Walk w(N, j, 16);
            auto pair_dist = [&](const Walk &p) __attribute__((always_inline)) {
                const double2 xa = *reinterpret_cast<const double2 *>(XYb + p.a);
                const double2 xc = *reinterpret_cast<const double2 *>(XYb + p.b);
                return pair_dist_pow<KC>(xa.x, xa.y, GCD ? CLv[p.a / 16] : 0.0, xc.x, xc.y, GCD ? CLv[p.b / 16] : 0.0,
                                         P, ET, CC);
            };
            auto pair_dbeta = [&](double da) __attribute__((always_inline)) {
                const double rs = scaled_dist(da, P.inv_beta, CC);
                return dbeta_raw<KC>(rs, exp_neg_staged(rs, ET, CC));
            };
            auto pair_weight = [&](const Walk &p) __attribute__((always_inline)) {
                const double2 ua = *reinterpret_cast<const double2 *>(UBb + p.a);
                const double2 vb = *reinterpret_cast<const double2 *>(UBb + p.b);
                return fma(ua.x, vb.y, vb.x * ua.y);
            };
            auto add_pair = [&](double da) __attribute__((always_inline)) {
                const double d = pair_dbeta(da);
                gb = fma(d, pair_weight(w), gb);
            };
            if constexpr (SPLIT) {
                constexpr int STEP = 16 * GPI;
                Walk own(N, 16 * sub + j, STEP);  // the pairs this lane evaluates, any of the set past the last item
                const uint32_t NPmax = ((uint32_t)kmax + 1) * (uint32_t)kmax / 2;
                for (uint32_t p = 0; p < NPmax; p += STEP) {
                    double d;
                    if constexpr (MATRIX) {
                        const uint32_t low = min(own.a, own.b), high = max(own.a, own.b);
                        d = M[(low / 16) * LD + high / 16];
                    } else {
                        d = pair_dbeta(pair_dist(own));
                    }
                    const double u = pair_weight(own);
                    own.next();
                    static_for<0, GPI>([&](auto sc) {
                        constexpr int q = decltype(sc)::value;
                        const double dq = from_group<q>(d, j4), uq = from_group<q>(u, j4);
                        gb = p + 16 * q + j < NP ? fma(dq, uq, gb) : gb;
                    });
                }
            } else if constexpr (SHARE) {
                Walk own(N, 16 * g + j, 64);  // the pairs whose distance this lane evaluates
                uint32_t p = 0;
                for (; p + 64 <= NP; p += 64) {
                    const double mine = pair_dist(own);
                    own.next();
                    static_for<0, 4>([&](auto sc) {
                        add_pair(from_group<decltype(sc)::value>(mine, j4));
                        w.next();
                    });
                }
                const double mine = pair_dist(own);  // any pair of the set past the last item
                static_for<0, 4>([&](auto sc) {
                    constexpr int q = decltype(sc)::value;
                    const double da = from_group<q>(mine, j4);
                    if (p + 16 * q + j < NP) add_pair(da);
                    w.next();
                });
            } else {
                const uint32_t whole = ((uint32_t)kmin + 1) * (uint32_t)kmin / 32;  // rounds every lane takes part in
                const uint32_t rounds = (((uint32_t)kmax + 1) * (uint32_t)kmax / 2 + 15) / 16;
                // four rounds at a time, each step's loads and chains in flight
                // together (m = 60, 2,000 points: 66.9 us one by one, 63.2 so; m =
                // 45, 100,000 points 512 and 486)
                constexpr int NB = 4;
                uint32_t c = 0;
                for (; c + NB <= whole; c += NB) {
                    double d[NB], u[NB];
                    static_for<0, NB>([&](auto x) {
                        d[x] = pair_dist(w);
                        u[x] = pair_weight(w);
                        w.next();
                    });
                    static_for<0, NB>([&](auto x) { d[x] = pair_dbeta(d[x]); });
                    static_for<0, NB>([&](auto x) { gb = fma(d[x], u[x], gb); });
                }
                for (; c < whole; ++c) {
                    add_pair(pair_dist(w));
                    w.next();
                }
                for (c = whole; c < rounds; ++c) {
                    if (16 * c + j < NP) add_pair(pair_dist(w));
                    w.next();
                }
            }
        }
        ub = row_sum16(ub);
        gb = row_sum16(gb);
        o.g2 = ub;
        o.g0 = (0.5 * fma(wv, wv, -1.0) - P.tau2 * ub) / P.sigma2;
        o.g1 = gb * dbeta_scale<KC>(P);
    }
    o.ell = -0.5 * (kLog2Pi + 2.0 * log_pos(Lkk) + wv * wv);
    o.var = Lkk * Lkk;
    o.mean = Z[k] - wv * Lkk;
    o.bad = !isfinite(o.ell) || !isfinite(o.g0) || !isfinite(o.g1) || !isfinite(o.g2);
    return o;
}

}  // namespace vecchia
