// HIP kernels for gfx950 (MI355X): the TSM2L family and the reductions along
// the contiguous dimension.
//
//  rowtile   O = X*Y with X tall (m x kin, kin <= 32): each lane loads its
//            16-byte row runs of X once and produces the output columns from
//            a Y panel held in registers.  This is TSM2L (Algorithm 6: a grid
//            smaller than m walks the horizontal tiles of A) and also the
//            gradient dA = dC*B^T for both problem classes.
//
//  tn        O = X^T*Y with X (R x ncols) and Y (R x n) column-major, i.e. a
//            reduction along the contiguous dimension: TSM2R with a row-major
//            A, and the gradient dB = A^T*dC.  Loads stream 4 columns x 256
//            bytes per instruction and are re-read in MFMA order from a
//            wavefront-private LDS tile; wavefronts and workgroups split the
//            reduction, finished in double precision in a fixed order.
//
// Also the fixed-order sum of split partials and a zero fill.  The TSM2R
// kernel itself is in tsm2x_tsm2r.hip.
//            and finish it in double precision in a fixed order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstdlib>

#include "tsm2x_internal.h"
#include "tsm2x_device.h"

namespace tsm {

// --------------------------------------------------------------------------
// rowtile: O(m x nout) = X(m x kin) * Y(kin x nout), kin <= 4*KS <= 32,
// Y(ji, jo) = Y[ji * ys_in + jo * ys_out] (so B and B^T are both views).
//
// TSM2L (Design of TSM2L, Algorithm 6): a grid of fewer wavefronts than row
// tiles walks the horizontal tiles of A; each lane loads its 16-byte row
// runs of all kin columns once and B, held whole in registers, never leaves
// the chip, so C is written once and never re-read.  The same kernel gives
// dA = dC * B^T, where nout = k may be large: workgroups then also split the
// output columns and a wavefront reuses its X registers for every 16*NT16
// output columns of its range.
//
// On the matrix cores: O^T = Y^T * X^T with S[rl][kk] = Y(4 st + kk,
// col0 + 16 t + rl) and T[kk][rl] = X[row(rl, q), 4 st + kk]; lane l holds
// O[row(rl, q), col0 + 16 t + mrow(kk, r)] in acc[g][q][t][r] with
// row(rl, q) = row0 + 16*RL*g + RL*rl + q.
//
// Row-major X (ROWX: row i at X + i*ldx, its kin values contiguous): the
// contraction may visit the columns in any order, so step st takes column
// jcol(st) = 4 W (st / W) + W kk + st % W (W = the values of a 16-byte piece,
// or KS if fewer) and a lane's W steps are one contiguous load of its row;
// the four rows q of a lane lie next to each other, so the loads of a tile
// cover it whole and each line is fetched once.  Nothing goes through LDS.
// --------------------------------------------------------------------------
template <typename T, int KS, int NT16, int RG, bool LINE, int ROWX>
__global__ __launch_bounds__(256) void rowtile_kernel(
    int64_t m, int kin, int64_t nout, const T* __restrict__ X, int64_t ldx,
    const T* __restrict__ Y, int64_t ys_in, int64_t ys_out, T* __restrict__ O,
    int64_t ldo, int64_t cols_per_block, double beta) {
    typedef Mfma<T> M;
    typedef typename M::acc Acc;
    constexpr int RL = 16 / (int)sizeof(T);
    constexpr int TR = 16 * RL * RG;
    constexpr int WPB = 4;
    constexpr int CW = 16 * NT16;        // output columns per pass

    const int lane = threadIdx.x & (WAVE - 1);
    const int rl = lane & 15, kk = lane >> 4;
    const int w = threadIdx.x / WAVE;
    const int64_t cb0 = (int64_t)blockIdx.y * cols_per_block;
    const int64_t cb1 = (cb0 + cols_per_block < nout) ? cb0 + cols_per_block : nout;

    constexpr int W = RL < KS ? RL : KS;     // columns of a lane's piece (ROWX)
    auto jcol = [&](int st) { return ROWX ? 4 * W * (st / W) + W * kk + st % W : 4 * st + kk; };

    T yv[KS][NT16];
    auto loadY = [&](int64_t c0) {
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int t = 0; t < NT16; ++t) {
                const int ji = jcol(st);
                const int64_t jo = c0 + 16 * t + rl;
                yv[st][t] = (ji < kin && jo < cb1) ? Y[ji * ys_in + jo * ys_out] : T(0);
            }
    };
    const bool one_pass = (cb1 - cb0) <= CW;
    if (one_pass) loadY(cb0);

    // ROWX: a piece that ends beyond kin loads the row's last W values, which
    // `place` shifts into order when the tile is used (the selects right
    // behind each load would wait for it); rows beyond m load row m - 1 (they
    // are not stored).  A row of fewer than W values is read value by value.
    auto loadX_row = [&](int64_t tile, T (&xv)[KS][RG][RL]) {
        typedef typename VecOf<T, W>::mem V;
        auto row = [&](int g, int q) {
            const int64_t r = tile * TR + 16 * RL * g + RL * rl + q;
            return X + (r < m ? r : m - 1) * ldx;
        };
        if (ROWX == 1 || kin >= W) {
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int q = 0; q < RL; ++q)
#pragma unroll
                    for (int h = 0; h < KS / W; ++h) {
                        const int j0 = 4 * W * h + W * kk;
                        const int jc = ROWX == 1 || j0 < kin - W ? j0 : kin - W;
                        const V v = *reinterpret_cast<const V*>(row(g, q) + jc);
#pragma unroll
                        for (int e = 0; e < W; ++e) xv[W * h + e][g][q] = v[e];
                    }
        } else {
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int q = 0; q < RL; ++q)
#pragma unroll
                    for (int st = 0; st < KS; ++st)
                        xv[st][g][q] = jcol(st) < kin ? row(g, q)[jcol(st)] : T(0);
        }
    };
    auto place = [&](T (&xv)[KS][RG][RL]) {
#pragma unroll
        for (int h = 0; h < KS / W; ++h) {
            const int j0 = 4 * W * h + W * kk;
            const int sh = j0 < kin - W ? 0 : j0 - (kin - W);
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int q = 0; q < RL; ++q)
#pragma unroll
                    for (int e = 0; e < W; ++e) {
                        T v = T(0);
#pragma unroll
                        for (int s = 0; s + e < W; ++s) v = sh == s ? xv[W * h + e + s][g][q] : v;
                        xv[W * h + e][g][q] = v;
                    }
        }
    };
    auto loadX = [&](int64_t tile, T (&xv)[KS][RG][RL]) {
        if constexpr (ROWX) {
            loadX_row(tile, xv);
            return;
        }
        const int64_t row0 = tile * TR;
        const bool full = (row0 + TR <= m);
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const int ji = 4 * st + kk;
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                const int64_t r = row0 + 16 * RL * g + RL * rl;
                if (ji < kin)
                    load_run<T, RL, LINE>(X + r + ji * ldx, m - r, full, xv[st][g]);
                else
#pragma unroll
                    for (int q = 0; q < RL; ++q) xv[st][g][q] = T(0);
            }
        }
    };

    const int64_t ntiles = (m + TR - 1) / TR;
    const int64_t tstride = (int64_t)gridDim.x * WPB;
    int64_t tile = (int64_t)blockIdx.x * WPB + w;
    T xv[KS][RG][RL];
    if (tile < ntiles) loadX(tile, xv);
    for (; tile < ntiles; tile += tstride) {
        const int64_t row0 = tile * TR;
        const bool full = (row0 + TR <= m);
        const bool more = tile + tstride < ntiles;
        if (ROWX == 2 && kin >= W) place(xv);
        for (int64_t c0 = cb0; c0 < cb1; c0 += CW) {
            if (!one_pass) loadY(c0);
            Acc acc[RG][RL][NT16];
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int q = 0; q < RL; ++q)
#pragma unroll
                    for (int t = 0; t < NT16; ++t) acc[g][q][t] = Acc{0, 0, 0, 0};
#pragma unroll
            for (int st = 0; st < KS; ++st)
#pragma unroll
                for (int g = 0; g < RG; ++g)
#pragma unroll
                    for (int q = 0; q < RL; ++q)
#pragma unroll
                        for (int t = 0; t < NT16; ++t)
                            acc[g][q][t] = M::op(yv[st][t], xv[st][g][q], acc[g][q][t]);
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                const int64_t r = row0 + 16 * RL * g + RL * rl;
#pragma unroll
                for (int t = 0; t < NT16; ++t)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int64_t col = c0 + 16 * t + M::mrow(kk, rr);
                        if (col < cb1) {
                            T v[RL];
#pragma unroll
                            for (int q = 0; q < RL; ++q) v[q] = acc[g][q][t][rr];
                            if (beta != 0.0) {     // O is read only then
                                T o[RL];
                                load_run<T, RL>(O + r + col * ldo, m - r, full, o);
#pragma unroll
                                for (int q = 0; q < RL; ++q)
                                    v[q] = ROWX ? (T)((double)v[q] + beta * (double)o[q])
                                                : (T)__builtin_fma((T)beta, o[q], v[q]);
                            }
                            store_run<T, RL, LINE>(O + r + col * ldo, m - r, full, v);
                        }
                    }
            }
        }
        if (more) {
            loadX(tile + tstride, xv);
        }
    }
}

// --------------------------------------------------------------------------
// tn: O(ncols x n) = X^T * Y with X (R x ncols) and Y (R x n) column-major:
// a reduction along the contiguous dimension.  TSM2R with a row-major A
// (X = A^T) and the gradient dB = A^T * dC.  (YR: Y row-major, n <= 16, loaded
// value by value; for small products.)
//
// D = O tile: S[rl][kk] = X[r, c0 + rl], T[kk][rl] = Y[r, 16 t + rl] with the
// reduction index r = rb + RL*kk + q for step q, so lane l needs RL
// consecutive rows of ONE column for each operand.  Loading that directly
// makes every load instruction touch 16 columns with 64-byte pieces, which
// (measured) caps HBM reads near 60 %.  Instead each wavefront loads blocks
// of SR = 16*RL rows with the 4-columns-x-256-bytes pattern of the other
// kernels (lane (rl, kk) reads rows RL*rl .. of column 4 c + kk), stages
// them in its own padded LDS tile [column][row], and reads them back in the
// MFMA layout (16-byte LDS reads, four blocks of 4*RL rows per stage).  LDS operations of one
// wavefront execute in order, so no barrier is needed between the stage and
// the read-back.  Lane l holds O[c0 + mrow(kk, r), 16 t + rl] in acc[t][r].
// The column groups of a slice run next to each other on one XCD, whose L2
// then fetches the slice's Y once for them (FP32 1000000 x 128, n = 8: 113 ->
// 93 us; FP64 x 48, n = 5: 77 -> 69); the steps of a wavefront start at a
// place that depends on its group and slice, so that groups whose columns lie
// a large power of two apart do not all read the same HBM channels at a time
// (FP32 16384^2, n = 8: 200 -> 170 us, 8192^2: 71 -> 44).
// The WK wavefronts of a workgroup split the workgroup's slice of R, and
// workgroups split R again; partials are added in double precision in a
// fixed order (workgroup level here, across workgroups by
// split_reduce_kernel).
// --------------------------------------------------------------------------
template <typename T, int NT16, int G, int CT, bool LINE, bool YC, bool YR>
__global__ __launch_bounds__(256) void tn_kernel(
    int64_t R, int64_t ncols, int n, const T* __restrict__ X, int64_t ldx,
    const T* __restrict__ Y, int64_t ldy, T* __restrict__ O, int64_t ldo,
    int64_t rslice, double* __restrict__ part, double beta, int pf) {
    typedef Mfma<T> M;
    typedef typename M::acc Acc;
    constexpr int RL = 16 / (int)sizeof(T);
    constexpr int WK = 4;
    constexpr int SR = 16 * RL;                // rows per stage
    constexpr int SROW = SR + RL;              // padded LDS column (16 more bytes)
    constexpr int NX = 16 * CT;                // staged X columns (CT output tiles)
    constexpr int NC = NX + 16 * NT16;         // then the Y columns
    constexpr int NV = 4 * NT16;
    // the staged tiles, and the wavefronts' sums: over the tiles (the loop is
    // done by then), except for n > 16, whose workgroups stream 3-5 % faster
    // with one to a CU than with the two that would fit
    constexpr size_t LB = sizeof(T) * WK * NC * SROW, SB = sizeof(double) * WK * WAVE * NV;
    constexpr bool OVER = NT16 == 1;
    __shared__ __align__(16) unsigned char smem[OVER ? (LB > SB ? LB : SB) : LB + SB];
    T (*lds)[NC][SROW] = reinterpret_cast<T (*)[NC][SROW]>(smem);
    double (*red)[WAVE][NV] = reinterpret_cast<double (*)[WAVE][NV]>(smem + (OVER ? 0 : LB));

    const int lane = threadIdx.x & (WAVE - 1);
    const int rl = lane & 15, kk = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);   // wavefront-uniform
    // a last group of columns that would leave the matrix starts early enough
    // to be whole (tn_finish writes only its own)
    const int nsl = gridDim.y;
    unsigned bx, s;
    xcd_runs(bx, s);
    const int64_t cg0 = (int64_t)bx * NX;
    const int64_t c0 = cg0 + NX > ncols && ncols >= NX ? ncols - NX : cg0;
    const int64_t sb0 = (int64_t)s * rslice;
    const int64_t sb1 = (sb0 + rslice < R) ? sb0 + rslice : R;
    const int64_t lw = rslice / WK;            // multiple of G * SR
    const int64_t wb0 = sb0 + w * lw;
    const int64_t wb1 = (wb0 + lw < sb1) ? wb0 + lw : sb1;
    T (*tile)[SROW] = lds[w];

    Acc acc[CT][NT16];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int t = 0; t < NT16; ++t) acc[ct][t] = Acc{0, 0, 0, 0};
    constexpr bool FL = sizeof(T) == 4;
    constexpr int NA = CT * NT16;
    typedef Acc Flat[NA];
    Acc tot[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) tot[i] = Acc{0, 0, 0, 0};
    auto flush_at = [&](int64_t done) {        // after `done` whole steps
        if (FL && done % (FLUSH / 8) == 0)
            flush<NA>(reinterpret_cast<Flat&>(acc), reinterpret_cast<Flat&>(tot));
    };

    // bounds checks, for groups of fewer than NX columns (clamped, the load
    // instructions without a live column cost more than the waits: FP32
    // 20000000 x 3, n = 1: 189 us, 160 so) and for fewer than RL rows.
    // staged column sc: sc < NX -> X column c0 + sc, else Y column sc - NX
    auto load = [&](int64_t rb, T (&v)[G][NC / 4][RL]) {
#pragma unroll
        for (int gs = 0; gs < G; ++gs) {
            const int64_t r = rb + gs * SR + RL * rl;
            const int64_t valid = wb1 - r;
            const bool full = valid >= RL;
#pragma unroll
            for (int cg = 0; cg < NC / 4; ++cg) {
                const int sc = 4 * cg + kk;
                if (cg < NX / 4) {
                    if (c0 + sc < ncols)
                        load_run<T, RL, LINE>(X + r + (c0 + sc) * ldx, valid, full, v[gs][cg]);
                    else
#pragma unroll
                        for (int q = 0; q < RL; ++q) v[gs][cg][q] = T(0);
                } else {
                    const T* src = Y + r + (int64_t)(sc - NX) * ldy;
                    if (YR) {
#pragma unroll
                        for (int q = 0; q < RL; ++q)
                            v[gs][cg][q] = sc - NX < n && q < valid ? Y[(r + q) * ldy + sc - NX] : T(0);
                    } else if (YC && sc - NX < n && full) {
                        typedef typename VecOf<T, RL>::mem V;
                        const V y = *reinterpret_cast<const V*>(src);
#pragma unroll
                        for (int q = 0; q < RL; ++q) v[gs][cg][q] = y[q];
                    } else if (sc - NX < n) {
                        load_run<T, RL, LINE>(src, valid, full, v[gs][cg]);
                    } else {
#pragma unroll
                        for (int q = 0; q < RL; ++q) v[gs][cg][q] = T(0);
                    }
                }
            }
        }
    };

    // stage the G stages of v and multiply; live: staged Y columns at or
    // beyond n are zeroed (the whole-step loads read column n - 1 there)
    auto stage_mul = [&](const T (&v)[G][NC / 4][RL], bool zero_dead) {
#pragma unroll
        for (int gs = 0; gs < G; ++gs) {
            // stage: column 4 cg + kk, rows RL*rl .. RL*rl + RL - 1
            wave_lds_fence();
#pragma unroll
            for (int cg = 0; cg < NC / 4; ++cg) {
                typedef typename VecOf<T, RL>::type V;
                const bool dead = zero_dead && cg >= NX / 4 && 4 * cg + kk - NX >= n;
                V x;
#pragma unroll
                for (int q = 0; q < RL; ++q) x[q] = dead ? T(0) : v[gs][cg][q];
                *reinterpret_cast<V*>(&tile[4 * cg + kk][RL * rl]) = x;
            }
            // read back in four blocks of 4*RL rows: X columns 16 ct + rl
            // and Y columns NX + 16 t + rl, rows 4*RL*h + RL*kk + q
            wave_lds_fence();
            typedef typename VecOf<T, RL>::type V;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                V ys[NT16];
#pragma unroll
                for (int t = 0; t < NT16; ++t)
                    ys[t] = *reinterpret_cast<const V*>(&tile[NX + 16 * t + rl][4 * RL * h + RL * kk]);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const V xs = *reinterpret_cast<const V*>(&tile[16 * ct + rl][4 * RL * h + RL * kk]);
#pragma unroll
                    for (int t = 0; t < NT16; ++t)
#pragma unroll
                        for (int q = 0; q < RL; ++q)
                            acc[ct][t] = M::op(xs[q], ys[t][q], acc[ct][t]);
                }
            }
        }
    };
    // whole steps: straight-line 16-byte loads (Y through the cache)
    auto load_full = [&](int64_t rb, T (&v)[G][NC / 4][RL]) {
        typedef typename VecOf<T, RL>::mem V;
#pragma unroll
        for (int gs = 0; gs < G; ++gs) {
            const int64_t r = rb + gs * SR + RL * rl;
#pragma unroll
            for (int cg = 0; cg < NC / 4; ++cg) {
                const int sc = 4 * cg + kk;
                if (cg < NX / 4) {
                    load_run<T, RL, LINE>(X + r + (c0 + sc) * ldx, RL, true, v[gs][cg]);
                } else {
                    const int p = sc - NX < n ? sc - NX : n - 1;
                    if (YR) {
#pragma unroll
                        for (int q = 0; q < RL; ++q) v[gs][cg][q] = Y[(r + q) * ldy + p];
                        continue;
                    }
                    const V* src = reinterpret_cast<const V*>(Y + r + (int64_t)p * ldy);
                    const V y = !YC && LINE ? __builtin_nontemporal_load(src) : *src;
#pragma unroll
                    for (int q = 0; q < RL; ++q) v[gs][cg][q] = y[q];
                }
            }
        }
    };

    // steps that end beyond the range: the same at clamped rows, which are
    // shifted into place once all are loaded.  (With a branch around each load
    // the waits behind them drained every load, one after the other where
    // some lanes had whole runs: FP32, row-major 300000 x 33, n = 32 239 us, 165
    // so; n = 8: 77 and 59; 300000 x 40: 74 and 59)
    auto load_part = [&](int64_t rb, T (&v)[G][NC / 4][RL]) {
#pragma unroll
        for (int gs = 0; gs < G; ++gs) {
            const int64_t r = rb + gs * SR + RL * rl;
#pragma unroll
            for (int cg = 0; cg < NC / 4; ++cg) {
                const int sc = 4 * cg + kk;
                if (cg < NX / 4) {
                    load_clamped(X + r + (c0 + sc) * ldx, wb1 - r, v[gs][cg]);
                } else {
                    const int p = sc - NX < n ? sc - NX : n - 1;
                    if (YR) {
#pragma unroll
                        for (int q = 0; q < RL; ++q)
                            v[gs][cg][q] = Y[(r + q < wb1 ? r + q : wb1 - 1) * ldy + p];
                    } else {
                        load_clamped(Y + r + (int64_t)p * ldy, wb1 - r, v[gs][cg]);
                    }
                }
            }
        }
    };
    auto place_part = [&](int64_t rb, T (&v)[G][NC / 4][RL]) {
#pragma unroll
        for (int gs = 0; gs < G; ++gs) {
            const int64_t valid = wb1 - (rb + gs * SR + RL * rl);
#pragma unroll
            for (int cg = 0; cg < NC / 4; ++cg) {
                if (YR && cg >= NX / 4) {
#pragma unroll
                    for (int q = 0; q < RL; ++q) v[gs][cg][q] = q < valid ? v[gs][cg][q] : T(0);
                } else {
                    place_clamped(valid, v[gs][cg]);
                }
            }
        }
    };

    // pf, whole steps: the next step held in flight across the waits
    // for this one (the scheduling barriers keep its loads ahead of them).
    // Not with four stages per step, whose two steps do not fit the
    // registers.
    // whole steps, each column group and slice starting at another one; for
    // n > 16 only slices do, where there is one group: the groups otherwise
    // gain more from reading the same rows of a large Y at a time (FP64
    // 16384^2, n = 32: 450 us with rotated groups, 431 without)
    const int64_t nit = wb1 > wb0 ? (wb1 - wb0) / (G * SR) : 0;
    const unsigned from = NT16 == 1 ? 3u * bx + WK * s : gridDim.x == 1 ? WK * s : 0u;
    const int64_t rot = nit > 0 ? from % (unsigned)nit : 0;
    auto at = [&](int64_t it) {
        const int64_t i = it + rot;
        return it < nit ? wb0 + (i < nit ? i : i - nit) * (G * SR) : wb0 + nit * (G * SR);
    };
    if (pf && nit > 0 && ncols >= NX) {
        T va[G][NC / 4][RL], vb[G][NC / 4][RL];
        load_full(at(0), va);
        int64_t it = 0;
        for (; it + 2 < nit; it += 2) {
            load_full(at(it + 1), vb);
            __builtin_amdgcn_sched_barrier(0);
            stage_mul(va, true);
            load_full(at(it + 2), va);
            __builtin_amdgcn_sched_barrier(0);
            stage_mul(vb, true);
            flush_at(it + 2);
        }
        if (it + 1 < nit) {
            load_full(at(it + 1), vb);
            __builtin_amdgcn_sched_barrier(0);
            stage_mul(va, true);
            stage_mul(vb, true);
        } else {
            stage_mul(va, true);
        }
        flush_at(nit);
        if (at(nit) < wb1) {
            load_part(at(nit), va);
            place_part(at(nit), va);
            stage_mul(va, true);
        }
    } else if (wb1 > wb0 && (ncols < NX || R < RL)) {
        const int64_t all = nit + (at(nit) < wb1 ? 1 : 0);
        T v[G][NC / 4][RL];
        load(at(0), v);
        for (int64_t it = 0; it < all; ++it) {
            T vn[G][NC / 4][RL];
            if (it + 1 < all) load(at(it + 1), vn);
            stage_mul(v, false);
            if (it < nit) flush_at(it + 1);
#pragma unroll
            for (int gs = 0; gs < G; ++gs)
#pragma unroll
                for (int cg = 0; cg < NC / 4; ++cg)
#pragma unroll
                    for (int q = 0; q < RL; ++q) v[gs][cg][q] = vn[gs][cg][q];
        }
    } else if (wb1 > wb0) {
        const int64_t all = nit + (at(nit) < wb1 ? 1 : 0);
        T v[G][NC / 4][RL];
        load_part(at(0), v);
        for (int64_t it = 0; it < all; ++it) {
            T vn[G][NC / 4][RL];
            if (it + 1 < all) load_part(at(it + 1), vn);
            __builtin_amdgcn_sched_barrier(0);
            if (it == nit) place_part(at(it), v);
            stage_mul(v, true);
            if (it < nit) flush_at(it + 1);
#pragma unroll
            for (int gs = 0; gs < G; ++gs)
#pragma unroll
                for (int cg = 0; cg < NC / 4; ++cg)
#pragma unroll
                    for (int q = 0; q < RL; ++q) v[gs][cg][q] = vn[gs][cg][q];
        }
    }

    if (FL) {
#pragma unroll
        for (int i = 0; i < NA; ++i) reinterpret_cast<Flat&>(acc)[i] += tot[i];
    }

    // one 16-column output tile at a time
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        if (OVER || ct > 0) __syncthreads();   // red lies over the tiles, and is reused
        tn_finish<T, NT16, WK>(ncols, n, O, ldo, beta, c0 + 16 * ct, cg0, s, nsl, part, red,
                               acc[ct], [](int kq, int r) { return Mfma<T>::mrow(kq, r); });
    }
}

// C := beta * C (zeros when beta == 0; C is then not read): the product of an
// empty k dimension.
template <typename T>
__global__ void fill_scale_kernel(int64_t m, int64_t n, T* __restrict__ C, int64_t ldc,
                                  T beta) {
    const int64_t total = m * n;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e % m, p = e / m;
        C[i + p * ldc] = beta != T(0) ? beta * C[i + p * ldc] : T(0);
    }
}

// O (k x n, ld ldo) := transpose of Bt (n x k, ld ldb): a B given transposed,
// copied once into the workspace in the layout the TSM2R kernels read.
template <typename T>
__global__ void transpose_kernel(int64_t k, int64_t n, const T* __restrict__ Bt, int64_t ldb,
                                 T* __restrict__ O, int64_t ldo) {
    const int64_t total = k * n;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e % n, j = e / n;      // consecutive threads read along Bt's column
        O[j + p * ldo] = Bt[p + j * ldb];
    }
}

// --------------------------------------------------------------------------
// Launchers
// --------------------------------------------------------------------------
// Resident workgroups per CU of a kernel instance (queried once).
template <typename K>
static int occupancy(K kernel, int threads) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, 0) != hipSuccess || nb < 1)
        nb = 1;
    return nb;
}

template <typename T, int KS, int NT16, int RG, bool LINE, int ROWX>
static int rowtile_launch_st(const LaunchRT& L, hipStream_t st) {
    // persistent grid: as many workgroups as fit at once (queried occupancy),
    // but no more than there are groups of 4 row tiles
    static const int occ = occupancy(rowtile_kernel<T, KS, NT16, RG, LINE, ROWX>, 256);
    constexpr int64_t TR = 16 * (16 / (int64_t)sizeof(T)) * RG;
    const int64_t ntiles = (L.m + TR - 1) / TR;
    int64_t bx = (int64_t)L.cus * occ / (L.blocks_y > 0 ? L.blocks_y : 1);
    const int64_t need = (ntiles + 3) / 4;
    if (bx > need) bx = need;
    if (L.blocks_x > 0 && bx > L.blocks_x) bx = L.blocks_x;
    if (bx < 1) bx = 1;
    dim3 grid((unsigned)bx, (unsigned)L.blocks_y), block(256);
    TSM_LAUNCH((rowtile_kernel<T, KS, NT16, RG, LINE, ROWX>), grid, block, 0, st, L.m, L.kin, L.nout,
               (const T*)L.X, L.ldx, (const T*)L.Y, L.ys_in, L.ys_out, (T*)L.O, L.ldo,
               (int64_t)L.cols_per_block, L.beta);
    return 0;
}

// LINE: X's and O's columns start on 128-byte lines; loads and stores are then
// non-temporal (they fill whole lines: four columns x 256 bytes per
// wavefront instruction).  Otherwise the ends of every run share a line with
// the next tile's: ordinary loads find it in the cache and ordinary stores
// merge there (FP64 10302943 x 23, n = 23: 1249 us with
// non-temporal accesses, 1002 without).  On 64 bytes, what a write to memory
// takes whole, non-temporal ones are the faster again for kin <= 16 (k = 6,
// n = 32, 10000004 rows: FP64 676 us and 751, FP32 341 and 373), and for more on
// up to 2^20 rows (500000 x 32, n = 8: FP32 17.5 and 19.6; 10000004: 354 and
// 327); for a few columns in and out also on less (10000004 x 3, n = 2, on 16
// bytes: FP32 59.9 and 62.3).  Wide outputs (dA of TSM2R), which a wavefront writes column after
// column of one row tile: on 64 bytes (FP64 1000 x 100000, kin = 16: 150 and
// 240; 10008 x 10000: 250 and 342 at kin = 32), and for kin > 16 on any
// alignment, whose tiles are half as high (FP32 10001 x 3000: 44 and 61; kin =
// 8: 57 and 41), but for a few tiles and below 8 MB, which the caches take
// (FP32 1017 x 1022, kin = 32: 9.9 and 8.5); from 2^16 rows on X too on 64
// bytes (FP64 296864 x 160, kin = 8, X off it: 104 and 98; but 128 x 400000, kin
// = 16: 131 and 161).  A next-tile register prefetch was measured and
// dropped: the extra waves it costs hid the latency better.
template <typename T, int KS, int NT16, int RG>
static int rowtile_launch(const LaunchRT& L, hipStream_t st) {
    const int64_t es = sizeof(T);
    bool line = (L.x_rowmajor || line_aligned(L.X, L.ldx * es)) && line_aligned(L.O, L.ldo * es);
    if (L.nout > 32 && L.m * L.nout * es >= (int64_t)1 << 23)
        line = (line_aligned(L.O, L.ldo * es, 64) && (L.m < 1 << 16 || line_aligned(L.X, L.ldx * es, 64))) ||
               (KS == 8 && L.m >= 256);
    else if (L.nout <= 32 && !L.x_rowmajor && (KS < 8 || L.m <= (int64_t)1 << 20))
        line = L.kin + L.nout <= 6 ||
               (line_aligned(L.X, L.ldx * es, 64) && line_aligned(L.O, L.ldo * es, 64));
    const int rowx = !L.x_rowmajor ? 0 : L.kin == 4 * KS ? 1 : 2;
    if (rowx == 2)
        return line ? rowtile_launch_st<T, KS, NT16, RG, true, 2>(L, st)
                   : rowtile_launch_st<T, KS, NT16, RG, false, 2>(L, st);
    if (rowx == 1)
        return line ? rowtile_launch_st<T, KS, NT16, RG, true, 1>(L, st)
                   : rowtile_launch_st<T, KS, NT16, RG, false, 1>(L, st);
    return line ? rowtile_launch_st<T, KS, NT16, RG, true, 0>(L, st)
               : rowtile_launch_st<T, KS, NT16, RG, false, 0>(L, st);
}

template <typename T>
static int rowtile_dispatch(const LaunchRT& L, hipStream_t st) {
    const bool wide = L.nout > 16;   // two 16-column tiles per pass
    switch (L.kp) {
        case 8: return wide ? rowtile_launch<T, 2, 2, 2>(L, st) : rowtile_launch<T, 2, 1, 2>(L, st);
        // k = 16 and 32 with n <= 16: one row group per lane (more waves per
        // SIMD) measured up to 16 % faster for float (k = 16) and 2.7 % on
        // average at k = 32, double the same or faster; for k = 8 and for the
        // wide instances with two groups it was slower
        case 16: return wide ? rowtile_launch<T, 4, 2, 2>(L, st) : rowtile_launch<T, 4, 1, 1>(L, st);
        case 32: return wide ? rowtile_launch<T, 8, 2, 1>(L, st) : rowtile_launch<T, 8, 1, 1>(L, st);
    }
    return 1;
}

int launch_rowtile(const LaunchRT& L, int dtype, hipStream_t st) {
    if (dtype == DT_F64) return rowtile_dispatch<double>(L, st);
    if (dtype == DT_F32) return rowtile_dispatch<float>(L, st);
    return 1;
}

template <typename T, int NT16, int G, int CT>
static int tn_launch(const LaunchTN& L, hipStream_t st) {
    // L.groups 16-column tiles, a multiple of CT: CT of them per workgroup.
    // Y is read by every column group: cached loads when there are several
    // (YC), non-temporal ones when it is streamed once.
    const int64_t gx = L.groups / CT;
    dim3 grid((unsigned)gx, (unsigned)L.S), block(256);
    const int64_t es = sizeof(T);
    const bool line = line_aligned(L.X, L.ldx * es) && line_aligned(L.Y, L.ldy * es);
#define TSM_TN(LINE, YC, YR)                                                                  \
    TSM_LAUNCH((tn_kernel<T, NT16, G, CT, LINE, YC, YR>), grid, block, 0, st, L.R, L.ncols,   \
               (int)L.n, (const T*)L.X, L.ldx, (const T*)L.Y, L.ldy, (T*)L.O, L.ldo, L.rslice, \
               L.part, L.beta, L.pf)
    if (L.y_rowmajor) {
        if constexpr (NT16 == 1) {
            if (line_aligned(L.X, L.ldx * es)) TSM_TN(true, true, true);
            else TSM_TN(false, true, true);
        } else {
            return 1;
        }
    } else if (gx > 1) {
        if (line) TSM_TN(true, true, false); else TSM_TN(false, true, false);
    } else {
        if (line) TSM_TN(true, false, false); else TSM_TN(false, false, false);
    }
#undef TSM_TN
    return 0;
}

template <typename T>
static int tn_dispatch(const LaunchTN& L, hipStream_t st) {
    int rc;
    if (L.n <= 16)
        rc = L.ct == 2 ? tn_launch<T, 1, 1, 2>(L, st) : tn_launch<T, 1, 2, 1>(L, st);
    else
        rc = L.ct == 2 ? tn_launch<T, 2, 1, 2>(L, st) : tn_launch<T, 2, 1, 1>(L, st);
    if (rc || L.S <= 1) return rc;
    return launch_split_reduce(sizeof(T) == 8 ? DT_F64 : DT_F32, L.groups, L.S,
                               L.n <= 16 ? 16 : 32, 16, L.ncols, (int)L.n, L.part, L.O, L.ldo,
                               L.beta, st);
}

int launch_tn(const LaunchTN& L, int dtype, hipStream_t st) {
    if (dtype == DT_F64) return tn_dispatch<double>(L, st);
    if (dtype == DT_F32) return tn_dispatch<float>(L, st);
    return 1;
}

int launch_split_reduce(int dtype, int64_t groups, int S, int NP, int W, int64_t rows, int n,
                        const double* part, void* O, int64_t ldo, double beta, hipStream_t st) {
    // Threads per output by the number of slices, so that each adds at most
    // eight or so, all in flight at once (FP32 2048^2, n = 16, 16 slices: 20.0
    // us with a wavefront per output, 14.4 with eight threads; 1500 x 28032,
    // n = 24, 21 slices: 49 us with a thread per output, 41 with eight).
    // In pieces of at most 2^31 threads: a launch takes fewer than 2^32.
    const int per = S > 64 ? 64 : S > 8 ? 8 : 1;
    const int64_t most = ((int64_t)1 << 31) / per / ((int64_t)n * W);
    if (most > 0 && groups > most) {
        const int64_t es = dtype == DT_F64 ? 8 : 4;
        for (int64_t g = 0; g < groups; g += most) {
            const int64_t gn = groups - g < most ? groups - g : most;
            const int rc = launch_split_reduce(dtype, gn, S, NP, W, rows - g * W, n, part + g * S * NP * W,
                                               (char*)O + g * W * es, ldo, beta, st);
            if (rc) return rc;
        }
        return 0;
    }
    const int64_t total = groups * n * W;
#define TSM_R(T, EL, NTH)                                                                         \
    TSM_LAUNCH((split_reduce_kernel<T, EL, NTH>), dim3((unsigned)((total + EL - 1) / EL)),        \
               dim3(NTH), 0, st, groups, S, NP, W, rows, n, part, (T*)O, ldo, beta)
    const int threads = S > 64 ? 1024 : S > 8 ? 512 : 256;
    if (dtype == DT_F64) {
        if (threads == 1024) TSM_R(double, 16, 1024);
        else if (threads == 512) TSM_R(double, 64, 512);
        else TSM_R(double, 256, 256);
    } else {
        if (threads == 1024) TSM_R(float, 16, 1024);
        else if (threads == 512) TSM_R(float, 64, 512);
        else TSM_R(float, 256, 256);
    }
#undef TSM_R
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

static dim3 flat_grid(int64_t total) {
    int64_t blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    return dim3((unsigned)blocks);
}

int launch_fill_scale(int64_t m, int64_t n, void* C, int64_t ldc, double beta, int dtype,
                      hipStream_t st) {
    const dim3 g = flat_grid(m * n);
    if (dtype == DT_F64)
        TSM_LAUNCH(fill_scale_kernel<double>, g, dim3(256), 0, st, m, n, (double*)C, ldc,
                           beta);
    else
        TSM_LAUNCH(fill_scale_kernel<float>, g, dim3(256), 0, st, m, n, (float*)C, ldc,
                           (float)beta);
    return 0;
}

int launch_transpose(int64_t k, int64_t n, const void* Bt, int64_t ldb, void* O, int64_t ldo,
                     int dtype, hipStream_t st) {
    const dim3 g = flat_grid(k * n);
    if (dtype == DT_F64)
        TSM_LAUNCH(transpose_kernel<double>, g, dim3(256), 0, st, k, n, (const double*)Bt,
                           ldb, (double*)O, ldo);
    else
        TSM_LAUNCH(transpose_kernel<float>, g, dim3(256), 0, st, k, n, (const float*)Bt,
                           ldb, (float*)O, ldo);
    return 0;
}

}  // namespace tsm
