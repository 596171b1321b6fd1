// TSM2R on gfx950 (MI355X): C = A*B with column-major A (m x k, k large) and
// B (k x n), up to 64 columns in one pass.  The kernel, its instances and the
// grid planner.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstdio>
#include <cstdlib>

#include "tsm2x_internal.h"
#include "tsm2x_device.h"

namespace tsm {

// --------------------------------------------------------------------------
// tsm2r_nn: C = A*B, A column-major m x k (k large), n <= 16*NT16.
//
// Outer-product form of the Design of TSM2R (Algorithm 2) on the matrix
// cores: C^T = B^T * A^T.  S is a 16 x 4 block of B^T (lane l: B[j, 16t+rl]),
// T a 4 x 16 block of A^T.  A chunk of 4*ST columns at j0 is consumed in
// steps st = 0..ST-1 with columns j = j0 + ST*kk + st; a lane's ST B values
// of a chunk, B[j0+ST*kk .. j0+ST*kk+ST-1, 16t+rl], are contiguous in B's
// column.  The next chunk's A and B are loaded while the current one is
// multiplied (the prefetching of Algorithm 4); where every chunk is whole
// and the host asks for it (pf), in straight-line code that keeps those
// loads outstanding across the waits for the current chunk.  Lane l ends up with
// C[row0 + 16*RL*g + RL*rl + q, 16t + mrow(kk, r)] in acc[g][q][t][r].
//
// A's columns may start at any element: the 16-byte loads need no alignment
// (element-wise loads there ran at half the rate: FP32 10007 x 9973, n = 5,
// 136 us, now 74), and a last tile or chunk that would leave the matrix is
// moved up, or clamped and zeroed, instead of loaded element by element.
//
// The k range is split across the WK wavefronts of a workgroup and across
// workgroups; the partial sums are added in double precision in a fixed
// order (in LDS within the workgroup, then by split_reduce_kernel).
// --------------------------------------------------------------------------
// Explicit prefetch of the next chunk (Algorithm 4's nextA/nextB).
#ifndef TSM2X_NN_PREFETCH
#define TSM2X_NN_PREFETCH 1
#endif
// Waves per SIMD each instance is compiled for: three for n <= 16 (the
// register budget is then 168), two beyond.
template <typename T, int NT16>
constexpr int nn_waves() { return NT16 == 1 ? 3 : 2; }

template <typename T, int NT16, int RG, int ST, int WK, bool LINE, bool BT,
          bool PF = TSM2X_NN_PREFETCH>
__global__ __launch_bounds__(WAVE * WK)
__attribute__((amdgpu_waves_per_eu(nn_waves<T, NT16>(), 8))) void tsm2r_nn_kernel(
    int64_t m, int64_t k, int n, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ B, int64_t ldb, T* __restrict__ C, int64_t ldc,
    int64_t kslice, double* __restrict__ part, int pf, double beta) {
    typedef Mfma<T> M;
    typedef typename M::acc Acc;
    constexpr int RL = 16 / (int)sizeof(T);
    constexpr int TR = 16 * RL * RG;     // rows per tile
    constexpr int CW = 4 * ST;           // columns per chunk
    constexpr int NP = 16 * NT16;
    constexpr int PG = 4;
    // B run of a lane: ST values in vector loads of at most 16 bytes
    constexpr int BW = ST * (int)sizeof(T) > 16 ? RL : ST;
    static_assert(WK * PG * TR * 8 <= 32768, "LDS budget");
    __shared__ __align__(16) unsigned char smem[WK * PG * TR * 8];

    const int lane = threadIdx.x & (WAVE - 1);
    const int rl = lane & 15, kk = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);   // wavefront-uniform
    const int nsl = gridDim.y;
    unsigned bx = blockIdx.x, s = blockIdx.y;
    if (!LINE) xcd_runs(bx, s);          // (nn_instance)
    const int64_t tile = bx;
    // a last tile that would leave the matrix starts early enough to be whole
    // (nn_finish writes only its own rows)
    const int64_t row0 = tile * TR + TR > m && m >= TR ? m - TR : tile * TR;
    const bool full = (row0 + TR <= m);
    const int64_t kb0 = (int64_t)s * kslice;
    const int64_t kb1 = (kb0 + kslice < k) ? kb0 + kslice : k;
    const int64_t lw = kslice / WK;
    const int64_t wk0 = kb0 + w * lw;
    const int64_t wk1 = (wk0 + lw < kb1) ? wk0 + lw : kb1;

    Acc acc[RG][RL][NT16];
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int q = 0; q < RL; ++q)
#pragma unroll
            for (int t = 0; t < NT16; ++t) acc[g][q][t] = Acc{0, 0, 0, 0};
    // the second set of sums, where registers allow it (n = 17..32 has none
    // to spare; with 49..64 columns 11 registers spill for a column-major B, 3 %,
    // and 52 or 84 for a row-major one, whose scratch accesses lie in the loop
    // and which runs no slower for it: 20480^2, n = 64, 500 us and 504
    // column-major.  FP64 spills 101 and 108 there, outside its loop, flush or not)
    constexpr bool FL = sizeof(T) == 4 && RG <= 2 && (NT16 == 1 || RG == 1);
    constexpr int NA = RG * RL * NT16;
    typedef Acc Flat[NA];
    Acc tot[FL ? NA : 1];
#pragma unroll
    for (int i = 0; i < (FL ? NA : 1); ++i) tot[i] = Acc{0, 0, 0, 0};
    auto flush_at = [&](int done) {            // after `done` chunks
        if constexpr (FL)
            if (done % FLUSH == 0) flush<NA>(reinterpret_cast<Flat&>(acc), reinterpret_cast<Flat&>(tot));
    };

    auto loadA = [&](int64_t j0, T (&av)[ST][RG][RL]) {
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            const int64_t j = j0 + ST * kk + st;
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                const int64_t r = row0 + 16 * RL * g + RL * rl;
                if (j < wk1)
                    load_run<T, RL, LINE>(A + r + j * lda, m - r, full, av[st][g]);
                else
#pragma unroll
                    for (int q = 0; q < RL; ++q) av[st][g][q] = T(0);
            }
        }
    };
    // a lane's ST values of B in a chunk are contiguous in B's column; B is
    // re-read by every row tile, so these are ordinary (cached) loads
    auto loadB = [&](int64_t j0, T (&bv)[NT16][ST]) {
#pragma unroll
        for (int t = 0; t < NT16; ++t) {
            const int p = 16 * t + rl;
            const int64_t jb = j0 + ST * kk;
            const T* __restrict__ src = B + (BT ? jb * ldb + p : jb + (int64_t)p * ldb);
            if (!BT && p < n && jb + ST <= wk1) {
                typedef typename VecOf<T, BW>::mem V;
#pragma unroll
                for (int h = 0; h < ST / BW; ++h) {
                    const V v = *reinterpret_cast<const V*>(src + h * BW);
#pragma unroll
                    for (int e = 0; e < BW; ++e) bv[t][h * BW + e] = v[e];
                }
            } else {
#pragma unroll
                for (int st = 0; st < ST; ++st)
                    bv[t][st] = (p < n && jb + st < wk1) ? src[BT ? st * ldb : st] : T(0);
            }
        }
    };

    auto mul = [&](const T (&av)[ST][RG][RL], const T (&bv)[NT16][ST]) {
#pragma unroll
        for (int st = 0; st < ST; ++st)
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int q = 0; q < RL; ++q)
#pragma unroll
                    for (int t = 0; t < NT16; ++t)
                        acc[g][q][t] = M::op(bv[t][st], av[st][g][q], acc[g][q][t]);
    };
    // a whole chunk of a full tile: straight-line 16-byte loads; B columns
    // p >= n read column n - 1 (in range) and are zeroed after the wait
    auto loadA_full = [&](int64_t j0, T (&av)[ST][RG][RL]) {
        const T* base = A + row0 + RL * rl + (j0 + ST * kk) * lda;
#pragma unroll
        for (int st = 0; st < ST; ++st)
#pragma unroll
            for (int g = 0; g < RG; ++g)
                load_run<T, RL, LINE>(base + st * lda + 16 * RL * g, RL, true, av[st][g]);
    };
    auto loadB_full = [&](int64_t j0, T (&bv)[NT16][ST]) {
        typedef typename VecOf<T, BW>::mem V;
#pragma unroll
        for (int t = 0; t < NT16; ++t) {
            const int p = 16 * t + rl, pc = p < n ? p : n - 1;
            const int64_t jb = j0 + ST * kk;
            if (BT) {
#pragma unroll
                for (int st = 0; st < ST; ++st) bv[t][st] = B[(jb + st) * ldb + pc];
                continue;
            }
            const T* __restrict__ src = B + jb + (int64_t)pc * ldb;
#pragma unroll
            for (int h = 0; h < ST / BW; ++h) {
                const V v = *reinterpret_cast<const V*>(src + h * BW);
#pragma unroll
                for (int e = 0; e < BW; ++e) bv[t][h * BW + e] = v[e];
            }
        }
    };
    auto mul_live = [&](const T (&av)[ST][RG][RL], const T (&bv)[NT16][ST]) {
        T bz[NT16][ST];
#pragma unroll
        for (int t = 0; t < NT16; ++t)
#pragma unroll
            for (int st = 0; st < ST; ++st) bz[t][st] = 16 * t + rl < n ? bv[t][st] : T(0);
        mul(av, bz);
    };

    // the last columns of a full tile, fewer than a chunk: loads at clamped
    // columns, zeroed beyond wk1 (A too: 0 * inf would be NaN)
    auto loadA_tail = [&](int64_t j0, T (&av)[ST][RG][RL]) {
        const T* base = A + row0 + RL * rl;
#pragma unroll
        for (int st = 0; st < ST; ++st) {
            const int64_t j = j0 + ST * kk + st;
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                load_run<T, RL, LINE>(base + (j < wk1 ? j : wk1 - 1) * lda + 16 * RL * g, RL, true,
                                av[st][g]);
#pragma unroll
                for (int q = 0; q < RL; ++q) av[st][g][q] = j < wk1 ? av[st][g][q] : T(0);
            }
        }
    };

    // Whole chunks: the next chunk held in flight across the waits for
    // this one (the scheduling barriers stop the compiler from sinking its
    // loads below them; with the bounds branches of the general loop, the
    // waits after each join counted nothing as in flight and drained every
    // load).  Not for the tall tiles (RG = 4), whose two chunks do not fit
    // the register budget.
    if (PF && RG <= 2 && pf && full && wk1 - wk0 >= CW) {
        const int ng = (int)((wk1 - wk0) / CW);
        T aa[ST][RG][RL], ab[ST][RG][RL], ba[NT16][ST], bb[NT16][ST];
        loadB_full(wk0, ba);
        loadA_full(wk0, aa);
        int gc = 0;
        for (; gc + 2 < ng; gc += 2) {
            loadB_full(wk0 + CW * (gc + 1), bb);
            loadA_full(wk0 + CW * (gc + 1), ab);
            __builtin_amdgcn_sched_barrier(0);
            mul_live(aa, ba);
            loadB_full(wk0 + CW * (gc + 2), ba);
            loadA_full(wk0 + CW * (gc + 2), aa);
            __builtin_amdgcn_sched_barrier(0);
            mul_live(ab, bb);
            flush_at(gc + 2);
        }
        if (gc + 1 < ng) {
            loadB_full(wk0 + CW * (gc + 1), bb);
            loadA_full(wk0 + CW * (gc + 1), ab);
            __builtin_amdgcn_sched_barrier(0);
            mul_live(aa, ba);
            mul_live(ab, bb);
        } else {
            mul_live(aa, ba);
        }
        flush_at(ng);
        if (wk0 + (int64_t)CW * ng < wk1) {
            loadB(wk0 + (int64_t)CW * ng, ba);
            loadA_tail(wk0 + (int64_t)CW * ng, aa);
            mul(aa, ba);
        }
    } else if (wk1 > wk0) {
        const int ng = (int)((wk1 - wk0 + CW - 1) / CW);
        T av[ST][RG][RL], bv[NT16][ST];
        if (PF) {
            loadA(wk0, av);
            loadB(wk0, bv);
        }
        for (int gc = 0; gc < ng; ++gc) {
            T an[ST][RG][RL], bn[NT16][ST];
            if (!PF) {
                loadA(wk0 + CW * gc, av);
                loadB(wk0 + CW * gc, bv);
            } else if (gc + 1 < ng) {
                loadA(wk0 + CW * (gc + 1), an);
                loadB(wk0 + CW * (gc + 1), bn);
            }
            mul(av, bv);
            if (full) flush_at(gc + 1);
            if (PF) {
#pragma unroll
                for (int st = 0; st < ST; ++st)
#pragma unroll
                    for (int g = 0; g < RG; ++g)
#pragma unroll
                        for (int q = 0; q < RL; ++q) av[st][g][q] = an[st][g][q];
#pragma unroll
                for (int t = 0; t < NT16; ++t)
#pragma unroll
                    for (int st = 0; st < ST; ++st) bv[t][st] = bn[t][st];
            }
        }
    }

    if constexpr (FL) {
#pragma unroll
        for (int i = 0; i < NA; ++i) reinterpret_cast<Flat&>(acc)[i] += tot[i];
    }
    nn_finish<T, NP, WK, TR, PG>(m, n, C, ldc, beta, tile, row0, s, nsl, part,
                                 reinterpret_cast<double*>(smem), [&](int pg, double* red) {
        const int t = pg / 16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int pp = 16 * t + M::mrow(kk, r) - pg;
            if (pp >= 0 && pp < PG) {
#pragma unroll
                for (int g = 0; g < RG; ++g)
#pragma unroll
                    for (int q = 0; q < RL; ++q)
                        red[(w * PG + pp) * TR + 16 * RL * g + RL * rl + q] =
                            (double)acc[g][q][t][r];
            }
        }
    });
}

// Resident workgroups per CU of a kernel instance (queried once).
template <typename K>
static int occupancy(K kernel, int threads) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, 0) != hipSuccess || nb < 1)
        nb = 1;
    return nb;
}

struct NNInstance {
    const void* fn;
    const void* fn_bt;      // the same for a row-major B
    int tile_rows;
    int chunk;        // columns per chunk of a wavefront
    int occ;          // resident workgroups per CU
    const char* name; // as profilers print the kernel
};

// LINE: every column of A starts on a 128-byte line.  Otherwise vertically
// neighbouring tiles share a line of every column, which both fetch unless
// the second finds it in a cache: neighbouring tiles run on one XCD then, and
// A's loads are not non-temporal.  FP32, n = 5, A 10007 x 9973: 82 us, 73 so;
// FP32 20011^2, n = 8: 302 and 283; FP64 7777 x 6001, n = 12: 75 and 68.
// Columns on 64 bytes of a tall matrix with few of them take it as well
// (aligned() in the dispatch): 1000000 x 64, n = 1: FP64 98 us without, 88
// with; FP32 541440 x 256, n = 16: 140 and 132; but 5000^2: 27 and 29.
// Line-aligned columns keep the workgroups' round-robin order (FP32 16384^2
// ran 2.5 % slower with neighbours on one XCD, others within 1.5 % either way).
template <typename T, int NT16, int RG, int ST, bool LINE>
static NNInstance nn_instance() {
    static const int occ = occupancy(tsm2r_nn_kernel<T, NT16, RG, ST, 4, LINE, false>, 256);
    static char name[80];
    static const bool named =
        std::snprintf(name, sizeof name, "tsm2r_nn_kernel<%s, %d, %d, %d, 4, %s, false, %s>",
                      sizeof(T) == 8 ? "double" : "float", NT16, RG, ST, LINE ? "true" : "false",
                      TSM2X_NN_PREFETCH ? "true" : "false") > 0;
    (void)named;
    return NNInstance{(const void*)tsm2r_nn_kernel<T, NT16, RG, ST, 4, LINE, false>,
                      (const void*)tsm2r_nn_kernel<T, NT16, RG, ST, 4, LINE, true>,
                      16 * (16 / (int)sizeof(T)) * RG, 4 * ST, occ, name};
}

// n <= 32: two tile heights per type, 16*RL*2 rows with 16-column chunks, and twice
// the rows with 8-column chunks.  Both keep 8 KB of A in flight per wavefront.
template <bool LINE>
static bool nn_pick(int dtype, int np, bool tall, NNInstance* out) {
    if (np > 32) {
        // half of a chunk (double) or of a tile (float) leaves two wavefronts
        // per SIMD room for the sums of 64 columns, so that one's matrix
        // instructions run behind the other's loads: 20480^2, n = 64, FP64 992 us
        // with whole ones at one wavefront, 946 so; FP32 587 and 551
        if (dtype == DT_F64)
            *out = np == 48 ? nn_instance<double, 3, 2, 2, LINE>() : nn_instance<double, 4, 2, 2, LINE>();
        else if (dtype == DT_F32)
            *out = np == 48 ? nn_instance<float, 3, 1, 4, LINE>() : nn_instance<float, 4, 1, 4, LINE>();
        return dtype == DT_F64 || dtype == DT_F32;
    }
    if (dtype == DT_F64) {
        if (tall)
            *out = np <= 16 ? nn_instance<double, 1, 4, 2, LINE>() : nn_instance<double, 2, 4, 2, LINE>();
        else
            *out = np <= 16 ? nn_instance<double, 1, 2, 4, LINE>() : nn_instance<double, 2, 2, 4, LINE>();
        return true;
    }
    if (dtype == DT_F32) {
        if (tall)
            *out = np <= 16 ? nn_instance<float, 1, 4, 2, LINE>() : nn_instance<float, 2, 4, 2, LINE>();
        else
            *out = np <= 16 ? nn_instance<float, 1, 2, 4, LINE>() : nn_instance<float, 2, 2, 4, LINE>();
        return true;
    }
    return false;
}

static inline int64_t cdiv64(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Grid of the TSM2R kernel.  Measured on gfx950, the streaming rate peaks when
// about 15/8 workgroups (7.5 wavefronts, 8 KB of A in flight each) are
// resident per CU: fewer leave HBM latency uncovered, more add concurrent
// streams without adding bandwidth, and a grid that leaves some CUs with one
// workgroup more than others runs at the pace of those CUs.  For each tile
// height the k split S is the one that brings tiles * S closest to that
// target; the tile height whose grid lands closer wins, ties going to fewer
// slices (longer streams per wavefront).  A pin from the caller (an
// autotuner) replaces either choice.
//
// With the next chunk held in flight (tsm2r_nn_kernel, pf) one workgroup per
// CU streams faster than 15/8 without it: where the shorter tiles can fill
// 7/8 to all of the CUs exactly once (tiles * S in [7/8, 1] x CUs), that plan
// is taken (A 10240^2 to 30720^2, n = 2..32: 0 to +14 %; grids of 320 on 256
// CUs, two rounds with a third of the CUs holding two, lost 14-24 %, and are
// never formed).  Where neither rule fills 7/8 of the CUs, for the 64 columns
// per wavefront or the 4 % for the partials, the split goes on to two chunks
// per wavefront: idle CUs cost more than partials do (FP32 3001^2, n = 20, 24
// workgroups 60 us, 240 18; 512 x 28032, n = 8, 136 and 252: 33 and 17; FP64
// 256 x 28032, n = 24, 136 and 252: 24 and 22).  pf is also on for n > 16 and
// FP32 with n <= 4, with any grid (tsm2r_nn_kernel), and for every grid of at
// most one workgroup per CU (FP64 4096^2, n = 8, 192 workgroups: 42 us without,
// 26 with).
static int nn_pf(int64_t n, int dtype, int tall, int64_t W, int cus) {
    if (tall) return 0;
    if (n > 16 || (dtype == DT_F32 && n <= 4)) return 1;
    return W <= cus ? 1 : 0;
}

int plan_tsm2r(int64_t m, int64_t k, int64_t n, int dtype, int cus, bool line, NNPlan* P,
               const NNPin* pin, bool fine) {
    // partial sums are stored at the kernel's padded width (16, 32, 48 or 64)
    const int np = (int)((n + 15) / 16) * 16;
    const int es = dtype == DT_F64 ? 8 : 4;
    const int WK = 4;
    int64_t target = (int64_t)cus * 15 / 8;
    const char* ft = std::getenv("TSM2X_NN_TARGET");
    if (ft && *ft && std::strtoll(ft, nullptr, 10) > 0) target = std::strtoll(ft, nullptr, 10);
    const char* fs = std::getenv("TSM2X_NN_S");
    const int64_t s_force = (fs && *fs) ? std::strtoll(fs, nullptr, 10) : 0;
    const char* fh = std::getenv("TSM2X_NN_TALL");     // 0 or 1 forces a tile height
    int64_t tall_force = (fh && *fh) ? std::strtoll(fh, nullptr, 10) : -1;
    int64_t s_pin = s_force;
    if (pin && pin->S > 0) s_pin = pin->S;
    if (pin && pin->tall >= 0) tall_force = pin->tall;

    if (np > 32) {
        // bound by the matrix cores: the split whose grid lasts least, counting
        // full rounds of one workgroup per CU, two chunks to fill a
        // wavefront's pipeline and the partials, written and read.  Only the
        // least S of each slice length is looked at (of up to 2048 splits in
        // turn, three divisions each, the query of FP32 33 x 1048576, n = 33
        // took 56 us of host time; 14 so)
        NNInstance I{};
        if (!(line ? nn_pick<true>(dtype, np, false, &I) : nn_pick<false>(dtype, np, false, &I)))
            return 1;
        const int64_t tiles = cdiv64(m, I.tile_rows), gran = (int64_t)WK * I.chunk;
        const int64_t chunks = cdiv64(k, gran);
        double best = 0;
        for (int64_t S = 1; S == 1 || (S <= k / (2 * gran) && tiles * S <= 8 * (int64_t)cus);) {
            const int64_t lc = cdiv64(chunks, S), ks = lc * gran, s = cdiv64(k, ks);
            const int64_t W = tiles * s;
            const double len = (double)lc;
            double t = (double)m * k * es * ((double)(cdiv64(W, cus) * cus) / (double)W) * (len + 2) / len;
            // fewer rows than a tile: no prefetch, one workgroup per CU is too few
            // (33 x 1000000, n = 33: FP64 243 us with up to 256, 165 with 512; FP32
            // 137 and 104)
            if (m < I.tile_rows && W <= cus) t *= 1.25;
            if (s > 1) t += 30e6 + (double)s * m * n * 16;
            if (S == 1 || t < best) {
                best = t;
                P->S = (int)s;
                P->kslice = ks;
            }
            if (lc == 1) break;
            S = cdiv64(chunks, lc - 1);
        }
        P->np = np;
        P->fn = I.fn;
        P->fn_bt = I.fn_bt;
        P->name = I.name;
        P->tiles = tiles;
        P->tile_rows = I.tile_rows;
        P->ws = P->S > 1 ? (size_t)tiles * P->S * np * I.tile_rows * 8 : 0;
        P->tall = 0;
        P->occ = I.occ;
        P->pf = 1;
        return 0;
    }
    bool found = false;
    double best_dev = 0;
    for (int tall = 0; tall < 2; ++tall) {
        if (tall_force >= 0 && tall != (int)tall_force) continue;
        NNInstance I{};
        if (!(line ? nn_pick<true>(dtype, np, tall, &I) : nn_pick<false>(dtype, np, tall, &I)))
            return 1;
        const int64_t tiles = cdiv64(m, I.tile_rows);
        const int64_t slots = (int64_t)cus * I.occ;
        const int64_t tgt = target < slots ? target : slots;
        int64_t S = (tgt + tiles / 2) / tiles;                        // nearest integer
        const int64_t s_len = k / (WK * 64);                          // >= 64 columns per wave
        const int64_t s_cost = (k * es) / ((int64_t)np * 200);         // partials <= ~4 % of A
        if (S > s_len) S = s_len;
        if (S > s_cost) S = s_cost;
        if (S < 1) S = 1;
        if (s_pin > 0) S = s_pin;
        const int64_t gran = (int64_t)WK * I.chunk;
        int64_t ks = cdiv64(k, S);
        ks = cdiv64(ks, gran) * gran;
        S = cdiv64(k, ks);
        if (S < 1) S = 1;
        const int64_t W = tiles * S;
        const double dev = (double)(W > tgt ? W - tgt : tgt - W) / (double)tgt;
        // a later (taller) instance must be clearly better to replace the first
        if (!found || dev < best_dev - 0.02) {
            found = true;
            best_dev = dev;
            P->np = np;
            P->fn = I.fn;
            P->fn_bt = I.fn_bt;
            P->name = I.name;
            P->tiles = tiles;
            P->tile_rows = I.tile_rows;
            P->kslice = ks;
            P->S = (int)S;
            P->ws = S > 1 ? (size_t)tiles * S * np * I.tile_rows * 8 : 0;
            P->tall = tall;
            P->occ = I.occ;
        }
    }
    if (!found) return 1;
    // one workgroup per CU with the prefetch, unless the caller or an
    // override fixed the plan
    const bool free_plan = s_pin <= 0 && tall_force < 0 && !(ft && *ft);
    if (free_plan) {
        NNInstance I{};
        if (line ? nn_pick<true>(dtype, np, false, &I) : nn_pick<false>(dtype, np, false, &I)) {
            const int64_t tiles = cdiv64(m, I.tile_rows);
            const int64_t gran = (int64_t)WK * I.chunk;
            // the split that fills the CUs once, its cost capped as above,
            // or (few) at least two chunks per wavefront and no more bytes
            // of partials, written and read, than A has
            auto split = [&](bool few) {
                int64_t S = cus / tiles;
                const int64_t s_len = few ? k / (2 * gran) : k / (WK * 64);
                const int64_t s_cost = few ? (k * es) / (n * 16) : (k * es) / ((int64_t)np * 200);
                if (S > s_len) S = s_len;
                if (S > s_cost) S = s_cost;
                return S < 1 ? 1 : S;
            };
            auto slice = [&](int64_t S) { return cdiv64(cdiv64(k, S), gran) * gran; };
            int64_t ks = slice(split(false)), W = tiles * cdiv64(k, ks);
            bool take = W <= cus && 8 * W >= 7 * (int64_t)cus;
            const int64_t have = P->tiles * P->S;
            if (fine && !take && 8 * have < 7 * (int64_t)cus) {
                // the plan so far leaves CUs idle
                ks = slice(split(true));
                W = tiles * cdiv64(k, ks);
                // time of either in bytes at the streaming rate: its share of
                // the CUs, two chunks to fill the pipeline, the partials, and
                // the second launch if it is a new one (4 to 5 us)
                const double a = 1.05 * cus * (double)m * k * es;
                const double len = (double)ks / gran;
                const double cost = a / W * (len + 2) / len + (double)m * n * 16 * cdiv64(k, ks) +
                                    (P->S == 1 && ks < k ? 30e6 : 0.0);
                take = W <= cus && (W > have || P->tall) && cost < a / have;
            }
            // float sums of 17..32 columns are not flushed (tsm2r_nn_kernel):
            // off the 128-byte lines no longer chains than the plan without
            // the prefetch has.  With them n = 32 would run 7 to 15 % faster
            // (30004 x 30000 665 and 618 us, 16004^2 208 and 182) at an error
            // half as large again (16004^2: 5.7e-7 and 8.0e-7); on the lines
            // the plan has them
            if (dtype == DT_F32 && np == 32 && !line && cdiv64(k, ks) < P->S) take = false;
            if (take) {
                P->fn = I.fn;
                P->fn_bt = I.fn_bt;
                P->name = I.name;
                P->tiles = tiles;
                P->tile_rows = I.tile_rows;
                P->kslice = ks;
                P->S = (int)cdiv64(k, ks);
                P->ws = P->S > 1 ? (size_t)tiles * P->S * np * I.tile_rows * 8 : 0;
                P->tall = 0;
                P->occ = I.occ;
            }
        }
    }
    P->pf = nn_pf(n, dtype, P->tall, P->tiles * P->S, cus);
    return 0;
}

int launch_tsm2r_nn(const LaunchNN& L, int dtype, hipStream_t st) {
    int n32 = (int)L.n;
    // the next chunk held in flight (see tsm2r_nn_kernel) where it measured
    // faster (the plan's choice, plan_tsm2r): one workgroup per CU; n > 16,
    // where the matrix cores' share of a chunk is largest, +15-25 % (FP32 at
    // 32768^2, n = 32: 5.1 -> 6.0 TB/s); FP32 with n <= 4, +2-9 %; with the
    // 15/8 grid and n = 8, 16 it measured -5..+1 %.  TSM2X_NN_PF=0/1
    // overrides (measurement).
    const char* pfe = std::getenv("TSM2X_NN_PF");
    int pf = (pfe && *pfe) ? (int)std::strtol(pfe, nullptr, 10) : L.pf;
    double beta = L.beta;
    void* args[] = {(void*)&L.m,   (void*)&L.k,      (void*)&n32,    (void*)&L.A,
                    (void*)&L.lda, (void*)&L.B,      (void*)&L.ldb,  (void*)&L.C,
                    (void*)&L.ldc, (void*)&L.kslice, (void*)&L.part, (void*)&pf,
                    (void*)&beta};
    hipError_t e;
    {
        LaunchTimer timer(L.fn, st);
        e = hipLaunchKernel(L.fn, dim3((unsigned)L.tiles, (unsigned)L.S), dim3(256), args, 0, st);
    }
    if (e != hipSuccess) return 1;
    if (L.S > 1)
        return launch_split_reduce(dtype, L.tiles, L.S, L.np, L.tile_rows, L.m, (int)L.n, L.part,
                                   L.C, L.ldc, L.beta, st);
    return 0;
}

}  // namespace tsm
