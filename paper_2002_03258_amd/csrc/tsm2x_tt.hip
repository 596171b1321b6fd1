// The product of two tall matrices held by rows on gfx950: O (ma x n) =
// X^T * Y with X (R x ma) and Y (R x n), ma, n <= 32, R large -- C = A*B for a
// column-major A of few rows and many columns (A = X^T), the shape
// tsmttsm() gives for row-major matrices.
//
// On the matrix cores with the long dimension as the contraction: D[16 x 16]
// += S[16 x 4] * T[4 x 16], S[rl][kk] = X[r, 16 a + rl] and T[kk][rl] =
// Y[r, 16 b + rl], one row r per kk.  Sixteen lanes read sixteen consecutive
// values of a row, so an instruction reads whole rows of a row-major X and Y
// in the operand order as they stand: no transposed copy of Y, nothing
// through LDS.  (The TSM2R kernel, which tiles the rows of C, keeps 4 to 8 of
// 64 lanes on such a matrix.)
//
// A column-major Y (YROW false) gives each lane RL consecutive rows of one
// column in one 16-byte load; the steps then take the rows in that order.
//
// Memory bound: 2 * 32 flops per loaded value at most.  A wavefront keeps one
// step of 4 * U rows in flight while it multiplies the step before; workgroups
// of 8 wavefronts, two per CU, take steps in turn, and their double partials
// are added in order by split_reduce_kernel.  R = 4194304, ma = n = 16, both
// row-major: FP32 93 us (5.8 TB/s), FP64 173 us (6.2); rows of few values
// leave lanes idle (ma = n = 3: 1.7 and 2.2 TB/s).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tsm2x_device.h"
#include "tsm2x_internal.h"

namespace tsm {

constexpr int TT_WK = 8;     // wavefronts per workgroup
constexpr int TT_U = 8;      // steps of 4 rows in flight per wavefront

template <typename T, int NTA, int NTB, bool YROW>
__global__ __launch_bounds__(WAVE * TT_WK) void tt_kernel(
    int64_t R, int ma, int n, const T* __restrict__ X, int64_t ldx, const T* __restrict__ Y,
    int64_t ldy, T* __restrict__ O, int64_t ldo, double* __restrict__ part, double beta) {
    typedef Mfma<T> M;
    typedef typename M::acc Acc;
    constexpr int RL = 16 / (int)sizeof(T);
    constexpr int U = TT_U, SR = 4 * U;      // rows per step
    static_assert(U % RL == 0, "whole 16-byte runs of a column-major Y");
    __shared__ double red[TT_WK][WAVE][4 * NTB];

    const int lane = threadIdx.x & (WAVE - 1);
    const int rl = lane & 15, kk = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);

    // columns beyond ma and n read the last one (their outputs are not stored)
    int xa[NTA], yb[NTB];
#pragma unroll
    for (int a = 0; a < NTA; ++a) xa[a] = 16 * a + rl < ma ? 16 * a + rl : ma - 1;
#pragma unroll
    for (int b = 0; b < NTB; ++b) yb[b] = 16 * b + rl < n ? 16 * b + rl : n - 1;
    // row of a step that lane group kk takes in instance u
    auto row = [&](int u) { return YROW ? 4 * u + kk : 4 * RL * (u / RL) + RL * kk + u % RL; };

    Acc acc[NTA][NTB];
#pragma unroll
    for (int a = 0; a < NTA; ++a)
#pragma unroll
        for (int b = 0; b < NTB; ++b) acc[a][b] = Acc{0, 0, 0, 0};

    auto load = [&](int64_t rb, T (&x)[U][NTA], T (&y)[U][NTB]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T* xr = X + (rb + row(u)) * ldx;
#pragma unroll
            for (int a = 0; a < NTA; ++a) x[u][a] = xr[xa[a]];
            if (YROW) {
                const T* yr = Y + (rb + row(u)) * ldy;
#pragma unroll
                for (int b = 0; b < NTB; ++b) y[u][b] = yr[yb[b]];
            } else if (u % RL == 0) {
                typedef typename VecOf<T, RL>::mem V;
#pragma unroll
                for (int b = 0; b < NTB; ++b) {
                    const V v = *reinterpret_cast<const V*>(Y + rb + row(u) + yb[b] * ldy);
#pragma unroll
                    for (int q = 0; q < RL; ++q) y[u + q][b] = v[q];
                }
            }
        }
    };
    // the last rows: clamped, both operands zero beyond R (0 * inf is NaN)
    auto load_tail = [&](int64_t rb, T (&x)[U][NTA], T (&y)[U][NTB]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = rb + row(u);
            const int64_t rc = r < R ? r : R - 1;
#pragma unroll
            for (int a = 0; a < NTA; ++a) {
                const T v = X[rc * ldx + xa[a]];
                x[u][a] = r < R ? v : T(0);
            }
#pragma unroll
            for (int b = 0; b < NTB; ++b) {
                const T v = YROW ? Y[rc * ldy + yb[b]] : Y[rc + yb[b] * ldy];
                y[u][b] = r < R ? v : T(0);
            }
        }
    };
    auto mul = [&](const T (&x)[U][NTA], const T (&y)[U][NTB]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a < NTA; ++a)
#pragma unroll
                for (int b = 0; b < NTB; ++b) acc[a][b] = M::op(x[u][a], y[u][b], acc[a][b]);
    };

    constexpr bool FL = sizeof(T) == 4;
    constexpr int NA = NTA * NTB;
    typedef Acc Flat[NA];
    Acc tot[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) tot[i] = Acc{0, 0, 0, 0};
    int done = 0;

    // whole steps go round the wavefronts of the grid; the next one is in
    // flight while this one is multiplied (the barriers keep the compiler
    // from sinking its loads below the waits)
    const int64_t nst = R / SR;
    const int64_t stride = (int64_t)gridDim.x * TT_WK;
    const int64_t first = (int64_t)blockIdx.x * TT_WK + w;
    T x0[U][NTA], y0[U][NTB], x1[U][NTA], y1[U][NTB];
    if (first < nst) {
        load(first * SR, x0, y0);
        int64_t i = first;
        for (; i + 2 * stride < nst; i += 2 * stride) {
            load((i + stride) * SR, x1, y1);
            __builtin_amdgcn_sched_barrier(0);
            mul(x0, y0);
            load((i + 2 * stride) * SR, x0, y0);
            __builtin_amdgcn_sched_barrier(0);
            mul(x1, y1);
            done += 2;
            if (FL && done % (FLUSH / 4) == 0)
                flush<NA>(reinterpret_cast<Flat&>(acc), reinterpret_cast<Flat&>(tot));
        }
        if (i + stride < nst) {
            load((i + stride) * SR, x1, y1);
            __builtin_amdgcn_sched_barrier(0);
            mul(x0, y0);
            mul(x1, y1);
        } else {
            mul(x0, y0);
        }
    }
    // the wavefront next in turn takes the remainder
    if (nst * SR < R && nst % stride == first) {
        load_tail(nst * SR, x0, y0);
        mul(x0, y0);
    }
    if (FL) {
#pragma unroll
        for (int i = 0; i < NA; ++i) reinterpret_cast<Flat&>(acc)[i] += tot[i];
    }

#pragma unroll
    for (int a = 0; a < NTA; ++a) {
        if (a > 0) __syncthreads();            // red is reused
        tn_finish<T, NTB, TT_WK>(ma, n, O, ldo, beta, 16 * a, 0, blockIdx.x, gridDim.x, part, red, acc[a],
                                 [](int kq, int r) { return Mfma<T>::mrow(kq, r); });
    }
}

// Workgroups: a step for each wavefront at least, two workgroups per CU at most.
static int tt_blocks(int64_t R, int cus) {
    const int64_t need = (R + 4 * TT_U * TT_WK - 1) / (4 * TT_U * TT_WK);
    const int64_t most = 2 * (int64_t)cus;
    return (int)(need < most ? need : most);
}

size_t tt_ws(int64_t R, int ma, int n, int cus) {
    const int S = tt_blocks(R, cus);
    return S > 1 ? (size_t)S * (ma <= 16 ? 1 : 2) * (n <= 16 ? 1 : 2) * 256 * 8 : 0;
}

const char* tt_name(int ma, int n, int dtype) {
    static const char* const names[2][2][2] = {
        {{"tt_kernel<double, 1, 1, false>", "tt_kernel<double, 1, 2, false>"},
         {"tt_kernel<double, 2, 1, false>", "tt_kernel<double, 2, 2, false>"}},
        {{"tt_kernel<float, 1, 1, false>", "tt_kernel<float, 1, 2, false>"},
         {"tt_kernel<float, 2, 1, false>", "tt_kernel<float, 2, 2, false>"}}};
    return names[dtype == DT_F64 ? 0 : 1][ma <= 16 ? 0 : 1][n <= 16 ? 0 : 1];
}

template <typename T, int NTA, int NTB>
static int tt_launch(const LaunchTT& L, hipStream_t st) {
    const int S = tt_blocks(L.R, L.cus);
    const dim3 g((unsigned)S), b(WAVE * TT_WK);
    if (L.y_rowmajor)
        TSM_LAUNCH((tt_kernel<T, NTA, NTB, true>), g, b, 0, st, L.R, L.ma, L.n, (const T*)L.X,
                   L.ldx, (const T*)L.Y, L.ldy, (T*)L.O, L.ldo, L.part, L.beta);
    else
        TSM_LAUNCH((tt_kernel<T, NTA, NTB, false>), g, b, 0, st, L.R, L.ma, L.n, (const T*)L.X,
                   L.ldx, (const T*)L.Y, L.ldy, (T*)L.O, L.ldo, L.part, L.beta);
    if (hipGetLastError() != hipSuccess) return 1;
    if (S == 1) return 0;
    return launch_split_reduce(sizeof(T) == 8 ? DT_F64 : DT_F32, NTA, S, 16 * NTB, 16, L.ma, L.n,
                               L.part, L.O, L.ldo, L.beta, st);
}

template <typename T>
static int tt_dispatch(const LaunchTT& L, hipStream_t st) {
    if (L.ma <= 16) return L.n <= 16 ? tt_launch<T, 1, 1>(L, st) : tt_launch<T, 1, 2>(L, st);
    return L.n <= 16 ? tt_launch<T, 2, 1>(L, st) : tt_launch<T, 2, 2>(L, st);
}

int launch_tt(const LaunchTT& L, int dtype, hipStream_t st) {
    if (dtype == DT_F64) return tt_dispatch<double>(L, st);
    if (dtype == DT_F32) return tt_dispatch<float>(L, st);
    return 1;
}

}  // namespace tsm
