// Several sweeps of the smoother in one launch, for matrices so small that a
// sweep of its own costs a launch (3.7 us on the host, 3.2 us on the device)
// and little else.
//
// Diagonal slices say how far a row reaches: a row of L_s reads at most wL rows
// back, a row of U_s at most wU rows on.  So a workgroup that owns the rows
// [t0, t1) can run the sweeps y_1 .. y_mL by itself if it starts from the rows
// [t0 - (mL - 1) wL, t1) and gives up wL of them with every sweep, and likewise
// the U loop from rows behind its own: the overlap is computed twice and
// nothing is exchanged.  The iterates stand in LDS.  Each row's sum takes its
// slots in the order of the sweep kernels and in the same precisions, so
// results are theirs bit for bit.
//
// A matrix that fits one workgroup takes one launch for the whole call.  Else
// the L loop (with or without the residual before it) and the U loop with the
// update take a launch each; the residual reads x of other workgroups' rows, so
// it is never in the launch that writes x.
#include "internal.h"

#pragma clang fp contract(off)

namespace silu {
namespace {

__device__ __forceinline__ int clamped(int c, int n) { return min(max(c, 0), n - 1); }

// sum_k val(row i, slot k) * get(i + d_k), slots ascending, up to SLOTS loads in
// flight.  A column outside the matrix only occurs on a slot whose value is 0.
template <class AT, class VT, class Get>
__device__ __forceinline__ AT slots_sum(const TileMatrix &M, int i, int n, Get get)
{
    constexpr int SLOTS = 8;
    const VT *v0 = (const VT *)M.val + diag_slot(i, 0, M.u);
    AT s = (AT)0;
    for (int k0 = 0; k0 < M.u; k0 += SLOTS) {
        VT v[SLOTS];
        decltype(get(0)) x[SLOTS];
#pragma unroll
        for (int k = 0; k < SLOTS; ++k)
            if (k0 + k < M.u) { // the same in the whole workgroup
                v[k] = v0[128 * (k0 + k)];
                x[k] = get(clamped(i + M.dtab[k0 + k], n));
            }
#pragma unroll
        for (int k = 0; k < SLOTS; ++k)
            if (k0 + k < M.u) s = s + (AT)v[k] * (AT)x[k];
    }
    return s;
}

// put(i, the sum of row i) for the rows [lo, hi), over the whole workgroup (two
// or four rows a lane at a time were slower: the ranges are one to three rows
// a lane, and what is past their end is work for nothing).
template <class AT, class VT, class Get, class Put>
__device__ __forceinline__ void sweep(const TileMatrix &M, int lo, int hi, int n, Get get, Put put)
{
    for (int i = lo + (int)threadIdx.x; i < hi; i += TILE_THREADS) put(i, slots_sum<AT, VT>(M, i, n, get));
}

// The whole workgroup over rows [lo, hi).
template <class F>
__device__ __forceinline__ void rows(int lo, int hi, F f)
{
    for (int i = lo + (int)threadIdx.x; i < hi; i += TILE_THREADS) f(i);
}

// put(i, get(i)) for the rows [lo, hi), four loads in flight a lane (one: 0.9 us
// for every 1,024 rows).
template <class Get, class Put>
__device__ __forceinline__ void fetch(int lo, int hi, Get get, Put put)
{
    constexpr int DEEP = 4;
    for (int i0 = lo + (int)threadIdx.x; i0 < hi; i0 += DEEP * TILE_THREADS) {
        decltype(get(0)) v[DEEP];
#pragma unroll
        for (int j = 0; j < DEEP; ++j) v[j] = get(min(i0 + j * TILE_THREADS, hi - 1));
#pragma unroll
        for (int j = 0; j < DEEP; ++j)
            if (i0 + j * TILE_THREADS < hi) put(i0 + j * TILE_THREADS, v[j]);
    }
}

// XT: the iterates' (and factors' and sums') type: double, or float in the
// FP32-inner form, whose residual and update stay in double.
template <class XT>
__global__ void __launch_bounds__(TILE_THREADS) k_smooth_tile(TileArgs a)
{
    __shared__ double room[TILE_LDS / 8];
    const int n = a.n, t0 = (int)blockIdx.x * a.tile, t1 = min(n, t0 + a.tile);
    // r on [lo, t1), in the U loop a third buffer of iterates; two such from row bo on
    const int lo = max(0, t0 - a.back), hi = min(n, t1 + a.ahead), bo = max(0, t0 - max(0, a.back - a.wL));
    double *r = room;
    XT *buf[2] = {(XT *)(room + a.buf0), (XT *)(room + a.buf1)};
    double *x = a.x; // not restrict: the residual of the next outer step reads what this one wrote
    for (int it = 0; it < a.outer; ++it) {
        const XT *s = nullptr; // z_1 = s
        int sb = 0;            // its buffer
        if (a.lower) {
            if (a.residual && !(a.zero && it == 0))
                sweep<double, double>(
                    a.A, lo, t1, n, [&](int c) { return x[c]; }, [&](int i, double t) { r[i - lo] = a.rhs[i] - t; });
            else
                fetch(lo, t1, [&](int i) { return a.rhs[i]; }, [&](int i, double t) { r[i - lo] = t; });
            __syncthreads();
            // y_1 = r, y_k = r - Ls y_{k-1}; the last one, times D^{-1}, is s
            for (int k = 1; k <= a.m_L; ++k) {
                const bool last = k == a.m_L;
                const XT *y = buf[k & 1]; // y_{k-1}; y_1 is read from r, rounded
                XT *out = buf[(k + 1) & 1];
                if (k == 1 && !last) continue;
                const int from = max(0, t0 - (a.m_L - k) * a.wL);
                auto put = [&](int i, XT sum) {
                    XT t = (XT)r[i - lo];
                    if (k > 1) t = t - sum;
                    if (last) t = (XT)(a.dinv[i] * (double)t);
                    if (last && a.s_out) ((XT *)a.s_out)[i] = t;
                    else out[i - bo] = t;
                };
                if (k == 1) rows(from, t1, [&](int i) { put(i, (XT)0); });
                else if (k == 2) sweep<XT, XT>(a.L, from, t1, n, [&](int c) { return (XT)r[c - lo]; }, put);
                else sweep<XT, XT>(a.L, from, t1, n, [&](int c) { return y[c - bo]; }, put);
                __syncthreads();
                sb = (k + 1) & 1;
            }
            s = buf[sb];
        } else { // s as the L loop's launch left it
            fetch(lo, hi, [&](int i) { return ((const XT *)a.s_in)[i]; }, [&](int i, XT t) { buf[0][i - bo] = t; });
            __syncthreads();
            s = buf[0];
        }
        if (!a.upper) return; // then there is one outer step
        // z_k = s - Us z_{k-1}; the last one is added to x
        XT *zb[2] = {buf[1 - sb], (XT *)r};
        const XT *z = s;
        for (int k = 2; k < a.m_U; ++k) {
            XT *out = zb[k & 1];
            sweep<XT, XT>(
                a.U, t0, min(n, t1 + (a.m_U - k) * a.wU), n, [&](int c) { return z[c - bo]; },
                [&](int i, XT sum) { out[i - bo] = s[i - bo] - sum; });
            __syncthreads();
            z = out;
        }
        auto update = [&](int i, XT sum) {
            XT t = s[i - bo];
            if (a.m_U > 1) t = t - sum;
            x[i] = x[i] + (a.dcol ? a.dcol[i] : 1.0) * (double)t;
        };
        if (a.m_U > 1) sweep<XT, XT>(a.U, t0, t1, n, [&](int c) { return z[c - bo]; }, update);
        else rows(t0, t1, [&](int i) { update(i, (XT)0); });
        __syncthreads(); // x and the buffers, before the next outer step
    }
}

} // namespace

hipError_t launch_smooth_tile(const TileArgs &a, int fp32, hipStream_t s)
{
    if (a.n <= 0) return hipSuccess;
    const dim3 g((a.n + a.tile - 1) / a.tile), b(TILE_THREADS);
    if (fp32) hipLaunchKernelGGL(k_smooth_tile<float>, g, b, 0, s, a);
    else hipLaunchKernelGGL(k_smooth_tile<double>, g, b, 0, s, a);
    return hipGetLastError();
}

} // namespace silu
