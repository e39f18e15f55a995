// Vector kernels of the Krylov solver around the smoother (FGMRES with
// modified Gram-Schmidt): deterministic dot products, and the orthogonalization
// of an Arnoldi step, whose scalars stay on the device.
//
// Dot products are two-stage and always reduce in the same order: stage one
// gives each of DOT_BLOCKS workgroups a fixed contiguous chunk, each lane adds
// its strided elements in index order and the workgroup combines its lanes by
// a fixed tree; stage two adds the partial sums the same way.  The result is
// reproducible run to run (it is not the sequential sum of the definition;
// the difference is rounding).
//
// Modified Gram-Schmidt takes h_i = v_i . (w - sum_{k<i} h_k v_k) one vector
// after the other: 3 dependent launches each, 2.6 to 2.9 us a kernel where the
// vectors are short, and 5 passes over long ones.  The same numbers are the
// solution of (I + S) h = V^T w with S the strictly lower part of V^T V (whose
// row j is v_j . v_i, i < j, computed when v_j is new), since that system is
// the recurrence written out; nothing is assumed about how orthogonal V is.
// So a step takes four launches whatever its number of vectors: all products
// with w and v_j in one pass over V (k_dots), the sums and the substitution
// (k_project), w -= V h with the partial sums of w . w in a second pass
// (k_subtract), and v_{j+1} = w / ||w|| (k_normalize).  48^3 Poisson operator,
// FGMRES(30) to 1e-8 in 96 or 97 steps: 18.7 to 21.6 ms with one vector at a time,
// 6.7 ms so, 4.2 to 4.6 ms with the next direction enqueued before the wait.
#include <algorithm>

#include "internal.h"

#pragma clang fp contract(off)

namespace silu {
namespace {

constexpr int DOT_THREADS = 256;

constexpr int COMBINE_MAX = 32; // vectors of one k_combine launch (their coefficients go by value)
struct Coeffs {
    double y[COMBINE_MAX];
};

__device__ __forceinline__ double block_sum(double v, double *lds)
{
    const int t = (int)threadIdx.x;
    lds[t] = v;
    __syncthreads();
    for (int s = DOT_THREADS / 2; s > 0; s >>= 1) {
        if (t < s) lds[t] = lds[t] + lds[t + s];
        __syncthreads();
    }
    return lds[0];
}

__global__ void __launch_bounds__(DOT_THREADS) k_dot_partial(int64_t n, const double *__restrict__ a,
                                                             const double *__restrict__ b, double *__restrict__ part)
{
    __shared__ double lds[DOT_THREADS];
    const int64_t chunk = (n + DOT_BLOCKS - 1) / DOT_BLOCKS;
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    double s = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += DOT_THREADS) s = s + a[i] * b[i];
    const double tot = block_sum(s, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// out[0] = the sum of the partials (sqrt of it with take_sqrt)
__global__ void __launch_bounds__(DOT_THREADS) k_dot_final(const double *__restrict__ part, double *__restrict__ out,
                                                           int take_sqrt)
{
    __shared__ double lds[DOT_THREADS];
    double s = 0.0;
    for (int i = (int)threadIdx.x; i < DOT_BLOCKS; i += DOT_THREADS) s = s + part[i];
    const double tot = block_sum(s, lds);
    if (threadIdx.x == 0) out[0] = take_sqrt ? sqrt(tot) : tot;
}

// part[(2 i + s) nx + x] = the share of workgroup x in a . v_i (s = 0) and
// b . v_i (s = 1) for the DOTS_VECS vectors from DOTS_VECS * blockIdx.y on;
// nx = gridDim.x.  a and b are read once for that many vectors.
constexpr int DOTS_VECS = 8;
constexpr int DOTS_PITCH = DOT_THREADS + 16; // LDS row of one sum (the 16 spread the columns over the banks)
__global__ void __launch_bounds__(DOT_THREADS) k_dots(int64_t n, const double *__restrict__ V, int64_t stride, int count,
                                                      const double *__restrict__ a, const double *__restrict__ b,
                                                      double *__restrict__ part)
{
    __shared__ double lds[2 * DOTS_VECS * DOTS_PITCH];
    const int t = (int)threadIdx.x, i0 = (int)blockIdx.y * DOTS_VECS, nv = min(DOTS_VECS, count - i0);
    const double *v0 = V + (int64_t)i0 * stride;
    double sa[DOTS_VECS], sb[DOTS_VECS];
#pragma unroll
    for (int k = 0; k < DOTS_VECS; ++k) sa[k] = sb[k] = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * DOT_THREADS + t; e < n; e += (int64_t)gridDim.x * DOT_THREADS) {
        const double ae = a[e], be = b[e];
        if (nv == DOTS_VECS) {
            double v[DOTS_VECS];
#pragma unroll
            for (int k = 0; k < DOTS_VECS; ++k) v[k] = v0[(int64_t)k * stride + e];
#pragma unroll
            for (int k = 0; k < DOTS_VECS; ++k) {
                sa[k] = sa[k] + ae * v[k];
                sb[k] = sb[k] + be * v[k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < DOTS_VECS; ++k)
                if (k < nv) {
                    const double v = v0[(int64_t)k * stride + e];
                    sa[k] = sa[k] + ae * v;
                    sb[k] = sb[k] + be * v;
                }
        }
    }
#pragma unroll
    for (int k = 0; k < DOTS_VECS; ++k) {
        lds[(2 * k) * DOTS_PITCH + t] = sa[k];
        lds[(2 * k + 1) * DOTS_PITCH + t] = sb[k];
    }
    __syncthreads();
    // 16 lanes on each sum: 16 of its terms a lane, then the 16 lanes
    const int q = t >> 4, l = t & 15;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < DOT_THREADS / 16; ++k) s = s + lds[q * DOTS_PITCH + l + 16 * k];
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) s = s + __shfl_xor(s, off, 16);
    if (l == 0 && (q >> 1) < nv) part[((int64_t)2 * i0 + q) * gridDim.x + blockIdx.x] = s;
}

// One workgroup: dots[] = the 2 * count sums of k_dots.
__device__ void sum_dots(int count, int nx, const double *__restrict__ part, double *dots)
{
    const int lane = (int)threadIdx.x & 63;
    for (int q = (int)threadIdx.x >> 6; q < 2 * count; q += (int)blockDim.x >> 6) {
        double s = 0.0;
        for (int x = lane; x < nx; x += 64) s = s + part[(int64_t)q * nx + x];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s = s + __shfl_xor(s, off);
        if (lane == 0) dots[q] = s;
    }
    __syncthreads();
}

// What lane k (the same in the whole wave) holds.
__device__ __forceinline__ double from_lane(double v, int k)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k),
                            __builtin_amdgcn_readlane(__double2loint(v), k));
}

// Row j = count - 1 of S into St[k ld + j] = v_j . v_k (k < j: the transpose,
// so that the substitution reads neighbouring words), and h from
// (I + S) h = V^T w.  dots holds V^T w and V^T v_j, interleaved.  Up to 64
// vectors one wave substitutes: lane i holds h_i, S comes from LDS (loaded
// ahead of the sums), and a step is a few instructions with no barrier.
__global__ void __launch_bounds__(1024) k_project(int count, int nx, const double *__restrict__ part, double *dots,
                                                  double *St, int ld, double *h)
{
    __shared__ double S[64 * 64];
    const int t = (int)threadIdx.x, lane = t & 63, j = count - 1;
    if (count <= 64)
        for (int k = t >> 6; k < j; k += 16)
            if (lane > k && lane < j) S[64 * k + lane] = St[(int64_t)k * ld + lane];
    sum_dots(count, nx, part, dots); // ends in a barrier
    if (count <= 64) {
        if (t >= 64) return;
        double c = t < count ? dots[2 * t] : 0.0;
        const double own = t < j ? dots[2 * t + 1] : 0.0; // S_jt
        if (t < j) St[(int64_t)t * ld + j] = own;
        for (int k = 0; k < j; ++k) {
            const double hk = from_lane(c, k), sjk = from_lane(own, k);
            if (t > k && t < count) c = c - (t < j ? S[64 * k + t] : sjk) * hk;
        }
        if (t < count) h[t] = c;
        return;
    }
    for (int i = t; i < count; i += 1024) {
        h[i] = dots[2 * i];
        if (i < j) St[(int64_t)i * ld + j] = dots[2 * i + 1];
    }
    __syncthreads();
    for (int k = 0; k < j; ++k) {
        const double hk = h[k];
        for (int i = k + 1 + t; i < count; i += 1024) h[i] = h[i] - St[(int64_t)k * ld + i] * hk;
        __syncthreads();
    }
}

__global__ void __launch_bounds__(1024) k_dots_final(int count, int nx, const double *__restrict__ part, double *dots)
{
    sum_dots(count, nx, part, dots);
}

// Short vectors: the whole orthogonalization of a step in one workgroup, w in
// its registers, one vector after the other as modified Gram-Schmidt is
// written.  Lane t holds elements [c t, c t + c), c = ceil(n / 1024) <= E, which
// are workgroup t's chunk of k_dot_partial, and sums are added in the order of
// that pair of kernels.  host[] (pinned) receives h and the norm; zero (where
// not null) is cleared.  A vector costs two barriers and some exchanges, about
// a microsecond, and a step is one launch rather than four.  A whole FGMRES(30)
// step takes 37 us at n = 1,728 and 43 us at 4,096 so; the four kernels take 42 us
// at 5,832 and 45 us at 8,000, where this one is 15 us slower, so the line is
// drawn at four elements a lane.
template <int E>
__global__ void __launch_bounds__(DOT_BLOCKS) k_mgs_short(int n, int c, const double *__restrict__ V, int64_t stride,
                                                          int count, const double *__restrict__ w,
                                                          double *__restrict__ out, double *__restrict__ zero,
                                                          double *__restrict__ host)
{
    __shared__ double part[DOT_BLOCKS];
    __shared__ double sum;
    const int t = (int)threadIdx.x, e0 = c * t, ne = max(0, min(c, n - e0));
    double we[E], v[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        we[k] = k < ne ? w[e0 + k] : 0.0;
        v[k] = k < ne ? V[e0 + k] : 0.0;
    }
    for (int i = 0; i <= count; ++i) { // the last round is the norm
        double a[E];
#pragma unroll
        for (int k = 0; k < E; ++k) a[k] = k < ne ? 0.0 + we[k] * (i < count ? v[k] : we[k]) : 0.0;
#pragma unroll
        for (int s = E / 2; s > 0; s >>= 1)
#pragma unroll
            for (int k = 0; k < s; ++k) a[k] = a[k] + a[k + s];
        part[t] = a[0];
        __syncthreads();
        if (t < 64) {
            double u[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                u[q] = 0.0;
#pragma unroll
                for (int k = 0; k < DOT_BLOCKS; k += DOT_THREADS) u[q] = u[q] + part[t + 64 * q + k];
            }
            double s = (u[0] + u[2]) + (u[1] + u[3]);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s = s + __shfl_down(s, off);
            if (t == 0) {
                if (i == count) s = sqrt(s);
                sum = s;
                host[i] = s;
            }
        }
        // the next vector's loads go out before the wait for the sum
        double next[E];
#pragma unroll
        for (int k = 0; k < E; ++k) next[k] = i + 1 < count && k < ne ? V[(int64_t)(i + 1) * stride + e0 + k] : 0.0;
        __syncthreads();
        const double h = sum;
        if (i == count) {
#pragma unroll
            for (int k = 0; k < E; ++k)
                if (k < ne) {
                    if (h != 0.0) out[e0 + k] = we[k] / h;
                    if (zero) zero[e0 + k] = 0.0;
                }
            return;
        }
#pragma unroll
        for (int k = 0; k < E; ++k) {
            we[k] = we[k] - h * v[k];
            v[k] = next[k];
        }
    }
}

// w = w - sum_i h_i v_i, i ascending (each projection in turn, as modified
// Gram-Schmidt subtracts them); part[x] = workgroup x's share of w . w
__global__ void __launch_bounds__(DOT_THREADS) k_subtract(int64_t n, const double *__restrict__ V, int64_t stride,
                                                          int count, const double *__restrict__ h,
                                                          double *__restrict__ w, double *__restrict__ part)
{
    __shared__ double lds[DOT_THREADS];
    double s = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * DOT_THREADS + threadIdx.x; e < n; e += (int64_t)gridDim.x * DOT_THREADS) {
        double we = w[e];
        int i = 0;
        for (; i + 8 <= count; i += 8) {
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = V[(int64_t)(i + k) * stride + e];
#pragma unroll
            for (int k = 0; k < 8; ++k) we = we - h[i + k] * v[k];
        }
        for (; i < count; ++i) we = we - h[i] * V[(int64_t)i * stride + e];
        w[e] = we;
        s = s + we * we;
    }
    const double tot = block_sum(s, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// ||w|| from k_subtract's shares (every workgroup adds them up for itself, in
// the same order), out = w / ||w|| unless it is 0; host[] (pinned) receives h
// and the norm behind it.  zero (where not null) is cleared: the start of the
// next direction.
__global__ void __launch_bounds__(DOT_THREADS) k_normalize(int64_t n, const double *__restrict__ w,
                                                           const double *__restrict__ part, int nx,
                                                           const double *__restrict__ h, int count,
                                                           double *__restrict__ out, double *__restrict__ zero,
                                                           double *__restrict__ host)
{
    __shared__ double lds[DOT_THREADS];
    double s = 0.0;
    for (int x = (int)threadIdx.x; x < nx; x += DOT_THREADS) s = s + part[x];
    const double norm = sqrt(block_sum(s, lds));
    if (blockIdx.x == 0) {
        for (int i = (int)threadIdx.x; i < count; i += DOT_THREADS) host[i] = h[i];
        if (threadIdx.x == 0) host[count] = norm;
    }
    for (int64_t e = (int64_t)blockIdx.x * DOT_THREADS + threadIdx.x; e < n; e += (int64_t)gridDim.x * DOT_THREADS) {
        if (norm != 0.0) out[e] = w[e] / norm;
        if (zero) zero[e] = 0.0;
    }
}

// out = w / s  (host scalar)
__global__ void __launch_bounds__(256) k_div_host(int64_t n, const double *__restrict__ w, double s,
                                                  double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = w[i] / s;
}

// x = x + sum_i y_i z_i, i ascending (host scalars)
__global__ void __launch_bounds__(256) k_combine(int64_t n, const double *__restrict__ Z, int64_t stride, int count,
                                                 Coeffs y, double *__restrict__ x)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    double xe = x[e];
    int i = 0;
    for (; i + 4 <= count; i += 4) {
        double z[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) z[k] = Z[(int64_t)(i + k) * stride + e];
#pragma unroll
        for (int k = 0; k < 4; ++k) xe = xe + y.y[i + k] * z[k];
    }
    for (; i < count; ++i) xe = xe + y.y[i] * Z[(int64_t)i * stride + e];
    x[e] = xe;
}

inline unsigned blocks256(int64_t n) { return (unsigned)((n + 255) / 256); }

} // namespace

hipError_t launch_dot(int64_t n, const double *a, const double *b, double *part, double *out, bool take_sqrt,
                      hipStream_t s)
{
    hipLaunchKernelGGL(k_dot_partial, dim3(DOT_BLOCKS), dim3(DOT_THREADS), 0, s, n, a, b, part);
    hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(DOT_THREADS), 0, s, part, out, take_sqrt ? 1 : 0);
    return hipGetLastError();
}

int arnoldi_blocks(int64_t n)
{
    // two elements a lane up to 1,024 workgroups (4 a CU), more beyond
    return (int)std::min<int64_t>((n + 2 * DOT_THREADS - 1) / (2 * DOT_THREADS), DOT_BLOCKS);
}

hipError_t launch_dots(int64_t n, const double *V, int64_t stride, int count, const double *a, const double *b,
                       double *part, hipStream_t s)
{
    hipLaunchKernelGGL(k_dots, dim3(arnoldi_blocks(n), (count + DOTS_VECS - 1) / DOTS_VECS), dim3(DOT_THREADS), 0, s, n,
                       V, stride, count, a, b, part);
    return hipGetLastError();
}

hipError_t launch_dots_final(int64_t n, int count, const double *part, double *dots, hipStream_t s)
{
    hipLaunchKernelGGL(k_dots_final, dim3(1), dim3(1024), 0, s, count, arnoldi_blocks(n), part, dots);
    return hipGetLastError();
}

hipError_t launch_project(int64_t n, int count, const double *part, double *dots, double *St, int ld, double *h,
                          hipStream_t s)
{
    hipLaunchKernelGGL(k_project, dim3(1), dim3(1024), 0, s, count, arnoldi_blocks(n), part, dots, St, ld, h);
    return hipGetLastError();
}

hipError_t launch_mgs_short(int64_t n, const double *V, int64_t stride, int count, const double *w, double *out,
                            double *zero, double *host, hipStream_t s)
{
    if (n <= 0 || n > MGS_SHORT_MAX) return hipErrorInvalidValue;
    const int c = (int)((n + DOT_BLOCKS - 1) / DOT_BLOCKS);
    const dim3 g(1), b(DOT_BLOCKS);
    if (c == 1) hipLaunchKernelGGL(k_mgs_short<1>, g, b, 0, s, (int)n, c, V, stride, count, w, out, zero, host);
    else if (c == 2) hipLaunchKernelGGL(k_mgs_short<2>, g, b, 0, s, (int)n, c, V, stride, count, w, out, zero, host);
    else hipLaunchKernelGGL(k_mgs_short<4>, g, b, 0, s, (int)n, c, V, stride, count, w, out, zero, host);
    return hipGetLastError();
}

hipError_t launch_subtract(int64_t n, const double *V, int64_t stride, int count, const double *h, double *w,
                           double *part, hipStream_t s)
{
    hipLaunchKernelGGL(k_subtract, dim3(arnoldi_blocks(n)), dim3(DOT_THREADS), 0, s, n, V, stride, count, h, w, part);
    return hipGetLastError();
}

hipError_t launch_normalize(int64_t n, const double *w, const double *part, const double *h, int count, double *out,
                            double *zero, double *host, hipStream_t s)
{
    const int nx = arnoldi_blocks(n);
    hipLaunchKernelGGL(k_normalize, dim3(nx), dim3(DOT_THREADS), 0, s, n, w, part, nx, h, count, out, zero, host);
    return hipGetLastError();
}

hipError_t launch_combine(int64_t n, const double *Z, int64_t stride, int count, const double *y, double *x,
                          hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    for (int i = 0; i < count; i += COMBINE_MAX) {
        Coeffs c;
        const int k = std::min(COMBINE_MAX, count - i);
        std::copy(y + i, y + i + k, c.y);
        hipLaunchKernelGGL(k_combine, dim3(blocks256(n)), dim3(256), 0, s, n, Z + (int64_t)i * stride, stride, k, c, x);
    }
    return hipGetLastError();
}

hipError_t launch_div_host(int64_t n, const double *w, double d, double *out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_div_host, dim3(blocks256(n)), dim3(256), 0, s, n, w, d, out);
    return hipGetLastError();
}

} // namespace silu
