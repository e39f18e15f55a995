// ILU(0) on the device by synchronous fixed-point sweeps (the fixed-point ILU
// of Chow and Patel, which Section 7 names for computing the factorization on
// GPUs).  For every (i,j) in the pattern S of A:
//   u_ij = a_ij - sum_{k < i} l_ik u_kj            (j >= i)
//   l_ij = (a_ij - sum_{k < j} l_ik u_kj) / u_jj    (j <  i)
// A sweep evaluates every equation from the previous sweep's values; the
// products are subtracted from a_ij in ascending k (the order of row-wise
// elimination), so a sweep's values do not depend on the launch shape and the
// standstill is the row-wise ILU(0) bit for bit.  L and U live in one value
// array aligned with A's entries until they are split.
//
// G lanes of a wave work on one row (G from the mean row length), lane t on
// entries t, t + G, ...: a row's columns and values are then read and written
// as whole segments.  (One lane per row or per entry touches a cache line a
// lane instead.)
#include <algorithm>

#include "internal.h"

#pragma clang fp contract(off)

namespace silu {
namespace {

// The first row of this lane's group (the next ones follow at row_stride).
// Workgroups are renumbered so that each of the 8 XCDs takes a contiguous
// slab of rows: a row reads the upper rows of its lower neighbours, which
// then lie in the same L2.
template <int G>
__device__ __forceinline__ int64_t first_row()
{
    const unsigned nb = gridDim.x, per = nb >> 3, b = blockIdx.x;
    const unsigned wg = b < 8 * per ? (b & 7) * per + (b >> 3) : b;
    return ((int64_t)wg * 256 + threadIdx.x) / G;
}

template <int G>
__device__ __forceinline__ int64_t row_stride()
{
    return (int64_t)gridDim.x * (256 / G);
}

// The initial guess u_ij = a_ij, l_ij = a_ij / a_jj.
template <int G>
__global__ void __launch_bounds__(256) k_fp_init(int n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                 const double *__restrict__ val, const int32_t *__restrict__ dpos,
                                                 double *__restrict__ LU)
{
    const int lane = (int)threadIdx.x & (G - 1);
    for (int64_t i = first_row<G>(); i < n; i += row_stride<G>())
        for (int p = rp[i] + lane, p1 = rp[i + 1]; p < p1; p += G) {
            const int j = col[p];
            LU[p] = j < i ? val[p] / val[dpos[j]] : val[p];
        }
}

// What the lane at byte address addr / 4 of the wave holds.
__device__ __forceinline__ int from(int addr, int v) { return __builtin_amdgcn_ds_bpermute(addr, v); }

__device__ __forceinline__ double from(int addr, double v)
{
    return __hiloint2double(from(addr, __double2hiint(v)), from(addr, __double2loint(v)));
}

// Orders a wave's own LDS accesses (its lanes run together; no instruction).
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One synchronous sweep: nw from old.  flags[1] is set to 1 when any value
// changed.
//
// Lane t of a row's group holds entry (i, j_t) and its sum.  Two lower entries
// (i, k) are taken at a time, each by one half of the group: the half loads
// row k's entries right of its diagonal, every lane finds its column among the
// j by a binary search across the group's registers (columns ascend, so lane
// order is column order), and stores l_ik u_kj in the LDS slot of that lane.
// Then every lane subtracts its two slots, in ascending k; a slot nobody wrote
// holds +0.0, which changes no sum.  No memory is touched but the rows, each
// read as a segment, and the next two rows' loads are issued before the
// search.  Bound by instruction issue: a 27-point row takes 7 such rounds,
// which is why the halves search row k's 13 upper entries in row i rather than
// all lanes row i's 27 in row k, one k at a time.  27-point operator on 80^3
// points: 2,430 us with a lane for each entry that searched the rows in
// memory, 500 us one k at a time, 340 us so (60 % of the vector issue slots
// taken, an LDS instruction every 8 cycles a CU).
template <int G>
__global__ void __launch_bounds__(256) k_fp_sweep(int n, const int32_t *__restrict__ rp,
                                                  const int32_t *__restrict__ col, const double *__restrict__ val,
                                                  const int32_t *__restrict__ dpos, const double *__restrict__ old,
                                                  double *__restrict__ nw, int32_t *flags)
{
    constexpr int H = G / 2;
    __shared__ double slots[256 / G][2 * G];
    const int lane = (int)threadIdx.x & (G - 1), half = lane / H, hl = lane % H;
    const int base = ((int)threadIdx.x & (63 & ~(G - 1))) * 4; // byte address of the group's first lane
    double *slot = slots[threadIdx.x / G];
    slot[lane] = 0.0;
    slot[G + lane] = 0.0;
    bool changed = false;
    // every loop runs while any row of the wave needs it, so that all lanes stay together
    for (int64_t i = first_row<G>(); __any(i < n); i += row_stride<G>()) {
        const bool row = i < n;
        const int p0 = row ? rp[i] : 0, p1 = row ? rp[i + 1] : 0, d = row ? dpos[i] : 0;
        for (int pb = p0; __any(pb < p1); pb += G) { // one round unless a row has more than G entries
            const int p = pb + lane;
            const bool live = p < p1;
            const int pc = live ? p : 0, cp = col[pc];
            const int j = live ? cp : INT32_MAX;
            const bool full = __any(lane == G - 1 && live); // else lane G - 1 holds INT_MAX
            double s = val[pc];
            const double was = old[pc], piv = old[dpos[cp]];
            for (int qb = p0; __any(qb < d); qb += G) {
                // this lane's lower entry: l_ik and the range of row k right of its diagonal (empty past the last)
                // (lanes past an end read entry 0: a load without a branch)
                const int q = qb + lane < d ? qb + lane : 0;
                const int k = col[q];
                const double lk = old[q];
                const int ub = dpos[k] + 1, ue = qb + lane < d ? rp[k + 1] : 0;
                int src = base + 4 * half; // the lane that holds this half's entry
                int u = from(src, ub) + hl, u1 = from(src, ue);
                int c = col[u < u1 ? u : 0];
                double v = old[u < u1 ? u : 0];
                for (int t = 0; t < G && __any(qb + t < d); t += 2) {
                    const double l = from(src, lk);
                    const int next = t + 2 < G ? src + 8 : src;
                    const int un = from(next, ub) + hl, un1 = from(next, ue);
                    const int cn = col[un < un1 ? un : 0];
                    const double vn = old[un < un1 ? un : 0];
                    for (;;) {
                        // the first j not below c: `at`, unless the search ends on lane G - 1, never looked at
                        int pos = base, at = INT32_MAX;
#pragma unroll
                        for (int w = H; w > 0; w >>= 1) {
                            const int x = from(pos + 4 * (w - 1), j);
                            if (x < c) pos += 4 * w;
                            else at = x;
                        }
                        if (full) at = from(pos, j);
                        if (at == c && u < u1) slot[half * G + ((pos - base) >> 2)] = l * v;
                        u += H;
                        if (!__any(u - hl < u1)) break;
                        c = col[u < u1 ? u : 0];
                        v = old[u < u1 ? u : 0];
                    }
                    wave_order();
                    const double a0 = slot[lane], a1 = slot[G + lane];
                    wave_order();
                    slot[lane] = 0.0;
                    slot[G + lane] = 0.0;
                    wave_order();
                    s = s - a0;
                    s = s - a1;
                    src = next;
                    u = un;
                    u1 = un1;
                    c = cn;
                    v = vn;
                }
            }
            if (live) {
                const double v = j < i ? s / piv : s;
                nw[p] = v;
                changed = changed || v != was;
            }
        }
    }
    // one lane of a wave, and only until the flag is seen set
    if (__any(changed) && (threadIdx.x & 63) == 0 &&
        __hip_atomic_load(&flags[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
        atomicOr(&flags[1], 1);
}

// Split the combined values into Ls (strict lower) and U (upper, diagonal
// first): row i's lower entries go to Lrp[i].., its upper ones to Urp[i]...
template <int G>
__global__ void __launch_bounds__(256) k_fp_split(int n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                  const int32_t *__restrict__ dpos, const double *__restrict__ LU,
                                                  const int32_t *__restrict__ Lrp, int32_t *__restrict__ Lcol,
                                                  double *__restrict__ Lval, const int32_t *__restrict__ Urp,
                                                  int32_t *__restrict__ Ucol, double *__restrict__ Uval, int64_t l_nnz,
                                                  int64_t u_nnz)
{
    const int lane = (int)threadIdx.x & (G - 1);
    for (int64_t i = first_row<G>(); i < n; i += row_stride<G>()) {
        const int p0 = rp[i], d = dpos[i];
        const int64_t ol = (int64_t)Lrp[i] - p0, ou = (int64_t)Urp[i] - d;
        for (int p = p0 + lane, p1 = rp[i + 1]; p < p1; p += G) {
            const int j = col[p];
            const double v = LU[p];
            if (p < d) {
                if (ol + p < l_nnz) {
                    Lcol[ol + p] = j;
                    Lval[ol + p] = v;
                }
            } else if (ou + p < u_nnz) {
                Ucol[ou + p] = j;
                Uval[ou + p] = v;
            }
        }
    }
}

template <int G>
dim3 grid_of(int n)
{
    return dim3((unsigned)std::min<int64_t>(((int64_t)n * G + 255) / 256, 1 << 23)); // a launch holds under 2^32 threads
}

} // namespace

// The body once for each group width.
#define SILU_BY_LANES(lanes, CALL)                                                                                    \
    switch (lanes) {                                                                                                  \
    case 8: CALL(8); break;                                                                                           \
    case 16: CALL(16); break;                                                                                         \
    case 32: CALL(32); break;                                                                                         \
    case 64: CALL(64); break;                                                                                         \
    default: return hipErrorInvalidValue;                                                                             \
    }

hipError_t launch_fp_init(int n, int lanes, const int32_t *rp, const int32_t *col, const double *val,
                          const int32_t *dpos, double *LU, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
#define CALL(G) hipLaunchKernelGGL(k_fp_init<G>, grid_of<G>(n), dim3(256), 0, s, n, rp, col, val, dpos, LU)
    SILU_BY_LANES(lanes, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_fp_sweep(int n, int lanes, const int32_t *rp, const int32_t *col, const double *val,
                           const int32_t *dpos, const double *old, double *nw, int32_t *flags, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
#define CALL(G) hipLaunchKernelGGL(k_fp_sweep<G>, grid_of<G>(n), dim3(256), 0, s, n, rp, col, val, dpos, old, nw, flags)
    SILU_BY_LANES(lanes, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_fp_split(int n, int lanes, const int32_t *rp, const int32_t *col, const int32_t *dpos,
                           const double *LU, const int32_t *Lrp, int32_t *Lcol, double *Lval, const int32_t *Urp,
                           int32_t *Ucol, double *Uval, int64_t l_nnz, int64_t u_nnz, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
#define CALL(G)                                                                                                       \
    hipLaunchKernelGGL(k_fp_split<G>, grid_of<G>(n), dim3(256), 0, s, n, rp, col, dpos, LU, Lrp, Lcol, Lval, Urp, Ucol, \
                       Uval, l_nnz, u_nnz)
    SILU_BY_LANES(lanes, CALL)
#undef CALL
    return hipGetLastError();
}

} // namespace silu
