// Level-scheduled substitution (Section 4) on a level-ordered copy of the
// triangle.
//
// The rows of a level depend on earlier levels only, and a factor has hundreds
// to thousands of levels of a few hundred to a few thousand rows: the solve is
// a chain of short dependent steps.  One launch per level costs 4.2 to 5.5 us
// whatever the level holds (its kernel, four dependent loads deep, and the
// gap).  So consecutive narrow levels are a run, solved by ONE workgroup in one
// launch (k_level_run), a barrier between levels.  What a run reads of earlier
// positions is known when it starts, and is subtracted from its right-hand
// sides by the whole chip first (k_level_far); wide levels, which one compute
// unit would stream for longer than a launch takes, are solved by that kernel
// alone.
//
// Layout: positions number the rows level by level; a slice is up to 64
// consecutive positions of one level, its entries stored pair-major (pair p of
// the slice's lane l at off + p nl + l), ascending as in the matrix.  The
// structure is built once per pattern; values, right-hand side and pivots are
// packed into it by every solve (k_level_pack, at the chip's bandwidth), and
// the solution is unpacked by another launch (k_level_unpack), so the one
// compute unit reads and writes whole segments only.  Rows far longer than
// their neighbours make a slice of their own, shared by 64 lanes.
#include "internal.h"

#pragma clang fp contract(off)

namespace silu {
namespace {

// The level of a position: the last that starts at or before it.
__device__ __forceinline__ int level_of(int depth, const int32_t *__restrict__ level_ptr, int at)
{
    int lo = 0, hi = depth;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (level_ptr[mid] <= at) lo = mid;
        else hi = mid;
    }
    return lo;
}

__global__ void __launch_bounds__(256) k_level_reach(int n, int depth, const int32_t *__restrict__ level_ptr,
                                                     const int32_t *__restrict__ perm, const int32_t *__restrict__ pos,
                                                     const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                     int32_t *reach)
{
    const int at = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (at >= n) return;
    const int lv = level_of(depth, level_ptr, at), horizon = level_ptr[lv + 1] - LEVEL_RING, r = perm[at];
    if (horizon <= 0) return;
    int hi = -1;
    for (int p = rp[r]; p < rp[r + 1]; ++p) {
        const int c = pos[col[p]];
        if (c < horizon) hi = max(hi, c);
    }
    if (hi > __hip_atomic_load(&reach[lv], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&reach[lv], hi);
}

__global__ void __launch_bounds__(256) k_level_count(int n, int depth, const int32_t *__restrict__ level_ptr,
                                                     const int32_t *__restrict__ start,
                                                     const int32_t *__restrict__ perm, const int32_t *__restrict__ pos,
                                                     const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                     int32_t *__restrict__ counts)
{
    const int at = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (at >= n) return;
    const int s0 = start[level_of(depth, level_ptr, at)], r = perm[at];
    int near = 0, far = 0;
    for (int p = rp[r]; p < rp[r + 1]; ++p) {
        const int j = col[p];
        if (j == r) continue;
        if (pos[j] >= s0) ++near;
        else ++far;
    }
    counts[at] = near;
    counts[(int64_t)n + at] = far;
}

__global__ void __launch_bounds__(256) k_level_diag(int n, const int32_t *__restrict__ perm,
                                                    const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                    int32_t *__restrict__ dsrc)
{
    const int at = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (at >= n) return;
    const int r = perm[at];
    int d = -1;
    for (int p = rp[r]; p < rp[r + 1]; ++p)
        if (col[p] == r) d = p;
    dsrc[at] = d;
}

// One wave per slice: codes and value sources of its kind of entries.  Padding
// has source -1 (value 0) and reads a place that always holds 0, so that no
// row meets a value it does not depend on: behind the ring, or y[n].
template <bool FAR>
__global__ void __launch_bounds__(256) k_level_fill(int nslice, int n, LevelSlice *__restrict__ slices,
                                                    const int32_t *__restrict__ perm, const int32_t *__restrict__ pos,
                                                    const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                                    void *__restrict__ code, int32_t *__restrict__ src)
{
    const int s = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    if (s >= nslice) return;
    const LevelSlice d = slices[s];
    const bool shared = d.rows < 0; // one row, 64 lanes
    const int nl = shared ? 64 : d.rows;
    if (lane >= nl) return;
    const int r = perm[d.row0 + (shared ? 0 : lane)];
    int k = 0;
    auto put = [&](int c, int p) {
        const int64_t slot = 2 * (d.off + (int64_t)(k >> 1) * nl + lane) + (k & 1);
        if (FAR) ((int32_t *)code)[slot] = c;
        else ((uint16_t *)code)[slot] = (uint16_t)c;
        src[slot] = p;
        ++k;
    };
    for (int p = rp[r] + (shared ? lane : 0); p < rp[r + 1]; p += shared ? 64 : 1) {
        const int j = col[p];
        if (j == r) continue;
        const int c = pos[j];
        if ((c < d.start) != FAR) continue;
        put(FAR ? c : c % LEVEL_RING, p);
    }
    while (k < 2 * d.pairs) put(FAR ? n : LEVEL_RING, -1);
    if (!FAR && lane == 0) slices[s].start = d.row0 % LEVEL_RING; // every lane has its copy
}

// A use of v: what loaded it is waited for here.
__device__ __forceinline__ void arrived(int v) { asm volatile("" ::"v"(v)); }

// Values into the layout (workgroups below `nv`), then right-hand side and
// pivots of the rows.  The near entries' codes are read for nothing but to have
// them in the memory-side cache, from which the runs' single workgroups read
// twice as fast as from HBM (114 against 62 GB/s): solving with three triangles
// in turn, of 80^3 rows of 20 entries each, 2.08 -> 1.78 ms a solve, where the
// whole chip reads the codes in a few us.
__global__ void __launch_bounds__(256) k_level_pack(int64_t slots, unsigned nv, int n, const int32_t *__restrict__ src,
                                                    const uint16_t *__restrict__ near, int64_t near_slots,
                                                    const double *__restrict__ val, const int32_t *__restrict__ perm,
                                                    const int32_t *__restrict__ dsrc, const double *__restrict__ rhs,
                                                    double *__restrict__ pval, double *__restrict__ pb,
                                                    double *__restrict__ piv)
{
    if (blockIdx.x < nv) {
        const int64_t i0 = (int64_t)blockIdx.x * 1024 + threadIdx.x;
        int s[4];
        unsigned code[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] = i0 + 256 * k < slots ? src[i0 + 256 * k] : -1;
#pragma unroll
        for (int k = 0; k < 4; ++k) code[k] = i0 + 256 * k < near_slots ? near[i0 + 256 * k] : 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i0 + 256 * k < slots) pval[i0 + 256 * k] = s[k] >= 0 ? val[s[k]] : 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) arrived(code[k]); // all that is wanted of it
        return;
    }
    const int64_t i = (int64_t)(blockIdx.x - nv) * 256 + threadIdx.x;
    if (i >= n) return;
    pb[i] = rhs[perm[i]];
    if (piv) piv[i] = dsrc[i] >= 0 ? val[dsrc[i]] : 0.0;
}

// The solution to its rows: out (or null), s_out = dinv * y, xupd += (dcol) y.
__global__ void __launch_bounds__(256) k_level_unpack(int n, const int32_t *__restrict__ perm,
                                                      const double *__restrict__ y, double *__restrict__ out,
                                                      const double *__restrict__ dinv, double *__restrict__ s_out,
                                                      double *__restrict__ xupd, const double *__restrict__ dcol)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int r = perm[i];
    const double v = y[i];
    if (out) out[r] = v;
    if (s_out) s_out[r] = dinv[r] * v;
    if (xupd) xupd[r] = xupd[r] + (dcol ? dcol[r] : 1.0) * v;
}

__device__ __forceinline__ int lanes_of(const LevelSlice &d) { return d.rows < 0 ? 64 : d.rows; }

// A slice's sum over its 64 lanes, where they share one row.
__device__ __forceinline__ double row_sum(const LevelSlice &d, double s)
{
    if (d.rows < 0)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s = s + __shfl_xor(s, off);
    return s;
}

// A wave a far slice, over the whole chip: what its rows read of positions
// before their run's first is subtracted from the right-hand side, or, for a
// wide level (SOLVE), the rows are finished.
template <bool SOLVE, bool UNIT, int FAR_PAIRS>
__global__ void __launch_bounds__(256) k_level_far(LevelView L, int f0, int f1)
{
    const int lane = (int)threadIdx.x & 63;
    const int f = f0 + (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (f >= f1) return;
    const LevelSlice d = L.far_slices[f];
    const int nl = lanes_of(d);
    const int64_t at = d.off + (lane < nl ? lane : 0);
    // FAR_PAIRS at a time: their codes and values, then their gathers, then the sum
    double s = 0.0;
    for (int p0 = 0; p0 < d.pairs; p0 += FAR_PAIRS) {
        int2 c[FAR_PAIRS];
        double2 v[FAR_PAIRS];
        double x[2 * FAR_PAIRS];
#pragma unroll
        for (int k = 0; k < FAR_PAIRS; ++k) {
            const int64_t e = at + (int64_t)min(p0 + k, d.pairs - 1) * nl;
            c[k] = ((const int2 *)L.far)[e];
            v[k] = ((const double2 *)L.far_val)[e];
        }
#pragma unroll
        for (int k = 0; k < FAR_PAIRS; ++k) {
            x[2 * k] = L.y[c[k].x];
            x[2 * k + 1] = L.y[c[k].y];
        }
#pragma unroll
        for (int k = 0; k < FAR_PAIRS; ++k)
            if (p0 + k < d.pairs) { // the same in the whole wave
                s = s + v[k].x * x[2 * k];
                s = s + v[k].y * x[2 * k + 1];
            }
    }
    s = row_sum(d, s);
    if (lane >= (d.rows < 0 ? 1 : d.rows)) return;
    const int row = d.row0 + lane;
    double v = L.b[row] - s;
    if (SOLVE) {
        if (!UNIT) v = v / L.piv[row];
        L.y[row] = v;
    } else {
        L.b[row] = v;
    }
}

// `bytes` from p on as a buffer: loads past them give 0, stores do nothing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t range(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0, bytes, 0x00020000);
}

// A near slice's operands in registers: up to KP pairs a lane, with their
// places in the ring, two to a word.
template <int KP>
struct SliceRegs {
    double2 v[KP];
    unsigned c[KP];
    double b, piv;
};

// FIXED: every slice takes the same number of loads, those past its pairs,
// lanes or rows out of their buffer's range (nothing is fetched): where the
// number depends on the slice, the compiler has the wait for one slice's
// operands wait for those of the slices behind it too.
template <int KP, bool UNIT, bool FIXED>
__device__ __forceinline__ void load_slice(const LevelView &L, const LevelSlice &d, int lane, SliceRegs<KP> &g)
{
    constexpr int NONE = 1 << 28; // a slice's operands are far smaller
    const int nl = lanes_of(d), words = min(d.pairs, KP) * nl;
    const auto val = range((const double2 *)L.val + d.off, words * 16);
    const auto near = range((const unsigned *)L.near + d.off, words * 4);
    int at_v = lane < nl ? lane * 16 : NONE, at_c = lane < nl ? lane * 4 : NONE;
#pragma unroll
    for (int p = 0; p < KP; ++p) {
        if (FIXED || p < d.pairs) {
            g.v[p] = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(val, at_v, 0, 0));
            g.c[p] = __builtin_amdgcn_raw_buffer_load_b32(near, at_c, 0, 0);
        }
        at_v += nl * 16;
        at_c += nl * 4;
    }
    const int bytes = (d.rows < 0 ? 1 : d.rows) * 8;
    g.b = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(range(L.b + d.row0, bytes), lane * 8, 0, 0));
    if (!UNIT)
        g.piv = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(range(L.piv + d.row0, bytes), lane * 8, 0, 0));
}

// Sum of a slice's products, each lane's in ascending order.
template <int KP, int P>
__device__ __forceinline__ double slice_sum(const SliceRegs<KP> &g, const double *ring)
{
    double x[2 * P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        x[2 * p] = ring[g.c[p] & 0xffff];
        x[2 * p + 1] = ring[g.c[p] >> 16];
    }
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        s = s + g.v[p].x * x[2 * p];
        s = s + g.v[p].y * x[2 * p + 1];
    }
    return s;
}

template <int KP, int P>
__device__ __forceinline__ double slice_sum_of(int pairs, const SliceRegs<KP> &g, const double *ring)
{
    if constexpr (P > 1)
        if (pairs < P) return slice_sum_of<KP, P - 1>(pairs, g, ring);
    return slice_sum<KP, P>(g, ring);
}

// More pairs than registers hold: the others from memory.
template <int KP>
__device__ __forceinline__ double slice_sum_long(const LevelView &L, const LevelSlice &d, const SliceRegs<KP> &g, int lane,
                                                 const double *ring)
{
    double s = slice_sum<KP, KP>(g, ring);
    const int nl = lanes_of(d);
    const int64_t at = d.off + (lane < nl ? lane : 0);
#pragma unroll 4
    for (int p = KP; p < d.pairs; ++p) {
        const double2 v = ((const double2 *)L.val)[at + (int64_t)p * nl];
        const unsigned c = ((const unsigned *)L.near)[at + (int64_t)p * nl];
        s = s + v.x * ring[c & 0xffff];
        s = s + v.y * ring[c >> 16];
    }
    return s;
}

// Workgroup barrier that orders LDS only: loads under way for the next slices
// stay under way (a full barrier waits for them).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A wave's next 64 slices (every RUN_WAVES-th from q on), lane k holding the k-th: they
// are handed out from registers, since a scalar load would have every LDS wait
// wait for it too.
constexpr int RUN_WAVES = 16; // waves of a level run
constexpr int RUN_DEPTH4 = 2; // slices of up to 4 pairs that each holds (1: 57 GB/s taken in, 2: 70 to 86, 3: the same)

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

struct SliceQueue {
    int64_t off;
    int row0, level;
    unsigned shape; // place in the ring, rows, and pairs where they fit
    int next = 64;
    __device__ __forceinline__ LevelSlice pop(const LevelView &L, int q, int end, int lane)
    {
        if (next == 64) {
            const int k = q + RUN_WAVES * lane;
            const LevelSlice s = L.slices[k < end ? k : end - 1];
            off = s.off;
            row0 = s.row0;
            level = s.level;
            shape = (unsigned)s.start | (unsigned)(s.rows < 0 ? 0 : s.rows) << 16 | (unsigned)min(s.pairs, MANY) << 24;
            // waits here: behind the branch it would wait for the operands under way whenever a slice is handed out
            arrived((int)off);
            arrived(row0);
            arrived(level);
            arrived(shape);
            next = 0;
        }
        LevelSlice d;
        const int lo = __builtin_amdgcn_readlane((int)(uint32_t)off, next),
                  hi = __builtin_amdgcn_readlane((int)(off >> 32), next);
        d.off = (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
        d.row0 = __builtin_amdgcn_readlane(row0, next);
        d.level = __builtin_amdgcn_readlane(level, next);
        const unsigned f = (unsigned)__builtin_amdgcn_readlane((int)shape, next);
        d.start = (int)(f & 0xffff);
        d.rows = (int)(f >> 16 & 0xff);
        if (d.rows == 0) d.rows = -1;
        d.pairs = (int)(f >> 24);
        if (d.pairs == MANY) d.pairs = L.slices[min(q, end - 1)].pairs;
        ++next;
        return d;
    }
    static constexpr int MANY = 255;
};

// Levels [l0, l1) in one workgroup of 16 waves.  The solution of the last
// LEVEL_RING positions stands in LDS; the host cuts runs so that every near
// entry finds its value there.  Slices go round
// the waves, and a wave holds its next DEPTH slices in registers: what bounds
// the run is the rate at which one compute unit takes the factor in (a plain
// stream of one: 112 GB/s with 256 KB in flight, 64 GB/s with 128 KB).  A
// slice's registers are loaded again after it was summed and, unless the wave's
// next slice is of the same level, after the barrier, so that the loads' issue
// does not stand between a level and the next (68 against 98 GB/s).  A slice
// knows its level, so that each wave counts its barriers and meets no branch
// whose loads would be waited for behind it.  Levels of 692 rows of 6 entries:
// 0.89 us each (0.96 where every sum waited for all loads in flight; a launch
// each: 4.3), of which memory is no longer the larger part: holding three
// slices, or operands that others had brought into the L2, changed nothing.
// Levels of 437 rows of 20 entries 1.2 us, of 350 rows of 3 0.43 us.
// Non-temporal loads came to 42 GB/s, touching the factor ahead by four further
// waves to 55.
template <int KP, int DEPTH, bool UNIT>
__global__ void __launch_bounds__(1024) k_level_run(LevelView L, int l0, int l1)
{
    __shared__ double ring[LEVEL_RING + 1]; // and a 0 for padding
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int end = L.first[l1];
    if (threadIdx.x == 0) ring[LEVEL_RING] = 0.0;
    lds_barrier();
    int q = L.first[l0] + wave, l = l0;
    SliceQueue queue;
    LevelSlice d[DEPTH];
    SliceRegs<KP> g[DEPTH];
#pragma unroll
    for (int k = 0; k < DEPTH - 1; ++k) {
        d[k] = queue.pop(L, q + RUN_WAVES * k, end, lane);
        load_slice<KP, UNIT, (DEPTH > 1)>(L, d[k], lane, g[k]);
    }
    while (q < end) {
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) {
            // the slice summed last: its registers take the one DEPTH - 1 behind the next (past the run's
            // end: the last slice, unused)
            constexpr int AHEAD = RUN_WAVES * (DEPTH - 1);
            LevelSlice &dl = d[(k + DEPTH - 1) % DEPTH];
            dl = queue.pop(L, q + AHEAD, end, lane);
            if (l < d[k].level) {
                lds_barrier();
                ++l;
            }
            load_slice<KP, UNIT, (DEPTH > 1)>(L, dl, lane, g[(k + DEPTH - 1) % DEPTH]);
            for (; l < d[k].level; ++l) lds_barrier();
            double s = 0.0;
            if (d[k].pairs > KP) s = slice_sum_long<KP>(L, d[k], g[k], lane, ring);
            else if (d[k].pairs > 0) s = slice_sum_of<KP, KP>(d[k].pairs, g[k], ring);
            s = row_sum(d[k], s);
            const int rows = d[k].rows < 0 ? 1 : d[k].rows, place = d[k].start + lane;
            double v = g[k].b - s;
            if (!UNIT) v = v / g[k].piv;
            if (lane < rows) ring[place < LEVEL_RING ? place : place - LEVEL_RING] = v;
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), range(L.y + d[k].row0, rows * 8), lane * 8, 0, 0);
            q += RUN_WAVES;
            if (q >= end) break;
        }
    }
    for (; l < l1; ++l) lds_barrier();
}

} // namespace

static_assert(LEVEL_RING < 65536, "places in the ring are 16-bit");

hipError_t launch_level_reach(int n, int depth, const int32_t *level_ptr, const int32_t *perm, const int32_t *pos,
                              const int32_t *rp, const int32_t *col, int32_t *reach, hipStream_t s)
{
    hipLaunchKernelGGL(k_level_reach, dim3((unsigned)(((int64_t)n + 255) / 256)), dim3(256), 0, s, n, depth, level_ptr, perm,
                       pos, rp, col, reach);
    return hipGetLastError();
}

hipError_t launch_level_count(int n, int depth, const int32_t *level_ptr, const int32_t *start, const int32_t *perm,
                              const int32_t *pos, const int32_t *rp, const int32_t *col, int32_t *counts, hipStream_t s)
{
    hipLaunchKernelGGL(k_level_count, dim3((unsigned)(((int64_t)n + 255) / 256)), dim3(256), 0, s, n, depth, level_ptr,
                       start, perm, pos, rp, col, counts);
    return hipGetLastError();
}

hipError_t launch_level_diag(int n, const int32_t *perm, const int32_t *rp, const int32_t *col, int32_t *dsrc,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_level_diag, dim3((unsigned)(((int64_t)n + 255) / 256)), dim3(256), 0, s, n, perm, rp, col, dsrc);
    return hipGetLastError();
}

hipError_t launch_level_fill(int nslice, int n, int far_kind, LevelSlice *slices, const int32_t *perm, const int32_t *pos,
                             const int32_t *rp, const int32_t *col, void *code, int32_t *src, hipStream_t s)
{
    if (nslice <= 0) return hipSuccess;
    const dim3 g((nslice + 3) / 4), b(256);
    if (far_kind) hipLaunchKernelGGL(k_level_fill<true>, g, b, 0, s, nslice, n, slices, perm, pos, rp, col, code, src);
    else hipLaunchKernelGGL(k_level_fill<false>, g, b, 0, s, nslice, n, slices, perm, pos, rp, col, code, src);
    return hipGetLastError();
}

hipError_t launch_level_pack(int64_t slots, int n, const int32_t *src, const uint16_t *near, int64_t near_slots,
                             const double *val, const int32_t *perm,
                             const int32_t *dsrc, const double *rhs, double *pval, double *pb, double *piv,
                             hipStream_t s)
{
    const unsigned nv = (unsigned)((slots + 1023) / 1024), nr = (unsigned)(((int64_t)n + 255) / 256);
    hipLaunchKernelGGL(k_level_pack, dim3(nv + nr), dim3(256), 0, s, slots, nv, n, src, near, near_slots, val, perm, dsrc, rhs, pval, pb,
                       piv);
    return hipGetLastError();
}

hipError_t launch_level_unpack(int n, const int32_t *perm, const double *y, double *out, const double *dinv,
                               double *s_out, double *xupd, const double *dcol, hipStream_t s)
{
    hipLaunchKernelGGL(k_level_unpack, dim3((unsigned)(((int64_t)n + 255) / 256)), dim3(256), 0, s, n, perm, y, out, dinv,
                       s_out, xupd, dcol);
    return hipGetLastError();
}

template <bool SOLVE, bool UNIT>
void go_far(const LevelView &L, int f0, int f1, int max_pairs, hipStream_t s)
{
    const dim3 g((f1 - f0 + 3) / 4), b(256);
    if (max_pairs <= 4) hipLaunchKernelGGL((k_level_far<SOLVE, UNIT, 4>), g, b, 0, s, L, f0, f1);
    else hipLaunchKernelGGL((k_level_far<SOLVE, UNIT, 10>), g, b, 0, s, L, f0, f1);
}

hipError_t launch_level_far(const LevelView &L, int f0, int f1, int solve, int unit, int max_pairs, hipStream_t s)
{
    if (f1 <= f0) return hipSuccess;
    if (!solve) go_far<false, true>(L, f0, f1, max_pairs, s);
    else if (unit) go_far<true, true>(L, f0, f1, max_pairs, s);
    else go_far<true, false>(L, f0, f1, max_pairs, s);
    return hipGetLastError();
}

hipError_t launch_level_run(const LevelView &L, int l0, int l1, int unit, int max_pairs, hipStream_t s)
{
    const dim3 g(1), b(1024);
    if (max_pairs <= 4) {
        if (unit) hipLaunchKernelGGL((k_level_run<4, RUN_DEPTH4, true>), g, b, 0, s, L, l0, l1);
        else hipLaunchKernelGGL((k_level_run<4, RUN_DEPTH4, false>), g, b, 0, s, L, l0, l1);
    } else {
        if (unit) hipLaunchKernelGGL((k_level_run<LEVEL_PAIRS, 1, true>), g, b, 0, s, L, l0, l1);
        else hipLaunchKernelGGL((k_level_run<LEVEL_PAIRS, 1, false>), g, b, 0, s, L, l0, l1);
    }
    return hipGetLastError();
}

} // namespace silu
