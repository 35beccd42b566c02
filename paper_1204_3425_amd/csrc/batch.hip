// Batched Lanczos for many small sectors (Sec. 2.2, Alg. 1; Sec. 4.3 H.v).
//
// A sector of a few thousand to a million states leaves most of the MI355X
// idle (the paper's Sec. 5 reports the same for small systems on its GPU).
// The batch engine advances every active instance by one Lanczos step with
// two launches in total, whatever the number of instances:
//     batched H.v + three-term update (work item = rows of one instance),
//         and one extra workgroup per instance that finishes the step before:
//         b_j, the Ritz value E_{j-1} of T_j and the stop test of the
//         single-instance driver, with the mailbox entry
//     batched q - a_j f_j update + partial norms
// Each workgroup derives the step's scalars itself: a_j from the instance's
// H.v partial sums and b_j from its update partial sums, summed in the same
// fixed order everywhere, so no launch is spent on reductions alone and the
// Ritz value (a multisection) runs beside the next H.v instead of before it.
// A step that a stop test ends is therefore followed by one more H.v whose
// result is never used.  Work items never span two instances and each
// instance's partial sums are added in a fixed order, so an instance's results
// do not depend on which other instances share the launches.  An instance
// that has stopped skips every kernel of later steps, so the host can read the
// step mailboxes a few steps behind without holding the device.
//
// H.v here is the one-launch form (as in tile.hip, several rows to a work item):
// a workgroup stages the rows of its item in LDS, gathers the down-spin hops from
// them and adds the up-spin rows from global memory (every vector of a batched
// instance is small enough to stay in the L2 and the Infinity Cache).
#include <hip/hip_runtime.h>

#include "batch.h"
#include "start.h"

namespace hub {

namespace {

__device__ inline double wg_sum(double v, double *scratch)
{
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0)
        scratch[wave] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); w++)
            s += scratch[w];
    __syncthreads();
    return s;
}

constexpr int kThreads = 256;

// Sum of an instance's n partial sums in a fixed order, by one wave (every lane
// gets it; every wave that needs it gets the same value).
__device__ inline double inst_sum(const double *__restrict__ part, int n)
{
    double s = 0.0;
    for (int i = threadIdx.x & 63; i < n; i += 8 * 64) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; u++)
            v[u] = part[i + 64 * u < n ? i + 64 * u : 0];
#pragma unroll
        for (int u = 0; u < 8; u++)
            s += i + 64 * u < n ? v[u] : 0.0;
    }
    for (int off = 32; off > 0; off >>= 1)
        s += __shfl_xor(s, off, 64);
    return s;
}

__device__ __forceinline__ void ritz_and_stop(const BatchInst &in, int j, double *__restrict__ mailbox);

__device__ inline float with_sign(float v, uint32_t sg) { return __int_as_float(__float_as_int(v) ^ (int)sg); }
__device__ inline double with_sign(double v, uint32_t sg)
{
    return __hiloint2double(__double2hiint(v) ^ (int)sg, __double2loint(v));
}

template <typename T>
struct Pair;
template <>
struct Pair<float> {
    typedef float2 type;
};
template <>
struct Pair<double> {
    typedef double2 type;
};

// H.v of a work item on pairs of rows.  A pair is staged interleaved, once as x
// and once as -x behind a zero slot, so a down-spin entry is an index alone (its
// sign picks the copy) and one address and one LDS read serve both rows: per
// element and entry one FMA and half an address, against six instructions with
// the sign in the entry.  A row's up-spin factors are scalars (+-t, 0 past its
// count: a non-finite x makes the step's coefficients non-finite either way).
// A wave takes 64 columns of a pair at a time; with rows of at most kBatchNarrow
// elements (NARROW, a row's up-spin entries then differ from lane to lane) as many
// pairs as fill its lanes.  One row at a time, 2,048 rows of one column were 256
// steps of each wave (20 FP64 steps, ms: 4x4 8u0d 12.2 / 0.85, 20-site ring 10u0d
// 15.5 / 1.1, 16 solves of 10u1d 55 / 33; element by element, before pairs, 1.9, 2.5, 40).
// Returns the thread's share of q.x.
template <typename T, bool NARROW>
__device__ __forceinline__ double batch_pairs(const BatchInst &in, const BatchItem &it, const T *__restrict__ x,
                                              T *__restrict__ y, const typename Pair<T>::type *xp, T a_s, T b_s)
{
    typedef typename Pair<T>::type V2;
    const T tm = (T)(-in.t), tp = (T)in.t, U = (T)in.U;
    const int ddn = (int)in.dim_dn, nrows = (int)it.nrows, npair = (nrows + 1) >> 1, width = 2 * (ddn + 1);
    const int64_t base = it.r0 * in.dim_dn;
    const uint32_t rowb = (uint32_t)ddn * (uint32_t)sizeof(T);
    const unsigned char *__restrict__ xb = reinterpret_cast<const unsigned char *>(x);
    double acc = 0.0;
    // tasks of a wave: 64 columns by a share of the pairs, as many shares as
    // leave the four waves about the same number of tasks
    const int lane = (int)threadIdx.x & 63, nch = NARROW ? 1 : (ddn + 63) >> 6;
    int cols = 64;  // lanes to a pair
    while (NARROW && cols >= 2 * ddn)
        cols >>= 1;
    const int shares = NARROW ? kThreads / 64 : min(npair, nch % 4 == 0 ? 1 : nch % 2 == 0 ? 2 : 4);
    for (int task = (int)threadIdx.x >> 6; task < nch * shares; task += kThreads / 64) {
        const int c = __builtin_amdgcn_readfirstlane(task % nch), sh = __builtin_amdgcn_readfirstlane(task / nch);
        const int d = NARROW ? lane & (cols - 1) : c * 64 + lane;
        const bool ok = d < ddn;
        const int dc = ok ? d : ddn - 1;
        const int nq = __builtin_amdgcn_readfirstlane((int)in.dn_nq[c]);
        const uint4 *__restrict__ dn = in.dn_pair + dc;
        uint4 e4[2];
#pragma unroll
        for (int g = 0; g < 2; g++)
            e4[g] = dn[(size_t)(g < in.gmax ? g : 0) * (size_t)ddn];
        const uint32_t sd = in.states_dn[dc];
        const uint32_t off = (uint32_t)dc * (uint32_t)sizeof(T);
        const int p0 = NARROW ? (int)threadIdx.x / cols : sh * npair / shares;
        const int p1 = NARROW ? npair : (sh + 1) * npair / shares, pstep = NARROW ? kThreads / cols : 1;
        for (int pl = p0; pl < p1; pl += pstep) {
            const bool two = 2 * pl + 1 < nrows;
            const int64_t r0 = it.r0 + 2 * pl, r1 = two ? r0 + 1 : r0;
            const uint32_t *__restrict__ ur[2] = {in.up_tile + r0 * in.w_up, in.up_tile + r1 * in.w_up};
            const int nu[2] = {in.nnz_up[r0], in.nnz_up[r1]};
            T uv[2][8];
            auto up_load = [&](int s, int k0) {
#pragma unroll
                for (int u = 0; u < 8; u++)
                    uv[s][u] = *reinterpret_cast<const T *>(xb + ((ur[s][k0 + u] & 0x7fffffffu) * rowb + off));
            };
            up_load(0, 0);
            up_load(1, 0);
            const int64_t J0 = base + (int64_t)(2 * pl) * ddn + dc, J1 = two ? J0 + ddn : J0;
            const T y0 = y[J0], y1 = y[J1];
            const V2 *__restrict__ xrow = xp + pl * width;
            const V2 xv = xrow[dc];
            T h[2] = {U * (T)__popc(in.states_up[r0] & sd) * xv.x, U * (T)__popc(in.states_up[r1] & sd) * xv.y};
            auto group = [&](const uint4 &e) {
                const uint32_t ev[4] = {e.x, e.y, e.z, e.w};
                V2 v[8];
#pragma unroll
                for (int u = 0; u < 8; u++)
                    v[u] = xrow[(u & 1) ? ev[u >> 1] >> 16 : ev[u >> 1] & 0xffffu];
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    h[0] = fma(tm, v[u].x, h[0]);
                    h[1] = fma(tm, v[u].y, h[1]);
                }
            };
#pragma unroll
            for (int g = 0; g < 2; g++)
                if (g < nq)
                    group(e4[g]);
            for (int g = 2; g < nq; g++)
                group(dn[(size_t)g * (size_t)ddn]);
            auto up_add = [&](int s, int k0) {
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    const T f = k0 + u < nu[s] ? ((ur[s][k0 + u] >> 31) ? tp : tm) : (T)0;
                    h[s] = fma(f, uv[s][u], h[s]);
                }
            };
#pragma unroll
            for (int s = 0; s < 2; s++) {
                up_add(s, 0);
                for (int k0 = 8; k0 < nu[s]; k0 += 8) {
                    up_load(s, k0);
                    up_add(s, k0);
                }
            }
            const T q0 = fma(a_s, h[0], b_s * y0), q1 = fma(a_s, h[1], b_s * y1);
            if (ok) {
                y[J0] = q0;
                acc += (double)q0 * (double)xv.x;
                if (two) {
                    y[J1] = q1;
                    acc += (double)q1 * (double)xv.y;
                }
            }
        }
    }
    return acc;
}

// Workgroups 0 .. n_inst-1 finish step j - 1 of their instance (ritz_and_stop);
// the others are the work items of step j.
//
// The item's rows are staged in LDS, each followed by a zero slot that the down
// table's padding points at.  A wave takes 64 columns of the item and goes
// through its rows: the column's down entries (eight 16-bit indices with signs to
// a 16-byte load) are read once for all of them, a row's up entries are scalars,
// and eight up-spin rows are in flight at a time.  Per element the hops are added
// in table order, one FMA by -t each, down-spin first.  Element by element, with
// each entry a 4-byte load of its own for either spin, the kernel spent 123 us on
// 32 rings of 10 to 12 sites (8.3 M FP32 elements; two such launches at a time);
// this form, on pairs of rows, 95 us, about half of it instruction issue and the
// rest the staging and the up-spin rows' trips to the L2.
// PAIRS: every listed instance takes the form on row pairs; NARROW: some of them
// have rows of at most kBatchNarrow elements.
template <typename T, bool PAIRS, bool NARROW>
__global__ __launch_bounds__(kThreads) void batch_hv_kernel(const BatchInst *__restrict__ insts,
                                                            const BatchItem *__restrict__ items, int n_inst, int k,
                                                            double *__restrict__ mailbox)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *xs = reinterpret_cast<T *>(smem_raw);
    __shared__ double red[kThreads / 64];
    if ((int)blockIdx.x < n_inst) {
        const BatchInst &in = insts[blockIdx.x];
        ritz_and_stop(in, in.j0 + k, mailbox);
        return;
    }
    const BatchItem it = items[blockIdx.x - n_inst];
    const BatchInst in = insts[it.inst];
    // the instance's Ritz workgroup may set the flag during this launch: one
    // read for the whole workgroup, so all its waves agree
    __shared__ int stopped;
    if (threadIdx.x == 0)
        stopped = in.st->stopped;
    const int j = in.j0 + k;  // this instance's step
    const int ddn = (int)in.dim_dn, nrows = (int)it.nrows;
    const int n = nrows * ddn;  // elements of the item (at most 16384)
    // x = s_j f_j with 1/s_j = S0: vec0 on even steps; y holds s_{j-1} f_{j-1}
    const T *__restrict__ x = reinterpret_cast<const T *>((j & 1) ? in.vec1 : in.vec0);
    T *__restrict__ y = reinterpret_cast<T *>((j & 1) ? in.vec0 : in.vec1);
    const int64_t base = it.r0 * in.dim_dn;
    typedef typename Pair<T>::type V2;
    const int npair = (nrows + 1) >> 1, width = 2 * (ddn + 1);
    const bool narrow = NARROW && ddn <= kBatchNarrow && in.dn_pair;
    if (narrow) {
        // rows are contiguous: element by element, each to its half of a pair
        V2 *xp = reinterpret_cast<V2 *>(smem_raw);
        int rl = (int)threadIdx.x / ddn, d = (int)threadIdx.x - rl * ddn;
        for (int i0 = 0; i0 < n; i0 += 8 * kThreads) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const int i = i0 + u * kThreads + (int)threadIdx.x;
                v[u] = x[base + (i < n ? i : 0)];
            }
#pragma unroll
            for (int u = 0; u < 8; u++) {
                if (i0 + u * kThreads + (int)threadIdx.x < n) {
                    T *half = reinterpret_cast<T *>(xp + (rl >> 1) * width) + (rl & 1);
                    half[2 * d] = v[u];
                    half[2 * (d + ddn + 1)] = -v[u];
                }
                rl += kThreads / ddn;
                d += kThreads % ddn;
                if (d >= ddn) {
                    d -= ddn;
                    rl++;
                }
            }
        }
        for (int r = threadIdx.x; r < npair; r += kThreads)
            xp[r * width + ddn] = V2{(T)0, (T)0};
    } else if (PAIRS || in.dn_pair) {
        V2 *xp = reinterpret_cast<V2 *>(smem_raw);
        // the threads as rows of a power of two of columns, each taking a pair
        int cols = kThreads;
        while (cols >= 2 * ddn && cols > 32)
            cols >>= 1;
        const int tc = (int)threadIdx.x & (cols - 1), tp = (int)threadIdx.x / cols, np = kThreads / cols;
        for (int pl = tp; pl < npair; pl += np) {
            const T *__restrict__ s0 = x + base + (int64_t)(2 * pl) * ddn;
            const T *__restrict__ s1 = s0 + (2 * pl + 1 < nrows ? ddn : 0);
            V2 *row = xp + pl * width;
            for (int d0 = tc; d0 < ddn; d0 += 4 * cols) {
                T v0[4], v1[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int d = min(d0 + u * cols, ddn - 1);
                    v0[u] = s0[d];
                    v1[u] = s1[d];
                }
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int d = min(d0 + u * cols, ddn - 1);
                    row[d] = V2{v0[u], v1[u]};
                    row[d + ddn + 1] = V2{-v0[u], -v1[u]};
                }
            }
        }
        for (int r = threadIdx.x; r < npair; r += kThreads)
            xp[r * width + ddn] = V2{(T)0, (T)0};
    } else {
        int rl = (int)threadIdx.x / ddn, d = (int)threadIdx.x - rl * ddn;
        for (int i0 = 0; i0 < n; i0 += 8 * kThreads) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const int i = i0 + u * kThreads + (int)threadIdx.x;
                v[u] = x[base + (i < n ? i : 0)];
            }
#pragma unroll
            for (int u = 0; u < 8; u++) {
                if (i0 + u * kThreads + (int)threadIdx.x < n)
                    xs[rl * (ddn + 1) + d] = v[u];
                d += kThreads;
                while (d >= ddn) {
                    d -= ddn;
                    rl++;
                }
            }
        }
        for (int r = threadIdx.x; r < nrows; r += kThreads)
            xs[r * (ddn + 1) + ddn] = (T)0;
    }
    // b_j from the update partials of step j - 1; b_{j-1} as recorded
    __shared__ T scal[2];
    if (threadIdx.x < 64) {
        const double bj = j >= 1 ? sqrt(inst_sum(in.part2, in.nparts2)) : 1.0;
        const double bjm1 = j >= 2 ? in.hist[2 * j - 3] : 1.0;
        const double s0 = bj > 0.0 ? 1.0 / bj : 0.0, s0_old = bjm1 > 0.0 ? 1.0 / bjm1 : 0.0;
        if (threadIdx.x == 0) {
            scal[0] = (T)s0;
            scal[1] = (T)(j >= 1 ? -bj * s0_old : 0.0);
        }
    }
    __syncthreads();
    if (stopped)
        return;
    const T a_s = scal[0], b_s = scal[1], tm = (T)(-in.t), U = (T)in.U;
    double acc = 0.0;
    if (PAIRS || in.dn_pair) {
        const V2 *xp = reinterpret_cast<const V2 *>(smem_raw);
        acc = narrow ? batch_pairs<T, NARROW>(in, it, x, y, xp, a_s, b_s) : batch_pairs<T, false>(in, it, x, y, xp, a_s, b_s);
        const double s = wg_sum(acc, red);
        if (threadIdx.x == 0)
            in.part[it.part] = s;
        return;
    }
    // tasks of a wave: 64 columns by a share of the rows, as many shares as
    // leave the four waves about the same number of tasks
    const int lane = (int)threadIdx.x & 63, nch = (ddn + 63) >> 6;
    const int shares = min(nrows, nch % 4 == 0 ? 1 : nch % 2 == 0 ? 2 : 4);
    for (int task = (int)threadIdx.x >> 6; task < nch * shares; task += kThreads / 64) {
        const int c = task % nch, sh = task / nch;
        const int d = c * 64 + lane;
        const bool ok = d < ddn;
        const int dc = ok ? d : ddn - 1;
        const int nq = __builtin_amdgcn_readfirstlane((int)in.dn_nq[c]);
        const uint4 *__restrict__ dn = in.dn_groups + dc;
        uint4 e4[2];
#pragma unroll
        for (int g = 0; g < 2; g++)
            e4[g] = dn[(size_t)(g < in.gmax ? g : 0) * (size_t)ddn];
        const uint32_t sd = in.states_dn[dc];
        const uint32_t off = (uint32_t)dc * (uint32_t)sizeof(T);
        for (int rl = __builtin_amdgcn_readfirstlane(sh * nrows / shares);
             rl < __builtin_amdgcn_readfirstlane((sh + 1) * nrows / shares); rl++) {
            const int64_t r = it.r0 + rl;
            const uint32_t *__restrict__ urow = in.up_tile + r * in.w_up;
            const int nu = in.nnz_up[r];
            auto row_at = [&](uint32_t e) -> T {
                const T *row = x + (int64_t)(e & 0x7fffffffu) * ddn;
                return *reinterpret_cast<const T *>(reinterpret_cast<const unsigned char *>(row) + off);
            };
            T uv[8];
#pragma unroll
            for (int u = 0; u < 8; u++)
                uv[u] = row_at(urow[u]);
            const int64_t J = base + (int64_t)rl * ddn + dc;
            const T yv = y[J];
            const T *__restrict__ xrow = xs + rl * (ddn + 1);
            const T xv = xrow[dc];
            T h = U * (T)__popc(in.states_up[r] & sd) * xv;
            auto group = [&](const uint4 &e) {
                const uint32_t ev[4] = {e.x, e.y, e.z, e.w};
                T v[8];
#pragma unroll
                for (int u = 0; u < 8; u++)
                    v[u] = xrow[(ev[u >> 1] >> ((u & 1) * 16)) & 0x7fffu];
#pragma unroll
                for (int u = 0; u < 8; u++)
                    h = fma(tm, with_sign(v[u], ((u & 1) ? ev[u >> 1] : ev[u >> 1] << 16) & 0x80000000u), h);
            };
#pragma unroll
            for (int g = 0; g < 2; g++)
                if (g < nq)
                    group(e4[g]);
            for (int g = 2; g < nq; g++)
                group(dn[(size_t)g * (size_t)ddn]);
            // slots past the row's count repeat its last hop's row and add
            // nothing (selected: a branch would take the load with it)
            for (int k0 = 0; k0 < nu; k0 += 8) {
                T nv[8];
                if (k0 + 8 < nu)
#pragma unroll
                    for (int u = 0; u < 8; u++)
                        nv[u] = row_at(urow[k0 + 8 + u]);
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    const T w = fma(tm, with_sign(uv[u], urow[k0 + u] & 0x80000000u), h);
                    h = k0 + u < nu ? w : h;
                }
#pragma unroll
                for (int u = 0; u < 8; u++)
                    uv[u] = nv[u];
            }
            const T q = fma(a_s, h, b_s * yv);
            if (ok) {
                y[J] = q;
                acc += (double)q * (double)xv;
            }
        }
    }
    const double s = wg_sum(acc, red);
    if (threadIdx.x == 0)
        in.part[it.part] = s;
}

// q <- q - a_j f_j with a_j from the H.v partial sums (recorded by the
// instance's first item), and the partial sums of |q|^2.  Items of their own:
// elements [r0, r0 + nrows) of the vector, on 16 bytes.
template <typename T>
__global__ __launch_bounds__(kThreads) void batch_axpy_kernel(const BatchInst *__restrict__ insts,
                                                              const BatchItem *__restrict__ items, int k)
{
    constexpr int E = 16 / (int)sizeof(T);
    typedef __attribute__((ext_vector_type(E))) T vec;
    __shared__ double red[kThreads / 64];
    const BatchItem it = items[blockIdx.x];
    const BatchInst &in = insts[it.inst];
    const BatchState *st = in.st;
    if (st->stopped)
        return;
    const int j = in.j0 + k;
    const T *__restrict__ v = reinterpret_cast<const T *>((j & 1) ? in.vec1 : in.vec0) + it.r0;
    T *__restrict__ w = reinterpret_cast<T *>((j & 1) ? in.vec0 : in.vec1) + it.r0;
    const vec *vv = reinterpret_cast<const vec *>(v);
    vec *wv = reinterpret_cast<vec *>(w);
    const int n = (int)it.nrows, nv = n / E;
    // the first vectors are loaded before the sums, which they do not need
    vec a = (vec)(T)0, b = (vec)(T)0;
    if ((int)threadIdx.x < nv) {
        a = wv[threadIdx.x];
        b = vv[threadIdx.x];
    }
    const double bj = j >= 1 ? in.hist[2 * j - 1] : 1.0;
    const double s0 = bj > 0.0 ? 1.0 / bj : 0.0;
    const double aj = inst_sum(in.part, in.nparts) * s0;
    if (it.part == 0 && threadIdx.x == 0)
        in.hist[2 * j] = aj;
    const T c = (T)(aj * s0);
    double acc = 0.0;
    for (int i = threadIdx.x; i < nv; i += kThreads) {
        vec q = a;
        const vec f = b;
        if (i + kThreads < nv) {
            a = wv[i + kThreads];
            b = vv[i + kThreads];
        }
#pragma unroll
        for (int e = 0; e < E; e++) {
            q[e] = q[e] - c * f[e];
            acc += (double)q[e] * (double)q[e];
        }
        wv[i] = q;
    }
    for (int i = nv * E + (int)threadIdx.x; i < n; i += kThreads) {
        const T q = w[i] - c * v[i];
        w[i] = q;
        acc += (double)q * (double)q;
    }
    const double s = wg_sum(acc, red);
    if (threadIdx.x == 0)
        in.part2[it.part] = s;
}

// T_m as the Ritz value reads it, scaled by 1/sigma (a power of two no smaller
// than any |a|, b): diagonal dg[i] and squared off-diagonal o2[i] (coupling of
// i-1 and i), staged in LDS when T_m is short enough (every step of the recurrence
// then reads LDS, not global memory), else read from the recorded coefficients.
constexpr int kRitzLds = 512;
struct TriView {
    const double *dg, *o2;     // LDS copies (m <= kRitzLds), or null
    const double *hist;        // a at 2i, b at 2i + 1
    double inv;                // 1 / sigma
    __device__ double d(int i) const { return dg ? dg[i] : hist[2 * i] * inv; }
    __device__ double e2(int i) const
    {
        if (o2)
            return o2[i];
        const double e = hist[2 * i - 1] * inv;
        return e * e;
    }
};

// Whether T_m has an eigenvalue below each of P points (or at one): the leading
// minors p_i of T_m - x I, p_i = (d_i - x) p_{i-1} - e_i^2 p_{i-2}, are all positive
// exactly when it has none (Sylvester).  The chain is one FMA per row (pivots
// would be a division per row, five times the latency), and the P chains hide
// each other's; every 16 rows both terms are scaled by a power of two.
template <int P>
__device__ void eigenvalue_below(const TriView &t, int m, const double *x, bool *below)
{
    double p0[P], p1[P];
#pragma unroll
    for (int k = 0; k < P; k++) {
        p0[k] = 1.0;
        p1[k] = t.d(0) - x[k];
        below[k] = !(p1[k] > 0.0);
    }
    auto row = [&](double d, double e2) {
#pragma unroll
        for (int k = 0; k < P; k++) {
            const double q = fma(d - x[k], p1[k], -e2 * p0[k]);
            below[k] = below[k] || !(q > 0.0);
            p0[k] = p1[k];
            p1[k] = q;
        }
    };
    for (int i0 = 1; i0 < m; i0 += 16) {
        if (t.dg) {
            // eight rows' coefficients in flight at a time (padded past m)
#pragma unroll
            for (int b = 0; b < 16; b += 8) {
                double d[8], e2[8];
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    d[i] = t.dg[i0 + b + i];
                    e2[i] = t.o2[i0 + b + i];
                }
#pragma unroll
                for (int i = 0; i < 8; i++)
                    row(d[i], e2[i]);
            }
        } else {
            for (int i = i0; i < min(i0 + 16, m); i++)
                row(t.d(i), t.e2(i));
        }
#pragma unroll
        for (int k = 0; k < P; k++) {
            const int ex = -__builtin_amdgcn_frexp_exp(p1[k]);
            p0[k] = ldexp(p0[k], ex);
            p1[k] = ldexp(p1[k], ex);
        }
    }
}

// Lowest eigenvalue of T_m (scaled) by multisection: the workgroup tests P * blockDim.x
// points of the bracket [lo, hi] (no eigenvalue below lo, at least one below hi),
// and the bracket shrinks to the two points around the first one with an
// eigenvalue below it, until no double lies strictly inside.  Returns hi, as the
// host's bisection does.  The bracket starts just below the previous step's value
// e_prev (by Cauchy interlacing the lowest eigenvalue of T_m is at most that of
// T_{m-1}), four times the last change wide, when the first round's end points
// confirm it; otherwise it is the Gershgorin interval.
__device__ double lowest_eigenvalue(const TriView &t, int m, double e_prev, double e_prev2, double *sh, int *first)
{
    constexpr int P = 2;
    const int np = (int)blockDim.x * P;
    const double one = t.inv;  // 1 in scaled units, the floor of the brackets' scale
    bool warm = m >= 3;
    double lo = 0.0, hi = 0.0;
    if (warm) {
        const double scale = fmax(one, fabs(e_prev));
        lo = e_prev - fmax(4.0 * fabs(e_prev - e_prev2), 1e-12 * scale);
        hi = e_prev + 4.0 * 0x1p-52 * scale;
    }
    for (int round = 0; round < 80; round++) {
        if (round == 0 && !warm) {
            if (threadIdx.x == 0) {
                double l = t.d(0), h = t.d(0);
                for (int i = 0; i < m; i++) {
                    const double rad = (i > 0 ? sqrt(t.e2(i)) : 0.0) + (i < m - 1 ? sqrt(t.e2(i + 1)) : 0.0);
                    l = fmin(l, t.d(i) - rad);
                    h = fmax(h, t.d(i) + rad);
                }
                const double pad = 0x1p-52 * (fabs(l) + fabs(h)) + 1e-290;
                sh[0] = l - pad;
                sh[1] = h + pad;
            }
            __syncthreads();
            lo = sh[0];
            hi = sh[1];
        }
        if (!warm && !(nextafter(lo, INFINITY) < hi))
            break;
        // points inside the bracket; the warm round includes its ends
        auto point = [&](int k) {
            const double f = warm ? (double)k / (double)(np - 1) : (double)(k + 1) / (double)(np + 1);
            return fmin(hi, fmax(lo, lo + (hi - lo) * f));
        };
        double x[P];
        bool below[P];
#pragma unroll
        for (int k = 0; k < P; k++)
            x[k] = point((int)threadIdx.x * P + k);
        if (threadIdx.x == 0)
            *first = np;
        __syncthreads();
        eigenvalue_below<P>(t, m, x, below);
        int mine = np;
#pragma unroll
        for (int k = P - 1; k >= 0; k--)
            if (below[k])
                mine = (int)threadIdx.x * P + k;
        if (mine < np)
            atomicMin(first, mine);
        __syncthreads();
        const int f = *first;
        __syncthreads();
        if (warm && (f == 0 || f == np)) {
            warm = false;  // not confirmed
            round = -1;
            continue;
        }
        const double nlo = f == 0 ? lo : point(f - 1), nhi = f == np ? hi : point(f);
        warm = false;
        if (nlo == lo && nhi == hi)
            break;
        lo = nlo;
        hi = nhi;
    }
    return hi;
}

// One workgroup per instance, beside step j's H.v: the end of step j - 1.
// b_j from the update partials, the Ritz value E_{j-1} of T_j (a_1..a_j,
// b_2..b_j), then the single-instance driver's stop tests in its order; the
// mailbox gets {a, b, E, code}.  A stop keeps every later kernel off the
// instance.
__device__ __forceinline__ void ritz_and_stop(const BatchInst &in, int j, double *__restrict__ mailbox)
{
    __shared__ double sh[2];
    __shared__ int first;
    BatchState *st = in.st;
    double *mb = mailbox + 4 * in.slot;
    if (st->stopped || j == 0) {
        if (threadIdx.x == 0) {
            mb[0] = mb[1] = mb[2] = 0.0;
            mb[3] = st->stopped ? kMailStopped : kMailNone;
        }
        return;
    }
    const int j0 = j - 1;  // the step finished here (0-based)
    const double b = sqrt(inst_sum(in.part2, in.nparts2));
    const double a = in.hist[2 * j0];
    if (threadIdx.x == 0)
        in.hist[2 * j0 + 1] = b;
    __syncthreads();
    const int m = j0 + 1;
    double code = kMailRunning;
    double e = 0.0;
    if (!isfinite(a) || !isfinite(b)) {
        code = kMailBad;
    } else {
        __shared__ double dg[kRitzLds + 16], o2[kRitzLds + 16];
        // sigma: a power of two above every coefficient
        __shared__ int top;
        if (threadIdx.x == 0)
            top = -1100;
        __syncthreads();
        int ex = -1100;
        for (int i = threadIdx.x; i < m; i += blockDim.x) {
            const double big = fmax(fabs(in.hist[2 * i]), i > 0 ? in.hist[2 * i - 1] : 0.0);
            if (big > 0.0)
                ex = max(ex, __builtin_amdgcn_frexp_exp(big));
        }
        for (int off = 32; off > 0; off >>= 1)
            ex = max(ex, __shfl_xor(ex, off, 64));
        if ((threadIdx.x & 63) == 0)
            atomicMax(&top, ex);
        __syncthreads();
        const int sx = top > -1100 ? top : 0;
        TriView t{nullptr, nullptr, in.hist, ldexp(1.0, -sx)};
        if (m <= kRitzLds) {
            // rows past m, up to a block of 16, keep the minors positive: d above
            // every point, no coupling
            for (int i = threadIdx.x; i < m + 16; i += blockDim.x) {
                dg[i] = i < m ? in.hist[2 * i] * t.inv : 8.0;
                const double o = i > 0 && i < m ? in.hist[2 * i - 1] * t.inv : 0.0;
                o2[i] = o * o;
            }
            __syncthreads();
            t.dg = dg;
            t.o2 = o2;
        }
        e = ldexp(lowest_eigenvalue(t, m, st->e_prev * t.inv, st->e_prev2 * t.inv, sh, &first), sx);
    }
    if (threadIdx.x == 0) {
        if (code == kMailRunning) {
            if (in.tol >= 0.0 && m >= 2 && fabs(e - st->e_prev) <= in.tol * fmax(1.0, fabs(e))) {
                code = HUBBARD_STOP_CONVERGED;
            } else {
                st->scale = fmax(st->scale, fabs(a) + (m > 1 ? in.hist[2 * j0 - 1] : 0.0));
                if (b == 0.0 || b <= 1e-12 * st->scale)
                    code = HUBBARD_STOP_BREAKDOWN;
                else if ((int64_t)m >= in.dim)
                    code = HUBBARD_STOP_EXHAUSTED;
                else if (m >= in.max_iter)
                    code = HUBBARD_STOP_MAXITER;
            }
        }
        st->e_prev2 = st->e_prev;
        st->e_prev = e;
        st->j = m;
        if (code != kMailRunning)
            st->stopped = 1;
        mb[0] = a;
        mb[1] = b;
        mb[2] = e;
        mb[3] = code;
    }
}

// Start vectors of the instances that joined, for all of them in two launches
// over their update items: the partial sums of |f|^2, then f_1 = f / |f| in the
// working precision (Alg. 1), the zero vector before it and the instance's state;
// the squared norm goes to host memory for the host's check.
__global__ __launch_bounds__(kThreads) void batch_norm_kernel(const BatchInst *__restrict__ insts,
                                                              const BatchItem *__restrict__ items)
{
    __shared__ double red[kThreads / 64];
    const BatchItem it = items[blockIdx.x];
    const BatchInst &in = insts[it.inst];
    double acc = 0.0;
    for (int64_t i = it.r0 + threadIdx.x; i < it.r0 + it.nrows; i += kThreads) {
        const double f = start_or_given(in.start, in.seed, i);
        acc += f * f;
    }
    const double s = wg_sum(acc, red);
    if (threadIdx.x == 0)
        in.part2[it.part] = s;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void batch_fill_kernel(const BatchInst *__restrict__ insts,
                                                              const BatchItem *__restrict__ items,
                                                              double *__restrict__ norms)
{
    const BatchItem it = items[blockIdx.x];
    const BatchInst &in = insts[it.inst];
    const double nrm2 = inst_sum(in.part2, in.nparts2), c = 1.0 / sqrt(nrm2);
    T *v0 = reinterpret_cast<T *>(in.vec0), *v1 = reinterpret_cast<T *>(in.vec1);
    for (int64_t i = it.r0 + threadIdx.x; i < it.r0 + it.nrows; i += kThreads) {
        v0[i] = (T)(c * start_or_given(in.start, in.seed, i));
        v1[i] = (T)0;
    }
    if (it.part == 0 && threadIdx.x == 0) {
        BatchState *st = in.st;
        st->scale = 0.0;
        st->e_prev = 0.0;
        st->e_prev2 = 0.0;
        st->j = 0;
        st->stopped = 0;
        norms[in.slot] = nrm2;
    }
}

}  // namespace

template <typename T>
void launch_batch_step(BatchInst *insts_dev, int n_inst, const BatchItem *items_dev, int n_items, int n_upd,
                       size_t lds_bytes, bool pairs, bool narrow, double *mailbox_dev, int k, hipStream_t s)
{
    auto hv = narrow ? (pairs ? batch_hv_kernel<T, true, true> : batch_hv_kernel<T, false, true>)
                     : (pairs ? batch_hv_kernel<T, true, false> : batch_hv_kernel<T, false, false>);
    if (lds_bytes > 64 * 1024)
        HUB_HIP(hipFuncSetAttribute((const void *)hv, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes));
    hipLaunchKernelGGL(hv, dim3(n_inst + n_items), dim3(kThreads), lds_bytes, s, insts_dev, items_dev, n_inst, k,
                       mailbox_dev);
    HUB_HIP(hipGetLastError());
    hipLaunchKernelGGL(batch_axpy_kernel<T>, dim3(n_upd), dim3(kThreads), 0, s, insts_dev, items_dev + n_items, k);
    HUB_HIP(hipGetLastError());
}

template void launch_batch_step<double>(BatchInst *, int, const BatchItem *, int, int, size_t, bool, bool, double *, int,
                                         hipStream_t);
template void launch_batch_step<float>(BatchInst *, int, const BatchItem *, int, int, size_t, bool, bool, double *, int,
                                        hipStream_t);

template <typename T>
void launch_batch_start(BatchInst *insts_dev, const BatchItem *items_dev, int n_items, double *norms_dev, hipStream_t s)
{
    hipLaunchKernelGGL(batch_norm_kernel, dim3(n_items), dim3(kThreads), 0, s, insts_dev, items_dev);
    HUB_HIP(hipGetLastError());
    hipLaunchKernelGGL(batch_fill_kernel<T>, dim3(n_items), dim3(kThreads), 0, s, insts_dev, items_dev, norms_dev);
    HUB_HIP(hipGetLastError());
}
template void launch_batch_start<double>(BatchInst *, const BatchItem *, int, double *, hipStream_t);
template void launch_batch_start<float>(BatchInst *, const BatchItem *, int, double *, hipStream_t);

}  // namespace hub
