// One-launch H.v for small and medium sectors (gfx950).
//
// With the state vector viewed as the dim_up x dim_dn matrix X (Siro & Harju,
// Sec. 4.3, Fig. slots) a workgroup owns one row.  It stages the row in LDS for
// the down-spin hops; the up-spin hops read whole row segments of x from
// memory, the row's entries arriving as scalars (they are the same for all of
// its columns).  A vector of such a sector stays in the L2s and the Infinity
// Cache, which makes re-reading its rows cheaper than the second pass over y
// (and, for a caller's dense rows, the copy to padded ones) that the two-pass
// form needs.
//
// What bounds it (14-site ring, 11.8 M states, FP64, 98 us): the lines the
// up-spin hops miss in the L2s, 0.7 GB per H.v at about 7 TB/s, and beside them
// the L1, busy 64 % of the time with the row segments and the table entries;
// the LDS is busy 16 % and the vector units 36 %.  So the loads are what is
// arranged: a column's entries and its first eight up-spin rows are issued
// together before the gathers, and each XCD takes a contiguous range of rows.
// Two or four rows per workgroup (one table entry for all of them) were slower
// (108 us FP64; FP32 65 and 87 us against 60), and so were entries split by sign
// (102 us): the table is not what the kernel waits for.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace hub {

namespace {

constexpr int kTileLds = 160 * 1024;

// sign bit of a 16-bit entry (low or high half of e) moved to bit 31
__device__ inline uint32_t entry_sign(uint32_t e, int half) { return (half ? e : e << 16) & 0x80000000u; }
__device__ inline float with_sign(float v, uint32_t sg) { return __int_as_float(__float_as_int(v) ^ (int)sg); }
__device__ inline double with_sign(double v, uint32_t sg)
{
    return __hiloint2double(__double2hiint(v) ^ (int)sg, __double2loint(v));
}

// Sum of part[0..n) in a fixed order, by one wave (every lane gets it): every
// wave of every workgroup that needs it forms the same value, so no launch and
// no barrier is spent on it.
__device__ inline double wave_total(const double *__restrict__ part, int n)
{
    double s = 0.0;
    for (int i = threadIdx.x & 63; i < n; i += 64)
        s += part[i];
    for (int off = 32; off > 0; off >>= 1)
        s += __shfl_xor(s, off, 64);
    return s;
}

__device__ inline double recip_norm(double b) { return b > 1e-300 ? 1.0 / b : 0.0; }

// Sum over the workgroup (fixed order), in thread 0.
__device__ inline double tile_sum(double v, double *red)
{
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); w++)
            s += red[w];
    __syncthreads();
    return s;
}

struct TileArgs {
    const uint16_t *nnz_up;
    const uint32_t *states_up;
    int64_t dim_up;
    int dim_dn, w_up, gmax;  // slots per up row, groups per column
    int nseg, span;          // workgroups per row, columns of each (a multiple of 64)
    double t, U;
    int64_t pair;  // element offset of the second half of a complex vector (gridDim.y = 2)
};

// GT: per-bond amplitudes.  The entries of all columns are laid out in slots
// of one amplitude each, so a slot's amplitude is a scalar; up-spin entries
// carry the class in bits 24..30.
template <typename T, int MODE, bool GT>
__global__ __launch_bounds__(1024) void hv_tile_kernel(TileArgs p, const uint4 *__restrict__ dn,
                                                       const uint8_t *__restrict__ dn_nq,
                                                       const double *__restrict__ dn_amp,
                                                       const uint32_t *__restrict__ up_rows,
                                                       const double *__restrict__ tcls,
                                                       const uint32_t *__restrict__ states_dn,
                                                       const T *__restrict__ x, int64_t ldx, const T *prev, T *out,
                                                       int64_t ldy, double shift, TileStep st)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *xs = reinterpret_cast<T *>(smem_raw);
    __shared__ double red[16];
    const int ddn = p.dim_dn, nth = (int)blockDim.x, tid = (int)threadIdx.x;
    if (blockIdx.y) {
        x += p.pair;
        out += p.pair;
        prev += p.pair;
    }
    // workgroup i runs on XCD i mod 8: each XCD takes a contiguous range of
    // rows, so the rows that neighbouring rows hop to are in its L2.  Where rows
    // are few, nseg workgroups share a row, each taking a range of its columns.
    const int unit = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    const int64_t r = unit / p.nseg;
    const int c0 = (unit % p.nseg) * p.span, c1 = min(c0 + p.span, ddn);
    const bool mine = r < p.dim_up;
    double acc0 = 0.0, acc1 = 0.0;
    T a_s = (T)1, b_s = (T)0;
    if (mine) {
        const T *xr = x + r * ldx;
        for (int d0 = 0; d0 < ddn; d0 += 4 * nth) {
            T v[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int d = d0 + u * nth + tid;
                v[u] = d < ddn ? xr[d] : (T)0;
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int d = d0 + u * nth + tid;
                if (d < ddn)
                    xs[d] = v[u];
            }
        }
        if (tid == 0)
            xs[ddn] = (T)0;  // the zero slot that padding entries point at
    }
    if (MODE == HV_LANCZOS) {
        // the scalars of step j: b_j is the norm of x (its partial sums), a
        // start vector of unit norm excepted; alpha = 1/b_j, beta = -b_j/b_{j-1}
        const double bj = st.j == 0 && st.unit ? 1.0 : sqrt(wave_total(st.norm2, st.n_norm2));
        const double bm = st.j > 0 ? st.b[st.j - 1] : 1.0;
        a_s = (T)recip_norm(bj);
        b_s = (T)(st.j > 0 ? -bj * recip_norm(bm) : 0.0);
        if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
            st.b[st.j] = bj;
            if (st.host_b)
                st.host_b[2 * st.j] = bj;
        }
    }
    __syncthreads();
    if (mine) {
        const T tm = (T)(-p.t), U = (T)p.U;
        constexpr uint32_t cmask = GT ? kClassColMask : 0x7fffffffu;
        constexpr int UB = 8;  // up-spin loads in flight before the down-spin gathers
        const uint32_t su = p.states_up[r];
        const int nu = p.nnz_up[r];
        const uint32_t *__restrict__ urow = up_rows + r * p.w_up;
        // factor of an up-spin entry: its sign (-t multiplies the sum), or -+ its amplitude
        auto coeff = [&](uint32_t e) -> T {
            if (GT) {
                const T a = (T)tcls[(e >> 24) & 0x7fu];
                return (e >> 31) ? a : -a;
            }
            return (e >> 31) ? (T)-1 : (T)1;
        };
        // the first hops of the row, in scalars for all of its columns
        uint32_t ue[UB];
        T uc[UB];
#pragma unroll
        for (int u = 0; u < UB; u++) {
            ue[u] = urow[u];
            uc[u] = coeff(ue[u]);
        }
        // amplitudes of the first two groups of slots
        T sa[16];
        if (GT)
#pragma unroll
            for (int u = 0; u < 16; u++)
                sa[u] = -(T)dn_amp[u];
        for (int d = c0 + tid; d < c1; d += nth) {
            const uint32_t off = (uint32_t)d * (uint32_t)sizeof(T);
            auto row_at = [&](uint32_t e) -> T {
                const T *row = x + (int64_t)(e & cmask) * ldx;
                return *reinterpret_cast<const T *>(reinterpret_cast<const unsigned char *>(row) + off);
            };
            // the down-spin entries first, then the first up-spin rows, which
            // stay in flight while the down-spin hops are summed; every load is
            // issued (groups past a column chunk's count read group 0, slots
            // past a row's count its last hop's row again, both unused), so the
            // wait counters stay exact
            uint4 e4[2];
#pragma unroll
            for (int g = 0; g < 2; g++)
                e4[g] = dn[(size_t)(g < p.gmax ? g : 0) * (size_t)ddn + (size_t)d];
            const int nq = __builtin_amdgcn_readfirstlane((int)dn_nq[d >> 6]);
            const uint32_t sd = states_dn[d];
            T uv[UB];
#pragma unroll
            for (int u = 0; u < UB; u++)
                uv[u] = row_at(ue[u]);
            const T xv = xs[d];
            // the hops are summed first (with one amplitude as +-x, exact
            // factors) and join the interaction term in one rounding
            T h = (T)0, h1 = (T)0;
            auto group = [&](const uint4 &e, auto &&amp) {
                const uint32_t ev[4] = {e.x, e.y, e.z, e.w};
                T v[8];
#pragma unroll
                for (int u = 0; u < 8; u++)
                    v[u] = xs[(ev[u >> 1] >> ((u & 1) * 16)) & 0x7fffu];
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    T &acc = (u & 1) ? h1 : h;
                    const T w = with_sign(v[u], entry_sign(ev[u >> 1], u & 1));
                    acc = GT ? fma(amp(u), w, acc) : acc + w;
                }
            };
#pragma unroll
            for (int g = 0; g < 2; g++)
                if (g < nq)
                    group(e4[g], [&](int u) { return sa[8 * g + u]; });
            for (int g = 2; g < nq; g++)
                group(dn[(size_t)g * (size_t)ddn + (size_t)d], [&](int u) { return -(T)dn_amp[8 * g + u]; });
#pragma unroll
            for (int u = 0; u < UB; u++)
                if (u < nu) {
                    T &acc = (u & 1) ? h1 : h;
                    acc = fma(uc[u], uv[u], acc);
                }
            for (int k = UB; k < nu; k += 4) {
                T v[4];
#pragma unroll
                for (int u = 0; u < 4; u++)
                    v[u] = row_at(urow[k + u]);
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (k + u < nu)
                        h = fma(coeff(urow[k + u]), v[u], h);
            }
            const T ud = U * (T)__popc(su & sd);
            h = GT ? fma(ud, xv, h + h1) : fma(tm, h + h1, ud * xv);
            const int64_t J = r * ldy + d;
            if (MODE == HV_STORE) {
                out[J] = h;
            } else if (MODE == HV_LANCZOS) {
                const T w = st.j > 0 ? a_s * h + b_s * prev[J] : a_s * h;
                out[J] = w;
                acc0 += (double)w * (double)xv;
            } else {
                const double z = (double)h - shift * (double)xv;
                acc0 += z * z;
                acc1 += (double)xv * (double)h;
            }
        }
    }
    if (MODE != HV_STORE) {
        const int b = (int)(blockIdx.y * gridDim.x + blockIdx.x);
        const double s0 = tile_sum(acc0, red);
        if (tid == 0)
            st.part[b] = s0;
        if (MODE == HV_RESIDUAL) {
            const double s1 = tile_sum(acc1, red);
            if (tid == 0)
                st.part[gridDim.x * gridDim.y + b] = s1;
        }
    }
}

}  // namespace

// One row per workgroup.  Threads: 512; 256 where FP32 rows leave room for
// eight workgroups or more on a CU (14-site ring 62 -> 60 us, 4x4 8u4d 206 ->
// 182); 1024 where a row takes more than half of the LDS (FP64 4x4 4u8d, rows
// of 12,870: 1024 threads 347 us, 512 508).
TilePlan make_tile_plan(const HvArgs &a, int elem_bytes)
{
    TilePlan pl;
    const int64_t ddn = a.dim_dn;
    const bool gt = a.tcls != nullptr;
    pl.lds = (size_t)(ddn + 1) * (size_t)elem_bytes;
    if ((gt ? a.dn_slots == nullptr : a.dn_groups16 == nullptr) || !a.up_tile || pl.lds > kTileLds - 512)
        return pl;
    if (a.dim_up * ddn * elem_bytes > kTileMaxBytes && (!gt || a.ncls <= kTwoPassClasses))
        return pl;
    // per-bond slots hold every class a column might have: on sparse sectors
    // most are empty (24-site ring, 2 electrons, 24 amplitudes: 24 slots for 4
    // hops, 11.6 us against 10.7 in the one-pass kernel)
    if (gt && a.dn_slot_groups * 8 > 4 * std::max(a.w_dn, 4) && a.ncls > kTwoPassClasses)
        return pl;
    const int64_t want = pl.lds > kTileLds / 2 ? 1024 : elem_bytes == 4 && pl.lds <= kTileLds / 8 ? 256 : 512;
    pl.threads = (int)std::min<int64_t>(want, (ddn + 63) / 64 * 64);
    // fewer rows than two workgroups per CU: split the columns, down to one
    // pass of the threads each (4x4 1u8d 27 -> 10 us)
    const int64_t most = (ddn + pl.threads - 1) / pl.threads;
    const int64_t seg = std::max<int64_t>(1, std::min(most, 512 / a.dim_up));
    pl.span = (int)(((ddn + seg - 1) / seg + 63) / 64 * 64);
    pl.nseg = (int)((ddn + pl.span - 1) / pl.span);
    pl.grid = 8 * (int)((a.dim_up * pl.nseg + 7) / 8);
    pl.ok = true;
    return pl;
}

template <typename T>
void launch_hv_tile(const HvArgs &a, const TilePlan &pl, const T *x, int64_t ldx, const T *prev, T *out, int64_t ldy,
                    int mode, double shift, const TileStep &st, int64_t pair, hipStream_t s)
{
    TileArgs p;
    const bool gt = a.tcls != nullptr;
    p.nseg = pl.nseg;
    p.span = pl.span;
    p.gmax = gt ? a.dn_slot_groups : std::max((a.w_dn + 7) / 8, 1);
    p.w_up = a.up_tile_w;
    p.nnz_up = a.nnz_up;
    p.states_up = a.states_up;
    p.dim_up = a.dim_up;
    p.dim_dn = (int)a.dim_dn;
    p.t = a.t;
    p.U = a.U;
    p.pair = pair;
    auto go = [&](auto kern) {
        if (pl.lds > 64 * 1024)
            HUB_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds));
        hipLaunchKernelGGL(kern, dim3(pl.grid, pair ? 2 : 1), dim3(pl.threads), pl.lds, s, p,
                           gt ? a.dn_slots : a.dn_groups16, gt ? a.dn_slot_nq : a.dn_nq8, a.dn_slot_amp, a.up_tile,
                           a.tcls, a.states_dn, x, ldx, prev, out, ldy,
                           shift, st);
        HUB_HIP(hipGetLastError());
    };
    auto by_mode = [&](auto gtc) {
        constexpr bool GT = decltype(gtc)::value;
        if (mode == HV_STORE)
            go(hv_tile_kernel<T, HV_STORE, GT>);
        else if (mode == HV_LANCZOS)
            go(hv_tile_kernel<T, HV_LANCZOS, GT>);
        else
            go(hv_tile_kernel<T, HV_RESIDUAL, GT>);
    };
    if (gt)
        by_mode(std::true_type());
    else
        by_mode(std::false_type());
}

template void launch_hv_tile<double>(const HvArgs &, const TilePlan &, const double *, int64_t, const double *,
                                     double *, int64_t, int, double, const TileStep &, int64_t, hipStream_t);
template void launch_hv_tile<float>(const HvArgs &, const TilePlan &, const float *, int64_t, const float *, float *,
                                    int64_t, int, double, const TileStep &, int64_t, hipStream_t);

}  // namespace hub
