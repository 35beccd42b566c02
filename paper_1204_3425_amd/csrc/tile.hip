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
// What bounds it (14-site ring, 11.8 M states, FP64, 95 us): the lines the
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
constexpr int kTileWaves = 16;  // of the largest workgroup

// Static LDS of hv_tile_kernel beside the staged row: one value per wave of each
// of its na sums (1 + 2 ND of a step with ND lower vectors, two of a residual).
constexpr int tile_red_bytes(int na) { return (int)sizeof(double) * kTileWaves * na; }
// kept free of the row in every plan: the sums of a step with one lower vector
constexpr int kTileLdsSpare = 512;
static_assert(tile_red_bytes(1 + 2 * 1) <= kTileLdsSpare && tile_red_bytes(2) <= kTileLdsSpare, "");

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
    // eight loads in flight (past the end: element 0, not added)
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
    double t, U, qscale;
    int64_t pair;            // element offset of the second half of a complex vector (gridDim.y = 2)
    const double *psi;       // deflated step: nd dense vectors, vector l at psi + l * pdim
    int nd;
    int64_t pdim;
};

// Sum over the workgroup of N values, one of each per thread (fixed order), in
// thread 0.
template <int N>
__device__ inline void tile_sums(double (&v)[N], double (*red)[N])
{
#pragma unroll
    for (int k = 0; k < N; k++)
        for (int off = 32; off > 0; off >>= 1)
            v[k] += __shfl_down(v[k], off, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < N; k++)
            red[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < (int)(blockDim.x >> 6); w++)
#pragma unroll
            for (int k = 0; k < N; k++)
                v[k] += red[w][k];
}

// GT: per-bond amplitudes.  The entries of all columns are laid out in slots
// of one amplitude each, so a slot's amplitude is a scalar; up-spin entries
// carry the class in bits 24..30.
// dn: [g][d] -> eight 16-bit entries (element index | sign << 15), dn_nq: groups
// per 64 columns, dn_amp: amplitude of each slot (GT, eight per group); up_rows:
// w_up slots per row, those past its count repeating its last hop; tcls:
// amplitude of each class (GT).  ND: room for lower vectors of a deflated step.
// HV_LANCZOS with the factor qscale on q.x (in the common kernel the factor would
// cost registers it does not have: 3x4 6u6d solve 2121 -> 2157 us).
constexpr int HV_LANCZOS_SCALED = 16;

// Waves a SIMD has to hold.  FP32 with amplitudes: 88 registers in a step where a
// product has 80, and a CU then held two workgroups of rows that leave it room for
// three (4x4 t-t' 3u8d, 51 KB rows: 223 us a step's H.v against a product's 154).
template <typename T, bool GT, int ND>
constexpr int tile_simd_waves()
{
    return sizeof(T) == 8 || ND > 0 ? 4 : GT ? 6 : 8;
}

template <typename T, int MODE, bool GT, int ND>
__global__ __launch_bounds__(64 * kTileWaves, (tile_simd_waves<T, GT, ND>()))
void hv_tile_kernel(TileArgs p, const uint4 *__restrict__ dn,
                                                       const uint8_t *__restrict__ dn_nq,
                                                       const double *__restrict__ dn_amp,
                                                       const uint32_t *__restrict__ up_rows,
                                                       const double *__restrict__ tcls,
                                                       const uint32_t *__restrict__ states_dn,
                                                       const T *__restrict__ x, int64_t ldx, T *__restrict__ out,
                                                       int64_t ldy, double shift, double *__restrict__ part)
{
    constexpr bool SCALED = MODE == HV_LANCZOS_SCALED, LANCZOS = MODE == HV_LANCZOS || SCALED;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *xs = reinterpret_cast<T *>(smem_raw);
    const int ddn = p.dim_dn, nth = (int)blockDim.x, tid = (int)threadIdx.x;
    if (blockIdx.y) {
        x += p.pair;
        out += p.pair;
    }
    // workgroup i runs on XCD i mod 8: each XCD takes a contiguous range of
    // rows, so the rows that neighbouring rows hop to are in its L2.  Where rows
    // are few, nseg workgroups share a row, each taking a range of its columns.
    const int unit = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    const bool mine = unit < p.nseg * p.dim_up;
    const int64_t r = mine ? unit / p.nseg : 0;
    const int c0 = mine ? (unit % p.nseg) * p.span : 0, c1 = mine ? min(c0 + p.span, ddn) : c0;

    const T tm = (T)(-p.t), U = (T)p.U;
    constexpr uint32_t cmask = GT ? kClassColMask : 0x7fffffffu;
    constexpr int UB = 8;  // up-spin rows in flight before the down-spin gathers
    // down-spin gathers at once, and up-spin rows in flight after the first
    // eight: with eight of each an FP64 wave needs 75 registers (14-site ring
    // 99 -> 95 us with four); FP32 has room (4x4 t-t' 4u4d 61 us, with four 74)
    constexpr int GB = sizeof(T) == 8 ? 4 : 8, LB = GB;
    const uint32_t su = p.states_up[r];
    const int nu = p.nnz_up[r];
    const uint32_t *__restrict__ urow = up_rows + r * p.w_up;
    // amplitude of an up-spin entry (GT)
    auto amp_of = [&](uint32_t e) -> T { return GT ? -(T)tcls[(e >> 24) & 0x7fu] : (T)1; };
    // the first hops of the row, in scalars for all of its columns
    uint32_t ue[UB];
    T uc[UB];
#pragma unroll
    for (int u = 0; u < UB; u++) {
        ue[u] = urow[u];
        uc[u] = amp_of(ue[u]);
    }
    // amplitudes of the first two groups of slots
    T sa[16];
    if (GT)
#pragma unroll
        for (int u = 0; u < 16; u++)
            sa[u] = -(T)dn_amp[u];
    auto row_at = [&](uint32_t e, uint32_t off) -> T {
        const T *row = x + (int64_t)(e & cmask) * ldx;
        return *reinterpret_cast<const T *>(reinterpret_cast<const unsigned char *>(row) + off);
    };
    // A column's entries, configuration and first up-spin rows.  Every load is
    // issued (columns past the end read the last one, groups past the table
    // group 0, slots past a row's count its last hop's row again, all unused),
    // so the wait counters stay exact.
    uint4 e4[2];
    uint32_t sd;
    int nq;
    T uv[UB];
    auto fetch = [&](int d) {
        const int dc = d < ddn ? d : ddn - 1;
#pragma unroll
        for (int g = 0; g < 2; g++)
            e4[g] = dn[(size_t)(g < p.gmax ? g : 0) * (size_t)ddn + (size_t)dc];
        nq = (int)dn_nq[dc >> 6];
        sd = states_dn[dc];
#pragma unroll
        for (int u = 0; u < UB; u++)
            uv[u] = row_at(ue[u], (uint32_t)dc * (uint32_t)sizeof(T));
    };
    // the row itself, and the first column's loads behind it, before the barrier
    {
        const T *xr = x + r * ldx;
        constexpr int CH = 4;
        for (int d0 = 0; d0 < ddn; d0 += CH * nth) {
            T v[CH];
#pragma unroll
            for (int u = 0; u < CH; u++) {
                const int d = d0 + u * nth + tid;
                v[u] = d < ddn ? xr[d] : (T)0;
            }
            if (d0 == 0)
                fetch(c0 + tid);
#pragma unroll
            for (int u = 0; u < CH; u++) {
                const int d = d0 + u * nth + tid;
                if (d < ddn)
                    xs[d] = v[u];
            }
        }
        if (tid == 0)
            xs[ddn] = (T)0;  // the zero slot that padding entries point at
        // the result rows' padding, which the update pass reads
        if (LANCZOS && mine && c1 == ddn && ddn + tid < ldy)
            out[r * ldy + ddn + tid] = (T)0;
    }
    __syncthreads();
    // partial sums: q.x (and psi_l.q, psi_l.x of a deflated step), or z.z and x.Hx
    constexpr int NA = MODE == HV_RESIDUAL ? 2 : 1 + 2 * ND;
    double acc[NA];
#pragma unroll
    for (int k = 0; k < NA; k++)
        acc[k] = 0.0;
    for (int d0 = c0; d0 < c1; d0 += nth) {
        const int d = d0 + tid;
        const bool ok = d < c1;
        const int dc = ok ? d : ddn - 1;
        // psi_l at this element, in flight while the hops are summed
        double pv[ND > 0 ? ND : 1];
        if (ND > 0)
#pragma unroll
            for (int l = 0; l < ND; l++)
                pv[l] = p.psi[(int64_t)(l < p.nd ? l : 0) * p.pdim + r * ddn + dc];
        const T xv = xs[dc];
        // the hops are summed first (with one amplitude as +-x, exact factors)
        // and join the interaction term in one rounding
        T h = (T)0, h1 = (T)0;
        auto group = [&](const uint4 &e, auto &&amp) {
            const uint32_t ev[4] = {e.x, e.y, e.z, e.w};
            T v[8];
#pragma unroll
            for (int b = 0; b < 8; b += GB) {
#pragma unroll
                for (int u = b; u < b + GB; u++)
                    v[u] = xs[(ev[u >> 1] >> ((u & 1) * 16)) & 0x7fffu];
#pragma unroll
                for (int u = b; u < b + GB; u++) {
                    T &a = (u & 1) ? h1 : h;
                    const T w = with_sign(v[u], entry_sign(ev[u >> 1], u & 1));
                    a = GT ? fma(amp(u), w, a) : a + w;
                }
            }
        };
        const int nqs = __builtin_amdgcn_readfirstlane(nq);
#pragma unroll
        for (int g = 0; g < 2; g++)
            if (g < nqs)
                group(e4[g], [&](int u) { return sa[8 * g + u]; });
        for (int g = 2; g < nqs; g++)
            group(dn[(size_t)g * (size_t)ddn + (size_t)dc], [&](int u) { return -(T)dn_amp[8 * g + u]; });
        // up-spin hops, eight rows in flight; a last, partial batch selects
        // (branching over single hops would let the compiler move each load
        // into its branch, one wait per hop)
        const uint32_t off = (uint32_t)dc * (uint32_t)sizeof(T);
        auto add = [&](auto &v, int k, auto &&ent, auto &&amp) {
            constexpr int N = (int)(sizeof(v) / sizeof(T));
            auto one = [&](int u, T a) {
                const T w = with_sign(v[u], ent(u) & 0x80000000u);
                return GT ? fma(amp(u), w, a) : a + w;
            };
            if (k + N <= nu) {
#pragma unroll
                for (int u = 0; u < N; u++) {
                    T &a = (u & 1) ? h1 : h;
                    a = one(u, a);
                }
            } else {
#pragma unroll
                for (int u = 0; u < N; u++) {
                    T &a = (u & 1) ? h1 : h;
                    const T w = one(u, a);
                    a = k + u < nu ? w : a;
                }
            }
        };
        auto later = [&](int k) {
            T v2[LB];
#pragma unroll
            for (int u = 0; u < LB; u++)
                v2[u] = row_at(urow[k + u], off);
            if (k == UB)
                add(uv, 0, [&](int u) { return ue[u]; }, [&](int u) { return uc[u]; });
            add(v2, k, [&](int u) { return urow[k + u]; }, [&](int u) { return amp_of(urow[k + u]); });
        };
        if (nu > UB) {
            later(UB);
            for (int k = UB + LB; k < nu; k += LB)
                later(k);
        } else {
            add(uv, 0, [&](int u) { return ue[u]; }, [&](int u) { return uc[u]; });
        }
        const T ud = U * (T)__popc(su & sd);
        h = GT ? fma(ud, xv, h + h1) : fma(tm, h + h1, ud * xv);
        if (d0 + nth < c1)
            fetch(d + nth);
        if (ok) {
            if (MODE != HV_RESIDUAL)
                out[r * ldy + d] = h;
            if (LANCZOS) {
                acc[0] += (SCALED ? (double)h * p.qscale : (double)h) * (double)xv;
#pragma unroll
                for (int l = 0; l < ND; l++) {
                    acc[1 + 2 * l] += (double)h * pv[l];
                    acc[2 + 2 * l] += (double)xv * pv[l];
                }
            } else if (MODE == HV_RESIDUAL) {
                const double z = (double)h - shift * (double)xv;
                acc[0] += z * z;
                acc[NA - 1] += (double)xv * (double)h;
            }
        }
    }
    if (MODE != HV_STORE) {
        __shared__ double red[kTileWaves][NA];
        static_assert(sizeof(red) == tile_red_bytes(NA), "");
        tile_sums<NA>(acc, red);
        const int b = (int)(blockIdx.y * gridDim.x + blockIdx.x), nb = (int)(gridDim.x * gridDim.y);
        if (tid == 0)
#pragma unroll
            for (int k = 0; k < NA; k++)
                if (MODE == HV_RESIDUAL || k <= 2 * p.nd)
                    part[(int64_t)k * nb + b] = acc[k];
    }
}

// The other half of a step.  With x_j = b_j f_j stored, q = H x_j and the sums
// part (q.x) and norm2 (|x_j|^2) known, b_j = |x_j|, a_j = q.x / b_j^2 and
//     x_{j+1} = q / b_j - (a_j / b_j) x_j - (b_j / b_{j-1}) x_{j-1}
// (formed in FP64, rounded once), with the partial sums of |x_{j+1}|^2.  Every
// workgroup forms the scalars itself from the same sums in the same order, so
// no launch is spent on them and the H.v needs none: on sectors of this size a
// launch, and a chain of dependent loads in front of the H.v, cost as much as
// the arithmetic.  A deflated step (ND > 0) takes sum_l g_l psi_l off as well,
// g_l = psi_l.x_{j+1} from the H.v's sums psi_l.q and psi_l.x_j of this step and
// psi_l.x_{j-1} of the one before: without the last two, which are rounding
// errors of the earlier projections, those would grow from step to step.
constexpr int kUpdThreads = 256;

template <typename T, int ND>
__global__ __launch_bounds__(kUpdThreads) void tile_update_kernel(T *__restrict__ q, const T *__restrict__ x,
                                                                  const T *__restrict__ xp, int64_t dim_up,
                                                                  int64_t dim_dn, int64_t ld, int halves, TileStep st,
                                                                  const double *__restrict__ psi, int nd)
{
    constexpr int E = 16 / (int)sizeof(T), NW = kUpdThreads / 64, NT = 2 + 3 * ND;
    typedef __attribute__((ext_vector_type(E))) T vec;
    __shared__ double tot[NT];
    __shared__ double red[NW];
    const int wave = (int)threadIdx.x >> 6;
    // the first vectors are loaded before the sums, which they do not need
    const int64_t nv = (int64_t)halves * dim_up * ld / E, stride = (int64_t)gridDim.x * kUpdThreads;
    vec *qv = reinterpret_cast<vec *>(q);
    const vec *xv = reinterpret_cast<const vec *>(x), *pv = reinterpret_cast<const vec *>(st.j > 0 ? xp : x);
    int64_t i = (int64_t)blockIdx.x * kUpdThreads + threadIdx.x;
    vec qn, xn, pn;
    auto load = [&](int64_t at) {
        const int64_t k = at < nv ? at : nv - 1;
        qn = qv[k];
        xn = xv[k];
        pn = pv[k];
    };
    if (ND == 0)
        load(i);
    // the sums, one per wave at a time
    for (int k = wave; k < 2 + 3 * nd; k += NW) {
        double s = 0.0;
        if (k == 0)
            s = st.j > 0 || !st.unit ? wave_total(st.norm2, st.n_norm2) : 1.0;
        else if (k == 1)
            s = wave_total(st.part, st.n_part);
        else if ((k - 2) % 3 < 2)  // psi_l.q, psi_l.x_j
            s = wave_total(st.part + (int64_t)(1 + 2 * ((k - 2) / 3) + (k - 2) % 3) * st.n_part, st.n_part);
        else if (st.j > 0)  // psi_l.x_{j-1}
            s = wave_total(st.part_prev + (int64_t)(2 + 2 * ((k - 2) / 3)) * st.n_part, st.n_part);
        if ((threadIdx.x & 63) == 0)
            tot[k] = s;
    }
    __syncthreads();
    const double bj = sqrt(tot[0]), s = recip_norm(bj), a = tot[1] * s * s * st.qunscale;
    const double c = a * s, e = st.j > 0 ? bj * recip_norm(st.b[st.j - 1]) : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st.b[st.j] = bj;
        st.hist[2 * st.j] = bj;
        st.hist[2 * st.j + 1] = a;
    }
    double acc = 0.0;
    if constexpr (ND == 0) {
        // e is 0 in step 0, where x stands in for the vector before it
        while (i < nv) {
            vec w;
#pragma unroll
            for (int k = 0; k < E; k++) {
                w[k] = (T)(s * (double)qn[k] - c * (double)xn[k] - e * (double)pn[k]);
                acc += (double)w[k] * (double)w[k];
            }
            qv[i] = w;
            i += stride;
            if (i < nv)
                load(i);
        }
    } else {
        double g[ND];
#pragma unroll
        for (int l = 0; l < ND; l++)
            g[l] = l < nd ? s * tot[2 + 3 * l] - c * tot[3 + 3 * l] - e * tot[4 + 3 * l] : 0.0;
        const int64_t dim = dim_up * dim_dn;
        for (int64_t r = blockIdx.x; r < dim_up; r += gridDim.x)
            for (int64_t d = threadIdx.x; d < dim_dn; d += kUpdThreads) {
                const int64_t i = r * ld + d;
                const double pn = st.j > 0 ? (double)xp[i] : 0.0;
                double v = s * (double)q[i] - c * (double)x[i] - e * pn;
                double w[ND];
#pragma unroll
                for (int l = 0; l < ND; l++)
                    w[l] = psi[(int64_t)(l < nd ? l : 0) * dim + r * dim_dn + d];
#pragma unroll
                for (int l = 0; l < ND; l++)
                    v -= g[l] * w[l];
                const T t = (T)v;
                q[i] = t;
                acc += (double)t * (double)t;
            }
    }
    const double sum = tile_sum(acc, red);
    if (threadIdx.x == 0)
        st.norm2_out[blockIdx.x] = sum;
}

// Projection of a vector in FP64 (rows at stride ld, psi_l dense), for the
// start vector and for steps with more lower vectors than the kernels above
// take: partial sums of psi_l.q, then q <- q - sum_l (psi_l.q) psi_l with the
// partial sums of |q|^2.
template <typename T>
__global__ __launch_bounds__(kUpdThreads) void tile_defl_dots_kernel(const T *__restrict__ q,
                                                                     const double *__restrict__ psi, int nd,
                                                                     int64_t dim_up, int64_t dim_dn, int64_t ld,
                                                                     double *__restrict__ dots)
{
    __shared__ double red[kUpdThreads / 64];
    double acc[kMaxDeflate];
#pragma unroll
    for (int l = 0; l < kMaxDeflate; l++)
        acc[l] = 0.0;
    const int64_t dim = dim_up * dim_dn;
    for (int64_t r = blockIdx.x; r < dim_up; r += gridDim.x)
        for (int64_t d = threadIdx.x; d < dim_dn; d += kUpdThreads) {
            const double v = (double)q[r * ld + d];
            const double *p = psi + r * dim_dn + d;
#pragma unroll
            for (int l = 0; l < kMaxDeflate; l++)
                if (l < nd)
                    acc[l] += v * p[l * dim];
        }
    for (int l = 0; l < nd; l++) {
        const double sl = tile_sum(acc[l], red);
        if (threadIdx.x == 0)
            dots[(int64_t)l * gridDim.x + blockIdx.x] = sl;
    }
}

template <typename T>
__global__ __launch_bounds__(kUpdThreads) void tile_defl_update_kernel(T *__restrict__ q,
                                                                       const double *__restrict__ psi, int nd,
                                                                       int64_t dim_up, int64_t dim_dn, int64_t ld,
                                                                       const double *__restrict__ dots,
                                                                       double *__restrict__ norm2)
{
    __shared__ double red[kUpdThreads / 64];
    __shared__ double c[kMaxDeflate];
    for (int l = (int)threadIdx.x >> 6; l < nd; l += kUpdThreads / 64) {
        const double s = wave_total(dots + (int64_t)l * gridDim.x, (int)gridDim.x);
        if ((threadIdx.x & 63) == 0)
            c[l] = s;
    }
    __syncthreads();
    const int64_t dim = dim_up * dim_dn;
    double acc = 0.0;
    for (int64_t r = blockIdx.x; r < dim_up; r += gridDim.x)
        for (int64_t d = threadIdx.x; d < dim_dn; d += kUpdThreads) {
            double v = (double)q[r * ld + d];
            const double *p = psi + r * dim_dn + d;
#pragma unroll
            for (int l = 0; l < kMaxDeflate; l++)
                if (l < nd)
                    v -= c[l] * p[l * dim];
            const T t = (T)v;
            q[r * ld + d] = t;
            acc += (double)t * (double)t;
        }
    const double s = tile_sum(acc, red);
    if (threadIdx.x == 0)
        norm2[blockIdx.x] = s;
}

// b_j of the vector stored last, which no update forms (and, for what 1, a_j
// of an H.v that no update follows).
__global__ __launch_bounds__(64) void tile_scalar_kernel(TileStep st, int what)
{
    const double b = sqrt(st.j > 0 || !st.unit ? wave_total(st.norm2, st.n_norm2) : 1.0);
    const double s = recip_norm(b);
    const double a = what ? wave_total(st.part, st.n_part) * s * s * st.qunscale : 0.0;
    if (threadIdx.x == 0) {
        st.b[st.j] = b;
        st.hist[2 * st.j] = b;
        if (what)
            st.hist[2 * st.j + 1] = a;
    }
}

}  // namespace

// One row per workgroup.  Threads: 512; 256 where FP32 rows leave room for
// eight workgroups or more on a CU (14-site ring 62 -> 60 us, 4x4 8u4d 206 ->
// 182); 1024 where a row takes more than half of the LDS (FP64 4x4 4u8d, rows
// of 12,870: 1024 threads 347 us, 512 508), in FP32 without amplitudes a third
// (3x6 3u6d, rows of 18,564: 152 -> 121).  Many short rows are another matter:
// one or two passes of the threads leave the loads of the next pass nothing to hide
// behind, and half of the last pass idle.  They take the number of at most 256
// (twice that at most the row) with the fewest idle lanes in the last pass, the
// larger one of two (FP64, before / after: 16 sites with diagonals 8u3d, 560
// columns, 280 / 156 us; 17-site ring 8u3d, 680, 225 / 139; 20-site ring 5u3d, 1,140,
// 170 / 124; 18-site ring 9u2d, 153, 108 / 76; FP32 114 / 92, 91 / 77, 80 / 79 and 93 /
// 51).  Rows of 1,287 elements and more are even, and so are fewer rows than a
// few per CU (3x4 6u6d, 924 rows of 924: 192 threads 19.1 us, 512 17.9).
constexpr int64_t kTileManyRows = 1024, kTileShortRow = 1280;
TilePlan make_tile_plan(const HvArgs &a, int elem_bytes)
{
    TilePlan pl;
    const int64_t ddn = a.dim_dn;
    const bool gt = a.tcls != nullptr;
    pl.lds = (size_t)(ddn + 1) * (size_t)elem_bytes;
    if ((gt ? a.dn_slots == nullptr : a.dn_groups16 == nullptr) || !a.up_tile || pl.lds > kTileLds - kTileLdsSpare)
        return pl;
    if (a.dim_up * ddn * elem_bytes > kTileMaxBytes && (!gt || a.ncls <= kTwoPassClasses))
        return pl;
    // per-bond slots hold every class a column might have: on sparse sectors
    // most are empty (24-site ring, 2 electrons, 24 amplitudes: 24 slots for 4
    // hops, 11.6 us against 10.7 in the one-pass kernel)
    if (gt && a.dn_slot_groups * 8 > 4 * std::max(a.w_dn, 4) && a.ncls > kTwoPassClasses)
        return pl;
    const bool fp32 = elem_bytes == 4;
    const int64_t want = pl.lds > kTileLds / 2 || (fp32 && !gt && pl.lds > kTileLds / 3) ? 1024
                         : fp32 && pl.lds <= kTileLds / 12                               ? 256
                                                                                         : 512;
    pl.threads = (int)std::min<int64_t>(want, (ddn + 63) / 64 * 64);
    if (a.dim_up >= kTileManyRows && ddn < kTileShortRow) {
        int64_t least = (ddn + 63) / 64 * 64;
        pl.threads = 64;
        for (int t = 128; t <= 256 && 2 * t <= ddn; t += 64)
            if ((ddn + t - 1) / t * t <= least)
                pl.threads = t;
    }
    // fewer rows than two workgroups per CU: split the columns, down to one
    // pass of the threads each (4x4 1u8d 27 -> 10 us)
    const int64_t most = (ddn + pl.threads - 1) / pl.threads;
    const int64_t seg = std::max<int64_t>(1, std::min(most, 512 / a.dim_up));
    pl.span = (int)(((ddn + seg - 1) / seg + 63) / 64 * 64);
    pl.nseg = (int)((ddn + pl.span - 1) / pl.span);
    pl.grid = 8 * (int)((a.dim_up * pl.nseg + 7) / 8);
    // instances with room for 4, 2 and 1 lower vectors: the largest whose sums fit
    // beside the row (FP64 rows of 20,349 elements, 21 sites with 5 electrons, leave
    // 1,040 bytes, and the sums of four take 1,152); more lower vectors than that
    // are projected out by launches of their own
    pl.defl = kTileDefl;
    while (pl.defl > 1 && pl.lds + (size_t)tile_red_bytes(1 + 2 * pl.defl) > (size_t)kTileLds)
        pl.defl /= 2;
    pl.ok = true;
    return pl;
}

template <typename T>
void launch_hv_tile(const HvArgs &a, const TilePlan &pl, const T *x, int64_t ldx, T *out, int64_t ldy, int mode,
                    double shift, double *part, hipStream_t s, const double *psi, int nd, int64_t pair)
{
    if (nd > pl.defl)
        fail(HUBBARD_EDEVICE, "one-launch step: more lower vectors than the row length leaves room for");
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
    p.qscale = a.qscale;
    p.pair = pair;
    p.psi = psi;
    p.nd = nd;
    p.pdim = a.dim_up * a.dim_dn;
    auto go = [&](auto kern) {
        if (pl.lds > 64 * 1024)
            HUB_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds));
        hipLaunchKernelGGL(kern, dim3(pl.grid, pair ? 2 : 1), dim3(pl.threads), pl.lds, s, p,
                           gt ? a.dn_slots : a.dn_groups16, gt ? a.dn_slot_nq : a.dn_nq8, a.dn_slot_amp, a.up_tile,
                           a.tcls, a.states_dn, x, ldx, out, ldy, shift, part);
        HUB_HIP(hipGetLastError());
    };
    auto step = [&](auto gtc, auto mc) {
        constexpr bool GT = decltype(gtc)::value;
        constexpr int M = decltype(mc)::value;
        if (nd > 2)
            go(hv_tile_kernel<T, M, GT, kTileDefl>);
        else if (nd == 2)
            go(hv_tile_kernel<T, M, GT, 2>);
        else if (nd == 1)
            go(hv_tile_kernel<T, M, GT, 1>);
        else
            go(hv_tile_kernel<T, M, GT, 0>);
    };
    auto by_mode = [&](auto gtc) {
        constexpr bool GT = decltype(gtc)::value;
        if (mode == HV_STORE)
            go(hv_tile_kernel<T, HV_STORE, GT, 0>);
        else if (mode == HV_RESIDUAL)
            go(hv_tile_kernel<T, HV_RESIDUAL, GT, 0>);
        else if (a.qscale != 1.0)
            step(gtc, std::integral_constant<int, HV_LANCZOS_SCALED>());
        else
            step(gtc, std::integral_constant<int, HV_LANCZOS>());
    };
    if (gt)
        by_mode(std::true_type());
    else
        by_mode(std::false_type());
}

int tile_update_blocks(int64_t n, int elem_bytes)
{
    // two 16-byte vectors per thread or more, and no more partial sums than a
    // wave adds up in a few loads
    const int64_t b = (n * elem_bytes / 16 + 2 * kUpdThreads - 1) / (2 * kUpdThreads);
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, 1024));
}

int tile_defl_blocks(int64_t dim_up) { return (int)std::min<int64_t>(dim_up, 1024); }

template <typename T>
int launch_tile_update(T *q, const T *x, const T *xp, int64_t dim_up, int64_t dim_dn, int64_t ld, int halves,
                       const TileStep &st, hipStream_t s, const double *psi, int nd)
{
    const int nb = nd > 0 ? tile_defl_blocks(dim_up) : tile_update_blocks(halves * dim_up * ld, sizeof(T));
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(nb), dim3(kUpdThreads), 0, s, q, x, xp, dim_up, dim_dn, ld, halves, st, psi, nd);
    };
    if (nd > 2)
        go(tile_update_kernel<T, kTileDefl>);
    else if (nd == 2)
        go(tile_update_kernel<T, 2>);
    else if (nd == 1)
        go(tile_update_kernel<T, 1>);
    else
        go(tile_update_kernel<T, 0>);
    HUB_HIP(hipGetLastError());
    return nb;
}

template <typename T>
int launch_tile_project(T *q, const double *psi, int nd, int64_t dim_up, int64_t dim_dn, int64_t ld, double *dots,
                        double *norm2, hipStream_t s)
{
    const int nb = tile_defl_blocks(dim_up);
    hipLaunchKernelGGL(tile_defl_dots_kernel<T>, dim3(nb), dim3(kUpdThreads), 0, s, q, psi, nd, dim_up, dim_dn, ld,
                       dots);
    HUB_HIP(hipGetLastError());
    hipLaunchKernelGGL(tile_defl_update_kernel<T>, dim3(nb), dim3(kUpdThreads), 0, s, q, psi, nd, dim_up, dim_dn, ld,
                       dots, norm2);
    HUB_HIP(hipGetLastError());
    return nb;
}

void launch_tile_scalar(const TileStep &st, int what, hipStream_t s)
{
    hipLaunchKernelGGL(tile_scalar_kernel, dim3(1), dim3(64), 0, s, st, what);
    HUB_HIP(hipGetLastError());
}

#define HUB_TILE_INST(T)                                                                                             \
    template void launch_hv_tile<T>(const HvArgs &, const TilePlan &, const T *, int64_t, T *, int64_t, int, double, \
                                    double *, hipStream_t, const double *, int, int64_t);                            \
    template int launch_tile_update<T>(T *, const T *, const T *, int64_t, int64_t, int64_t, int, const TileStep &,  \
                                       hipStream_t, const double *, int);                                           \
    template int launch_tile_project<T>(T *, const double *, int, int64_t, int64_t, int64_t, double *, double *,     \
                                        hipStream_t);
HUB_TILE_INST(double)
HUB_TILE_INST(float)

}  // namespace hub
