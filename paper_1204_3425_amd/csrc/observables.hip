// Site observables of a state: the occupations n_{i sigma} and their products,
// which are diagonal in the configuration basis (Sec. 1, eq. H; Sec. 2.1: bit i
// of a spin's configuration word is the occupation of site i).
//
// With w_J = psi_J^2 over the dim_up x dim_dn view of psi (J = r * dim_dn + d),
//   UU[i][j] = sum_J w_J bit_i(up_r) bit_j(up_r)     <n_{i up} n_{j up}>
//   DD[i][j] = sum_J w_J bit_i(dn_d) bit_j(dn_d)     <n_{i dn} n_{j dn}>
//   C[i][j]  = sum_J w_J bit_i(up_r) bit_j(dn_d)     <n_{i up} n_{j dn}>
//   norm     = sum_J w_J
// (unnormalised).  One pass reads psi once, and its sums run on the matrix
// cores: the occupation bits of four up rows are the 16 x 4 operand U (0 or 1, so
// every product is exact), w of those rows in 16 columns the 4 x 16 operand, and
//   A_i(x) = sum_r bit_i(up_r) w(r, x)
// accumulates over the rows in FP64.  With the rows' totals R_r (a rotation sum
// over the 16 lanes that hold a row) UU takes one more product per four rows, U
// times (U^T R).  A tile of columns ends with C = sum_x A_i(x) bit_j(dn_x) and DD =
// sum_x q(x) bit_i(dn_x) bit_j(dn_x), q(x) the column totals, again as products,
// from LDS.  A workgroup takes a range of rows, its four waves every fourth
// group of four, and one or more tiles of columns; it writes one partial of
// 3 * NS * NS + 1 values and a second kernel sums the partials in a fixed order,
// so the result is reproducible.
//
// What bounds it: reading psi (4x4 6u6d, 513 MB: 100 us at the 5.1 TB/s of a large
// copy).  Per 512 elements a wave spends nine products of 16 x 16 x 4 and about
// fifty vector instructions, half of what the memory allows.  The form before
// this one added w to 16 sums per element on the vector units, with a wave
// reduction and 16 conversions and products for UU per 128 elements, and took
// 322 us (1.6 TB/s).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "internal.h"

namespace hub {

template <int NS>
constexpr int obs_partial_size()
{
    return 3 * NS * NS + 1;
}

typedef __attribute__((ext_vector_type(4))) double d4;
constexpr int kObsThreads = 256;
// columns of a tile: its sums A take eight (NS = 16) or two times four accumulators
template <int NS>
constexpr int obs_tile()
{
    return NS <= 16 ? 128 : 64;
}

// v plus the values of the other 15 lanes of its row of 16 (in every lane)
__device__ inline double row16_sum(double v)
{
    auto add = [&](auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), C, 0xf, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), C, 0xf, 0xf, false);
        v += __hiloint2double(hi, lo);
    };
    // row rotations by 8, 4, 2 and 1
    add(std::integral_constant<int, 0x128>());
    add(std::integral_constant<int, 0x124>());
    add(std::integral_constant<int, 0x122>());
    add(std::integral_constant<int, 0x121>());
    return v;
}

// Operands of the 16 x 16 x 4 product (lane l): A[l % 16][l / 16], B[l / 16][l % 16];
// element v of the accumulator is D[4 v + l / 16][l % 16].
// E = 2: a lane loads two neighbouring columns (16 bytes; even dim_dn, psi on 16
// bytes), which go to two accumulators; E = 1 otherwise.
template <int NS, int E>
__global__ __launch_bounds__(kObsThreads, NS <= 16 ? 3 : 2) void obs_accumulate_kernel(const double *__restrict__ psi,
                                                                     const uint32_t *__restrict__ states_up,
                                                                     const uint32_t *__restrict__ states_dn,
                                                                     int64_t dim_up, int64_t dim_dn, int ntiles,
                                                                     int ncols, int64_t rows_per,
                                                                     double *__restrict__ part)
{
    constexpr int NH = NS / 16, XT = obs_tile<NS>(), NT = XT / 16, NL = NT / E, NW = kObsThreads / 64;
    typedef typename std::conditional<E == 2, double2, double>::type V;
    __shared__ double a_lds[NS][XT + 1];
    __shared__ double q_lds[XT];
    __shared__ uint32_t dn_lds[XT];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15, kk = lane >> 4;
    // workgroup: column range of tiles, row range
    const int cg = blockIdx.x % ncols;
    const int64_t rbeg = (int64_t)(blockIdx.x / ncols) * rows_per;
    const int64_t rend = rbeg + rows_per < dim_up ? rbeg + rows_per : dim_up;
    const int t0 = (int)((int64_t)cg * ntiles / ncols), t1 = (int)((int64_t)(cg + 1) * ntiles / ncols);
    d4 UU[NH][NH], C[NH][NH], DD[NH][NH];
#pragma unroll
    for (int h = 0; h < NH; h++)
#pragma unroll
        for (int g = 0; g < NH; g++)
            UU[h][g] = C[h][g] = DD[h][g] = (d4)0.0;
    double norm = 0.0;
    for (int t = t0; t < t1; t++) {
        const int64_t x0 = (int64_t)t * XT;
        d4 A[NH][NT];
        double q[NT];
#pragma unroll
        for (int m = 0; m < NT; m++) {
            q[m] = 0.0;
#pragma unroll
            for (int h = 0; h < NH; h++)
                A[h][m] = (d4)0.0;
        }
        // four rows from r, one per 16 lanes; past the range (and the columns) an
        // element in range is read and weighted 0
        auto load = [&](int64_t r, V (&v)[NL], uint32_t &up) {
            const int64_t row = min(r + kk, dim_up - 1);
            const double *p = psi + row * dim_dn;
#pragma unroll
            for (int m = 0; m < NL; m++) {
                const int64_t x = x0 + (16 * m + n) * E;
                v[m] = *reinterpret_cast<const V *>(p + (x < dim_dn ? x : 0));
            }
            up = states_up[row];
        };
        V v[NL], vn[NL];
        uint32_t up = 0, upn = 0;
        int64_t r = rbeg + 4 * wave;
        if (r < rend)
            load(r, v, up);
        for (; r < rend; r += 4 * NW) {
            load(r + 4 * NW, vn, upn);
            const bool ok = r + kk < rend;
            double w[NT], R = 0.0;
#pragma unroll
            for (int m = 0; m < NL; m++) {
                const bool in = ok && x0 + (16 * m + n) * E < dim_dn;
                const double *e = reinterpret_cast<const double *>(&v[m]);
#pragma unroll
                for (int k = 0; k < E; k++) {
                    const double y = in ? e[k] : 0.0;
                    w[m * E + k] = y * y;
                    q[m * E + k] += w[m * E + k];
                    R += w[m * E + k];
                }
            }
            R = row16_sum(R);
            double u[NH];
#pragma unroll
            for (int h = 0; h < NH; h++)
                u[h] = (double)((up >> (16 * h + n)) & 1u);
#pragma unroll
            for (int h = 0; h < NH; h++) {
#pragma unroll
                for (int m = 0; m < NT; m++)
                    A[h][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[h], w[m], A[h][m], 0, 0, 0);
#pragma unroll
                for (int g = 0; g < NH; g++)
                    UU[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[h], u[g] * R, UU[h][g], 0, 0, 0);
            }
#pragma unroll
            for (int m = 0; m < NL; m++)
                v[m] = vn[m];
            up = upn;
        }
        // the waves' A and q added up in LDS, one wave at a time
        for (int x = threadIdx.x; x < XT; x += kObsThreads)
            dn_lds[x] = x0 + x < dim_dn ? states_dn[x0 + x] : 0u;
        for (int k = 0; k < NW; k++) {
            if (wave == k) {
#pragma unroll
                for (int m = 0; m < NT; m++) {
                    const int x = (16 * (m / E) + n) * E + m % E;
#pragma unroll
                    for (int h = 0; h < NH; h++)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            double &a = a_lds[16 * h + 4 * e + kk][x];
                            a = k == 0 ? A[h][m][e] : a + A[h][m][e];
                        }
                    double s = q[m];
                    s += __shfl_xor(s, 16, 64);
                    s += __shfl_xor(s, 32, 64);
                    if (kk == 0)
                        q_lds[x] = k == 0 ? s : q_lds[x] + s;
                }
            }
            __syncthreads();
        }
        // C and DD over the tile, four columns per product, the waves taking turns
        for (int c = wave; c < XT / 4; c += NW) {
            const int x = 4 * c + kk;
            const uint32_t dn = dn_lds[x];
            const double qx = q_lds[x];
            double bit[NH];
#pragma unroll
            for (int h = 0; h < NH; h++)
                bit[h] = (double)((dn >> (16 * h + n)) & 1u);
#pragma unroll
            for (int h = 0; h < NH; h++) {
                const double ax = a_lds[16 * h + n][x];
#pragma unroll
                for (int g = 0; g < NH; g++) {
                    C[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax, bit[g], C[h][g], 0, 0, 0);
                    DD[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(qx * bit[h], bit[g], DD[h][g], 0, 0, 0);
                }
            }
            if (n == 0)
                norm += qx;
        }
        __syncthreads();
    }
    // the waves' sums, one wave at a time, straight to the partial
    double *out = part + (int64_t)blockIdx.x * obs_partial_size<NS>();
    __shared__ double nw[NW];
    for (int off = 32; off > 0; off >>= 1)
        norm += __shfl_down(norm, off, 64);
    if (lane == 0)
        nw[wave] = norm;
    double *acc = &a_lds[0][0];  // NS * NS values
    auto sum_out = [&](const d4 (&m)[NH][NH], int at) {
        for (int k = 0; k < NW; k++) {
            if (wave == k)
#pragma unroll
                for (int h = 0; h < NH; h++)
#pragma unroll
                    for (int g = 0; g < NH; g++)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            double &a = acc[(16 * h + 4 * e + kk) * NS + 16 * g + n];
                            a = k == 0 ? m[h][g][e] : a + m[h][g][e];
                        }
            __syncthreads();
        }
        for (int e = threadIdx.x; e < NS * NS; e += kObsThreads)
            out[at + e] = acc[e];
        __syncthreads();
    };
    sum_out(UU, 0);
    sum_out(DD, NS * NS);
    sum_out(C, 2 * NS * NS);
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int k = 0; k < NW; k++)
            s += nw[k];
        out[3 * NS * NS] = s;
    }
}

// Sum of the per-workgroup partials in a fixed order: a workgroup takes eight
// elements, 32 threads each adding every 32nd partial, then the 32 in order.
constexpr int kObsSumElems = 8;

__global__ __launch_bounds__(256) void obs_sum_kernel(const double *__restrict__ part, int nparts, int psize,
                                                      double *__restrict__ out)
{
    __shared__ double red[256 / kObsSumElems][kObsSumElems];
    const int i = threadIdx.x % kObsSumElems, g = threadIdx.x / kObsSumElems, G = 256 / kObsSumElems;
    const int e = blockIdx.x * kObsSumElems + i;
    double s = 0.0;
    if (e < psize) {
#pragma unroll 8
        for (int b = g; b < nparts; b += G)
            s += part[(int64_t)b * psize + e];
    }
    red[g][i] = s;
    __syncthreads();
    if (g == 0 && e < psize) {
        s = red[0][i];
        for (int k = 1; k < G; k++)
            s += red[k][i];
        out[e] = s;
    }
}

int obs_ns_max(int sites) { return sites <= 16 ? 16 : 32; }

// Workgroups: as many column ranges as there are tiles (one or more tiles
// each), and row ranges of a multiple of 16 rows to make up max_blocks.
static void obs_grid(int ns, int64_t dim_up, int64_t dim_dn, int &ntiles, int &ncols, int64_t &rows_per, int &nblocks,
                     int max_blocks)
{
    const int xt = ns <= 16 ? obs_tile<16>() : obs_tile<32>();
    ntiles = (int)((dim_dn + xt - 1) / xt);
    ncols = std::min(ntiles, max_blocks);
    const int64_t nr = std::max<int64_t>(1, max_blocks / ncols);
    rows_per = ((dim_up + nr - 1) / nr + 15) / 16 * 16;
    nblocks = ncols * (int)((dim_up + rows_per - 1) / rows_per);
}

int obs_partial_count(int ns, int64_t dim_up, int64_t dim_dn, int max_blocks)
{
    int ntiles, ncols, nblocks;
    int64_t rows_per;
    obs_grid(ns, dim_up, dim_dn, ntiles, ncols, rows_per, nblocks, max_blocks);
    return nblocks;
}

template <int NS>
static void launch_obs(const double *psi, const uint32_t *states_up, const uint32_t *states_dn, int64_t dim_up,
                       int64_t dim_dn, double *part, double *out, int max_blocks, hipStream_t s)
{
    int ntiles, ncols, nblocks;
    int64_t rows_per;
    obs_grid(NS, dim_up, dim_dn, ntiles, ncols, rows_per, nblocks, max_blocks);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(nblocks), dim3(kObsThreads), 0, s, psi, states_up, states_dn, dim_up, dim_dn,
                           ntiles, ncols, rows_per, part);
        HUB_HIP(hipGetLastError());
    };
    if (dim_dn % 2 == 0 && (uintptr_t)psi % 16 == 0)
        go(obs_accumulate_kernel<NS, 2>);
    else
        go(obs_accumulate_kernel<NS, 1>);
    const int ps = obs_partial_size<NS>();
    hipLaunchKernelGGL(obs_sum_kernel, dim3((ps + kObsSumElems - 1) / kObsSumElems), dim3(256), 0, s, part, nblocks, ps,
                       out);
    HUB_HIP(hipGetLastError());
}

void launch_observables(const double *psi, const uint32_t *states_up, const uint32_t *states_dn, int ns,
                        int64_t dim_up, int64_t dim_dn, double *part, double *out, int max_blocks, hipStream_t s)
{
    if (ns <= 16)
        launch_obs<16>(psi, states_up, states_dn, dim_up, dim_dn, part, out, max_blocks, s);
    else
        launch_obs<32>(psi, states_up, states_dn, dim_up, dim_dn, part, out, max_blocks, s);
}

// Scratch of the entry point that allocates nothing (hubbard_observables_noalloc):
// the workgroups' partial sums and the final sums live in this
// array, one copy per device for the life of the process.  Host code never
// passes the array's name to a kernel: its device address comes from
// hipGetSymbolAddress, taken once per device with that device current.
static __device__ __align__(256) double scratch[kObsScratchBytes / sizeof(double)];

static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kObsMaxDevices] = {};

double *obs_scratch(int device)
{
    if (device < 0 || device >= kObsMaxDevices)
        fail(HUBBARD_EDEVICE, "device index out of range for the observables scratch");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            fail(HUBBARD_EDEVICE, std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
        g_scratch_ptr[device] = ptr;
    }
    return static_cast<double *>(g_scratch_ptr[device]);
}

int obs_noalloc_blocks(int ns, int64_t dim_up, int64_t dim_dn)
{
    (void)dim_up;
    (void)dim_dn;
    const int ps = ns <= 16 ? obs_partial_size<16>() : obs_partial_size<32>();
    // partials and the final sums must fit the scratch
    const int64_t cap = (int64_t)(kObsScratchBytes / sizeof(double)) / ps - 1;
    return (int)std::min<int64_t>(kObsDefaultBlocks, cap);
}

}  // namespace hub
