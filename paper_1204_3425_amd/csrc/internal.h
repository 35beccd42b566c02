// Internal declarations of the Hubbard library (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/hubbard.h"

namespace hub {

// Error raised inside the library; converted to a return code at the ABI.
struct Error {
    int code;
    std::string msg;
};

[[noreturn]] void fail(int code, const std::string &msg);
void hip_check(hipError_t e, const char *what);
#define HUB_HIP(call) ::hub::hip_check((call), #call)

// One spin's basis and hopping table as built on the host.
struct SpinTable {
    int n = 0;                      // electrons of this spin
    int64_t dim = 0;                // C(sites, n)
    int32_t width = 0;              // ELL width = max entries of a row
    int64_t nnz = 0;
    std::vector<uint32_t> states;   // ascending configuration words
    std::vector<int32_t> col;       // column-major ELL: entry k of row r at k*dim + r
    std::vector<int8_t> sgn;        // +1 / -1, padding 0
    std::vector<uint16_t> row_nnz;  // entries used in each row
    std::vector<uint16_t> bond;     // column-major like col: the bond (edge index) of each entry
};

// Packed device form of a hopping entry: bits 0..30 column, bit 31 set when
// the element is +t (sgn = -1).
inline uint32_t pack_entry(int32_t col, int8_t sgn) { return (uint32_t)col | (sgn < 0 ? 0x80000000u : 0u); }
// With per-bond amplitudes (columns below 2^24): bits 24..30 hold the
// amplitude class, the element is -tcls[class] * sgn.
inline uint32_t pack_entry_class(int32_t col, int8_t sgn, int cls)
{
    return (uint32_t)col | ((uint32_t)cls << 24) | (sgn < 0 ? 0x80000000u : 0u);
}
constexpr uint32_t kClassColMask = 0x00FFFFFFu;
constexpr int kMaxAmpClasses = 127;
// per-bond handles with at most this many classes also get the two-pass tables
// (two class bits in the row-pass groups and the up-spin entries)
constexpr int kTwoPassClasses = 4;
// longest row the FP64 row pass stages in LDS (plus one zero slot: 160 KB)
constexpr int kRow64Max = 20000;

constexpr int kMaxBlockRows = 1024;  // rows of a block of the up-spin pass at most
constexpr int kClsGroups = 4;  // row pass by class: groups of eight per class and column at most

struct DeviceTables {
    uint32_t *states_up = nullptr, *states_dn = nullptr;
    uint32_t *up_rows = nullptr;   // row-major: entry k of row r at r*w_up + k (row entries are wave-uniform)
    uint32_t *dn_cols = nullptr;   // column-major: entry k of row d at k*dim_dn + d (coalesced across lanes)
    uint16_t *nnz_up = nullptr, *nnz_dn = nullptr;
    // down table for the row pass: groups of four entries holding the byte
    // offset of the source element in a staged row (FP64 and FP32 layouts),
    // sign in bit 31, padding pointing at the zero slot after the row
    uint32_t *dn_groups64 = nullptr, *dn_groups32 = nullptr;
    uint8_t *dn_nq = nullptr;      // groups needed by the 64 columns of a wave
    int dn_ngroups = 0;
    // the same table at half the size, for rows of at most 32767 elements:
    // groups of eight 16-bit entries (element index | sign<<15)
    uint16_t *dn_groups16 = nullptr;
    uint8_t *dn_nq8 = nullptr;     // groups of eight needed by the 64 columns of a wave
    // the same groups with the sign in the index (rows of at most 2,048 elements,
    // the batched engine's): element e of x, or ddn + 1 + e where the row's
    // negative follows it and its zero slot
    uint16_t *dn_pair16 = nullptr;
    // FP64 row pass (one amplitude, rows of at most kRow64Max elements): per
    // column the hops of sign + in groups of eight 16-bit element indices and
    // those of sign - in groups of four, each in ascending column order
    // (padding: the zero slot at index dim_dn), and per 64 columns the two
    // group counts (one byte each); dn_np, dn_nn: the largest counts
    uint16_t *dn_pidx = nullptr, *dn_nidx = nullptr;
    uint8_t *dn_pn = nullptr;
    // two amplitude classes: per column the hops of class 0 in groups of eight
    // 16-bit entries, then (from group slot dn_cls_g1 on) those of class 1; the
    // first entry of a word has its sign in bit 0 and its index above, the second
    // its sign in bit 31.  Group counts of both per 64 columns.
    uint16_t *dn_cls = nullptr;
    uint8_t *dn_cls_n = nullptr;
    int dn_cls_g1 = 0, dn_cls_ng = 0;
    int dn_np = 0, dn_nn = 0;
    // up table for the blocked slab pass: rows are grouped in blocks of equal
    // occupation of the top sites; per row the hops that stay in the block come
    // first (block-local row | sign<<31), then the others (row | sign<<31)
    uint32_t *up_blk = nullptr;
    uint16_t *up_nint = nullptr, *up_next = nullptr;
    int32_t *up_bstart = nullptr;  // nblocks + 1 row offsets
    int up_nblocks = 0, up_max_block = 0;
    // the same entries with one 32-slot line per row (two, 64 slots, for rows
    // of 33 to 64 hops, or where 32 slots leave no room for the padding):
    // internal hops from the front, external from the back; per row one word
    // with the internal and external counts and their largest values over the
    // row's group of eight (bytes 0..3).  Padded lines (up_line_ipad): the
    // slots past a row's internal count, up to the largest count of its group,
    // hold the block's zero row
    uint32_t *up_line = nullptr, *up_cnt = nullptr;
    // two amplitude classes: per row a padded line of 32 slots for each class and
    // a count word for each (null where a row's class has no room in 32)
    uint32_t *up_cls_line = nullptr, *up_cls_cnt = nullptr;
    // one-launch H.v: the up entries as up_tile_w slots per row (a multiple of
    // eight; slots past a row's count repeat its last hop), and for per-bond
    // handles the down entries in slots of one amplitude each: groups of eight
    // 16-bit entries like dn_groups16, the amplitude of every slot, and the
    // groups needed by the 64 columns of a wave
    uint32_t *up_tile = nullptr;
    int up_tile_w = 0;
    uint16_t *dn_slots = nullptr;
    double *dn_slot_amp = nullptr;
    uint8_t *dn_slot_nq = nullptr;
    int dn_slot_groups = 0;
    bool tile_only = false;  // no two-pass tables: every call takes the one-launch form
    size_t bytes = 0;
    double *tcls = nullptr;  // amplitude of each class (per-bond amplitudes only)
    int up_line_w = 32;      // slots per row of up_line (32 or 64)
    int up_line_ipad = 0;
};

// Device and pinned host buffers a handle keeps between its calls.  A solve
// that allocates its vectors anew each time is bound by it once it is repeated:
// the 227 MB chunks of a resident basis (3x4 6u6d) cost 1 ms a call in hipMalloc
// and hipFree, and 16 ms after some two hundred calls, when the driver no longer
// keeps up with clearing freed memory (2.9 -> 19.4 ms a solve).  Blocks given
// back are kept up to kKeepAll over all handles of the process, the oldest going
// first, and freed with the handle; a call that finds no block of its own handle
// takes one that another handle of the device keeps.  (With at most 1 GiB a
// handle the chunks of mid-sized sectors were allocated by every solve, faster
// than the driver clears them: 20-site ring 10u1d, 40 steps with psi, 12 to 1,800
// ms a call, now 11.)  take() hands out a kept block of at least the size asked
// for and at most twice that (a quarter more from 64 MiB on), else allocates.
// Where the device is full, an allocation of the library frees the kept blocks of
// every handle and tries again.  Safe from several threads; the work that used a
// block has to be complete when it is given back.
constexpr size_t kKeepAll = (size_t)8 << 30;
class Workspace {
  public:
    Workspace();
    Workspace(const Workspace &) = delete;
    Workspace &operator=(const Workspace &) = delete;
    void *take(size_t bytes, size_t *got);
    void *take_kept(size_t bytes, size_t *got);  // as take, or null where no kept block fits
    void *take_own(size_t bytes, size_t most, size_t *got);
    void give(void *p, size_t bytes);
    void *take_host(size_t bytes, size_t *got);
    void give_host(void *p, size_t bytes);
    void release();
    ~Workspace();
    int device = 0;  // of the handle: its calls run, and allocate, there
    // age of the oldest kept block (0: none), and freeing that one
    uint64_t oldest();
    void drop_oldest();

  private:
    struct Block {
        void *p;
        size_t bytes;
        uint64_t age;  // order of giving back over all handles, from 1
    };
    void drop(size_t k);
    std::mutex mu_;
    std::vector<Block> dev_, host_;
    size_t held_ = 0;
};

// Allocations of the library (pinned host memory: mapped and coherent); out of
// memory, they free what handles keep before they fail.
void *device_alloc(size_t bytes);
void *host_alloc(size_t bytes);
// Frees every handle's kept blocks.
void release_kept();

// Device buffer, from a handle's workspace or (null) an allocation of its own.
struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
    Workspace *ws = nullptr;
    DevBuf() = default;
    explicit DevBuf(size_t n, Workspace *w = nullptr);
    static std::unique_ptr<DevBuf> kept(size_t n, Workspace *w);  // null where w keeps none that fits
    ~DevBuf();
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    template <typename T>
    T *as() const { return static_cast<T *>(p); }
};

// Pinned host memory, mapped and coherent: kernels may write it directly
// (through dev), and the host reads it once the writing work has completed.
struct PinnedBuf {
    void *p = nullptr;
    void *dev = nullptr;
    size_t bytes = 0;
    Workspace *ws = nullptr;
    explicit PinnedBuf(size_t n, Workspace *w = nullptr);
    ~PinnedBuf();
    PinnedBuf(const PinnedBuf &) = delete;
    PinnedBuf &operator=(const PinnedBuf &) = delete;
    template <typename T>
    T *as() const { return static_cast<T *>(p); }
};

// Slots for a resident Lanczos basis, allocated in chunks of kBasisChunk
// vectors as a run needs them and reusable by the next run of the same call.
constexpr size_t kBasisChunk = 32;
struct BasisPool {
    Workspace *ws = nullptr;
    std::vector<std::unique_ptr<DevBuf>> chunks;
    size_t vb = 0;  // bytes per vector
    // the padding of the rows (bytes pad_off..pitch of each row, rows per vector):
    // zeroed when a chunk is allocated, since the kernels write only the row
    // elements and the fix-up of a flagged fused step reads whole padded rows
    size_t pitch = 0, pad_off = 0;
    int64_t rows = 0;
    size_t capacity() const { return chunks.size() * kBasisChunk; }
    void *slot(size_t j) const { return static_cast<char *>(chunks[j / kBasisChunk]->p) + (j % kBasisChunk) * vb; }
    // room for vector j within limit (bytes the pool may hold in total); false
    // when it cannot grow.  A chunk that the handle keeps is taken as it is; memory
    // from the device leaves 2 GiB of it free, kept buffers counting as free.
    bool reserve(size_t j, size_t limit, hipStream_t s);

  private:
    bool seen_free = false;
    size_t free_left = 0;
};

}  // namespace hub

struct hubbard {
    int sites = 0, n_up = 0, n_dn = 0;
    double t = 0, U = 0;
    std::vector<int32_t> edges;  // 2 per bond
    hub::SpinTable up, dn;
    int64_t dim = 0;
    hub::DeviceTables dev;
    std::vector<double> tcls;      // per-bond amplitudes: distinct values (empty: one amplitude t)
    std::vector<uint8_t> bond_cls; // class of each bond
    int device = 0;
    hipStream_t stream = nullptr;
    int precision = HUBBARD_FP64;
    uint64_t seed = 12043425ull;
    // device bytes a solve with psi may hold for its resident Lanczos basis
    size_t basis_limit = SIZE_MAX;
    // padded work rows for hubbard_apply on rows not on 128 bytes (two vectors
    // at the library's row stride, allocated on first use), and the event of
    // their last use, so that a call on another stream waits for it
    void *apply_work = nullptr;
    size_t apply_work_bytes = 0;
    hipEvent_t apply_ev = nullptr;
    hub::Workspace ws;
};

namespace hub {

// capi.cpp: the single-instance Lanczos driver (throws hub::Error)
void validate_opts(const hubbard_opts &o);
// two_vectors: the run holds no more than two work vectors (the server's
// footprint rule counts two)
int lanczos_impl(hubbard *h, const hubbard_opts &o, hubbard_result *res, bool two_vectors = false);

// builder.cpp
void build_spin_table(int sites, const std::vector<int32_t> &edges, int n, SpinTable &out);
uint64_t binomial(int n, int k);

// tridiag.cpp: symmetric tridiagonal T with diagonal d[0..m-1] and
// off-diagonal e[i] between rows i and i+1 (i < m-1).
// near, width: a guess that the value lies in (near - width, near] (width 0: none); the
// result does not depend on it.
double tridiag_lowest(const double *d, const double *e, int m, double near = 0.0, double width = 0.0);
void tridiag_lowest_vector(const double *d, const double *e, int m, double lam, double *y);
// c = exp(-i tau T) e_1 (real and imaginary parts, m each); e holds the m-1 off-diagonals
void tridiag_expm_e1(const double *d, const double *e, int m, double tau, double *c_re, double *c_im);

// kernels.hip: launchers (all asynchronous on `s`).
struct HvArgs {
    // per-bond amplitudes: the distinct values, indexed by the class bits of
    // up_rows / dn_cols entries (NULL: every hop has amplitude t)
    const double *tcls = nullptr;
    int ncls = 0;
    double amp4[4] = {0.0, 0.0, 0.0, 0.0};  // the classes, for the two-pass kernels (ncls <= kTwoPassClasses)
    int up_line_w = 32;  // slots per row of up_line: 32 (one 128-byte line) or 64 (two)
    int up_line_ipad = 0;  // internal slots padded with the zero row up to the group's largest count
    const uint32_t *states_up, *states_dn, *up_rows, *dn_cols;
    const uint16_t *nnz_up, *nnz_dn;
    const uint4 *dn_groups64, *dn_groups32;
    const uint8_t *dn_nq;
    int dn_ngroups;
    const uint4 *dn_groups16;  // null when rows exceed 32767 elements
    const uint8_t *dn_nq8;
    const uint4 *dn_pidx = nullptr;       // FP64 row pass: + hops, eight per group (null: not built)
    const uint2 *dn_nidx = nullptr;       // - hops, four per group
    const uint8_t *dn_pn = nullptr;       // group counts per 64 columns
    const uint4 *dn_cls = nullptr;        // two classes: groups by class (see DeviceTables)
    const uint8_t *dn_cls_n = nullptr;
    int dn_cls_g1 = 0, dn_cls_ng = 0;  // first slot of class 1, most groups of a class
    const uint32_t *up_cls_line = nullptr, *up_cls_cnt = nullptr;
    int dn_np = 0, dn_nn = 0;             // their largest values
    const uint32_t *up_blk;
    const uint16_t *up_nint, *up_next;
    const int32_t *up_bstart;
    int up_nblocks, up_max_block;
    const uint32_t *up_line, *up_cnt;  // null when a row has more than 64 hops
    int64_t dim_up, dim_dn;
    int32_t w_up, w_dn;
    double t, U;
    const uint32_t *up_tile = nullptr;  // one-launch H.v (null: not built)
    int up_tile_w = 0;
    const uint4 *dn_slots = nullptr;
    const double *dn_slot_amp = nullptr;
    const uint8_t *dn_slot_nq = nullptr;
    int dn_slot_groups = 0;
    double hops_up = 0.0, hops_dn = 0.0;  // mean hops of a row
    // a power of two near 1 / max(|t|, |U|) where those are very small or large (else
    // 1), and its inverse (see TileStep)
    double qscale = 1.0, qunscale = 1.0;
};

// Launch shape of the two-pass H.v for one element size (hv.hip).
struct HvPlan {
    int elem_bytes = 8;
    bool two_pass = false;  // false: rows too wide for LDS, one-pass kernel
    int64_t ld = 0;         // row stride of internal vectors (elements)
    int rows_rpb = 1, rows_threads = 64, rows_grid = 1;
    size_t rows_lds = 0;
    int slab_rw = 1, slab_grid = 8, nslab = 1;
    size_t slab_lds = 0;
    int blk_grid = 0, blk_nslab = 0, blk_threads = 1024;  // blocked slab pass (0: not available)
    size_t blk_lds = 0;
    int nparts = 1;         // largest number of partial sums any launch writes
};
enum HvMode { HV_STORE = 0, HV_LANCZOS = 1, HV_RESIDUAL = 2, HV_FUSED = 3, HV_FUSED_DEFL = 4 };
enum RedMode { RED_PLAIN = 0, RED_DOT = 1, RED_NORM = 2, RED_FUSED = 3, RED_START = 4, RED_FIX = 5 };
// Lower states a fused deflated step projects out (more take the unfused step).
constexpr int kFusedDefl = 2;
// Deflation data of HV_FUSED_DEFL: nd FP64 vectors in dense J order (vector l
// at psi + l * pdim) and their coefficients g (device, nd values).
struct HvDefl {
    const double *psi = nullptr;
    int nd = 0;
    int64_t pdim = 0;
    const double *g = nullptr;
};
// Fused Lanczos step: below this ratio b_{j+1}^2 / |q|^2 the expanded norm
// has lost too many digits and the step is finished by the explicit fix-up
// (device scalars S[kFixFlag], S[kFixScale]).
constexpr double kFixRatio = 1e-4;
constexpr int kFixFlag = 6, kFixScale = 7;

// HV_STORE:    y = H x
// HV_LANCZOS:  y = alpha H x + beta y (in place), alpha = coef[0], beta = coef[1];
//              partials[b] = block b's share of y.x
// HV_RESIDUAL: nothing stored; partials[b] = share of |Hx - alpha x|^2,
//              partials[nblocks + b] = share of x.Hx
// HV_FUSED:    (two-pass plans, padded rows) x <- x - c y is formed and written
//              back first, then y = alpha H x + beta y; coef = S (S[1] alpha,
//              S[2] beta, S[3] c); partials [3][n] = shares of y.x, y.y, x.x
// HV_FUSED_DEFL: as HV_FUSED with x <- x - c y - sum_l g_l psi_l (HvDefl,
//              nd <= kFusedDefl, line layout of the up-spin entries);
//              partials [3 + 2l][n] = shares of psi_l.y, [4 + 2l][n] of psi_l.x
template <typename T>
void launch_hv(const HvArgs &a, const T *x, T *y, int mode, double alpha, const double *coef, double *partials,
               int nblocks, hipStream_t s);
int hv_blocks(const HvArgs &a, int elem_bytes);

HvPlan make_hv_plan(const HvArgs &a, int elem_bytes);
// x, y (and scratch) are row-major dim_up x dim_dn with row strides ldx, ldy
// (lds_); scratch (the row-pass output) is used by HV_RESIDUAL only, where y
// is not written.  Partial sums: pl.nparts values (HV_RESIDUAL: twice that).
// Returns the number of partial sums written (HV_RESIDUAL: twice that many values).
// xpad, ypad: null, or dim_up x pl.ld work arrays.  When the rows of x or y do
// not start on 128 bytes, HV_STORE with both (HV_RESIDUAL with xpad) routes
// through them: the row pass writes its result to ypad (scratch) and a copy
// of x to xpad, and the up-spin pass runs on those and writes y.
// yout (fused modes, line layout): the result goes to yout (stride ldy) and y
// is only read (the beta and c terms).  pair > 0: the same step on a second
// vector pair at element offset pair from x, y and yout (the imaginary halves
// of complex vectors); the partial sums cover both pairs.
template <typename T>
int launch_hv2(const HvArgs &a, const HvPlan &pl, const T *x, int64_t ldx, T *y, int64_t ldy, T *scratch,
               int64_t lds_, int mode, double alpha, const double *coef, double *partials, hipStream_t s,
               T *xpad = nullptr, T *ypad = nullptr, const HvDefl *defl = nullptr, T *yout = nullptr,
               int64_t pair = 0);

// tile.hip: the one-launch H.v of small and medium sectors.  It reads the x rows
// of the up-spin hops from the Infinity Cache, so x has to fit there beside what
// else is live (192 MB of the 256).  Dense apply, two-pass / one launch in us:
// FP64 3x4 6u6d (853,776 states) 36.4 / 16.6, 14-site ring (11.8 M) 156 / 95,
// 4x4 8u4d (23.4 M) 390 / 342, 4x4 6u5d (35 M, 280 MB) 551 / 547, 4x4 6u6d (64 M)
// 1076 / 1224; FP32 14-site ring 96 / 60, 4x4 6u5d 326 / 273, 6u6d 598 / 625.
// Handles of more than four amplitude classes have no two-pass form and take it
// at any size where a row fits in LDS (a class per bond, apply, one-pass kernel /
// one launch in us: FP64 4x4 6u6d, 513 MB, 2530 / 1420, 4x4 8u8d, 1.3 GB, 7720 / 4180,
// 16-site ring 8u8d 4260 / 2420; FP32 2130 / 720, 6460 / 2310, 3740 / 1260).
constexpr int64_t kTileMaxBytes = (int64_t)192 << 20;
// Lanczos steps (vectors of one H.v, two launches a step against the fused
// two-pass step's five; us a step, fused / one-launch form): FP64 3x4 4u4d 30.3 /
// 17.4, 3x4 6u6d 48.4 / 29.1, 14-site ring 180 / 162, 4x4 5u5d (19 M, 153 MB) 415 /
// 384, 4x4 8u4d (187 MB) 429 / 503; FP32 14-site ring 114 / 98, 4x4 8u4d 264 / 242.
// More than four classes again at any size: FP64 4x4 6u6d 3040 / 1700, 8u8d 9080 /
// 5090, FP32 2410 / 1060 and 7210 / 3230; three vectors to the one-pass step's two.
constexpr int64_t kTileStepBytes = (int64_t)160 << 20;
// Sectors within those sizes whose steps (and products on rows on 128 bytes), or
// products on other rows (dense), the two-pass form is faster with.  What the
// one-launch form spends is the up-spin rows it reads again, the vector's bytes
// times its mean hops hu; what the two-pass form is good at depends on the rows and
// the precision.  Two-pass / one launch, us:
//   FP64, one amplitude, du >= dd: beyond 2,200 MB * hops steps lose (3x5 7u5d, 2,359:
//     279 / 308; 4x4 7u4d, 2,669: 391 / 432; with diagonals 7u4d, 5,337: 520 / 649),
//     below they gain (4x4 6u4d, 1,779: 292 / 280; 3x6 6u3d, 1,958: 296 / 239); dense
//     products lose beyond 5,000 (diagonals 7u4d 461 / 506, 6u4d, 3,558: 347 / 332).  With
//     du < dd they do not (diagonals 4u7d, 4,067: 615 / 577)
//   FP32, one amplitude, rows of 4,096 and more: steps beyond 1,400 (3x5 6u6d, 1,474: 240 /
//     258; 7u7d, 2,527: 390 / 456; 16-site ring 6u5d, 1,067: 281 / 250); with many
//     down-spin hops (hd >= 24: diagonals) du >= dd beyond 2,400 in both kinds (8u4d, 3,050:
//     326 / 377, dense 265 / 314; 6u4d, 1,779: 247 / 231)
//   FP32, two classes: steps beyond 2,300 (3x5 7u5d, 2,359: 341 / 372; 4x4 4u8d, 2,287: 585 /
//     512), dense products beyond 3,900; three and four classes: steps beyond 3,000
//   one row to a CU and few of them (11,000 <= dd <= 13,312, 256 < du < 1,024) with many
//     hops: 4x4 3u7d FP64, product on its rows 89 / 97; diagonals 3u7d 148 / 168; two
//     classes 3u8d FP32 150 / 173 a step (two classes FP64, 3u8d: 262 / 216)
struct SectorShape {
    int64_t du = 0, dd = 0;
    double hu = 0.0, hd = 0.0;  // mean hops of an up and a down row
    int ncls = 0;               // amplitude classes (0: one amplitude)
};
inline bool two_pass_better(const SectorShape &s, int elem_bytes, bool dense)
{
    if (s.ncls > kTwoPassClasses)
        return false;
    const bool fp32 = elem_bytes == 4, diag = s.hd >= 24.0;
    const double read = (double)s.du * (double)s.dd * elem_bytes / (1 << 20) * s.hu;
    if (s.du > 256 && s.du < 1024 && s.dd >= 11000 && s.dd <= 13312 && s.hu + s.hd >= 24.0 && (fp32 || s.ncls == 0))
        return diag || !dense;
    if (!fp32)
        return s.ncls == 0 && s.du >= s.dd && read > (dense ? 5000.0 : 2200.0);
    if (s.ncls > 2)
        return !dense && read > 3000.0;
    if (s.ncls == 2)
        return read > (dense ? 3900.0 : 2300.0);
    if (diag)
        return s.du >= s.dd && read > 2400.0;
    return !dense && s.dd >= 4096 && read > 1400.0;
}
// Sectors up to this size (and rows of at most 64 KB in FP64) take the
// one-launch form in every call and precision, but for those above; the server
// batches them.
constexpr int64_t kTileOnlyDim = 16000000;
static_assert(kTileOnlyDim * 8 <= kTileStepBytes && kTileOnlyDim * 8 <= kTileMaxBytes, "");
inline bool tile_only_sector(const SectorShape &s)
{
    if ((long double)s.du * (long double)s.dd > (long double)kTileOnlyDim || s.dd * 8 > 64 * 1024)
        return false;
    for (int es : {8, 4})
        for (bool dense : {false, true})
            if (two_pass_better(s, es, dense))
                return false;
    return true;
}
struct TilePlan {
    bool ok = false;
    int threads = 64, grid = 8, nseg = 1, span = 64;
    int defl = 0;  // lower vectors that a step's two launches project out at this row length
    size_t lds = 0;
};
// Lanczos step j (0-based) in two launches: the H.v (HV_LANCZOS) writes q = H x_j
// and partial sums of q.x_j; the update forms b_j = |x_j| from norm2, a_j from
// those sums, x_{j+1} = q / b_j - (a_j / b_j) x_j - (b_j / b_{j-1}) x_{j-1} in
// place of q, and the partial sums of its square (norm2_out).  With |x_j| = b_j the
// product q.x_j is of the order of b_j^2 |H|, three powers of the couplings where
// |x_j|^2 has two, so with extreme couplings the H.v sums qscale q.x_j (exact,
// |H| qscale near 1) and the update takes the factor out of a_j: the sums then fit
// a double wherever the norms do.  b[j] holds |x_j|;
// hist (may be mapped host memory): b_j at 2j, a_j at 2j + 1.  unit: x_0 is taken as a unit vector.  Where the
// H.v writes more than kTileDirectParts sums the caller reduces them to one first.
constexpr int kTileDirectParts = 4096;
constexpr int kTileDefl = 4;  // most lower vectors the two launches project out themselves
struct TileStep {
    const double *norm2 = nullptr;  // partial sums of |x_j|^2
    int n_norm2 = 0;
    double *norm2_out = nullptr;
    const double *part = nullptr;       // sums of q.x_j, then psi_l.q and psi_l.x_j in turn (n_part each)
    const double *part_prev = nullptr;  // those of step j - 1 (deflated steps)
    int n_part = 0;
    double qunscale = 1.0;  // as in HvArgs
    double *b = nullptr;
    double *hist = nullptr;
    int j = 0;
    int unit = 0;
};
TilePlan make_tile_plan(const HvArgs &a, int elem_bytes);
// HV_STORE: out = H x.  HV_LANCZOS: as above, with nd <= pl.defl dense lower
// vectors psi.  HV_RESIDUAL: partial sums of |Hx - shift x|^2, then of x.Hx.
// pl.grid sums of each (twice that with pair > 0: both halves of a complex
// vector at that element offset).
template <typename T>
void launch_hv_tile(const HvArgs &a, const TilePlan &pl, const T *x, int64_t ldx, T *out, int64_t ldy, int mode,
                    double shift, double *part, hipStream_t s, const double *psi = nullptr, int nd = 0,
                    int64_t pair = 0);
// vectors of halves * dim_up rows at stride ld (16-byte aligned, ld a multiple
// of four); xp is not read in step 0.  Returns the number of partial sums.
template <typename T>
int launch_tile_update(T *q, const T *x, const T *xp, int64_t dim_up, int64_t dim_dn, int64_t ld, int halves,
                       const TileStep &st, hipStream_t s, const double *psi = nullptr, int nd = 0);
// q <- q - sum_l (psi_l.q) psi_l and the partial sums of |q|^2; dots: nd * tile_defl_blocks values
template <typename T>
int launch_tile_project(T *q, const double *psi, int nd, int64_t dim_up, int64_t dim_dn, int64_t ld, double *dots,
                        double *norm2, hipStream_t s);
// b_j of the vector stored last (what 0), or a_j of an H.v no update follows (what 1)
void launch_tile_scalar(const TileStep &st, int what, hipStream_t s);
int tile_update_blocks(int64_t n, int elem_bytes);
int tile_defl_blocks(int64_t dim_up);

template <typename T>
void launch_axpy_norm(T *w, const T *v, const double *coef, int64_t n, double *partials, int nblocks, hipStream_t s);
// the fix-up of a flagged fused step (a no-op when S[kFixFlag] is clear)
template <typename T>
void launch_fused_fix(T *w, const T *v, const double *S, int64_t n, double *partials, int nblocks, hipStream_t s);
// the same for a fused deflated step: w <- w - S[3] v - sum_l S[8 + l] psi_l,
// rows at stride ld (returns the number of partial sums)
template <typename T>
int launch_fused_fix_defl(T *w, const T *v, const double *S, const double *psi, int nd, int64_t pdim, int64_t dim_up,
                          int64_t dim_dn, int64_t ld, double *partials, hipStream_t s);
void launch_start_raw(uint64_t seed, double *f, int64_t n, hipStream_t s);
void launch_start_norm2(const double *given, uint64_t seed, int64_t n, double *partials, int nblocks, hipStream_t s);
// out[r*ld + d] = (T)(c f[r*dim_dn + d]) and 0 in the row padding; zero (if
// not NULL) is cleared including its padding
template <typename T>
void launch_start_fill(const double *given, uint64_t seed, double c, T *out, T *zero, int64_t dim_up, int64_t dim_dn,
                       int64_t ld, hipStream_t s);
// psi[r*dim_dn + d] (+)= c * v[r*ld + d]
template <typename T>
void launch_psi_acc(double *psi, const T *v, double c, int64_t dim_up, int64_t dim_dn, int64_t ld, bool first,
                    hipStream_t s);
void launch_psi_stats(const double *psi, const double *given, uint64_t seed, int64_t n, double *partials, int nblocks,
                      hipStream_t s);
// psi[r*dim_dn + d] = sum_{j < m} c[j] * vecs[j][r*ld + d] (the resident Lanczos vectors)
template <typename T>
void launch_psi_combine(double *psi, const T *const *vecs, const double *c, int m, int64_t dim_up, int64_t dim_dn,
                        int64_t ld, hipStream_t s);
void launch_scale(double *v, double c, int64_t n, hipStream_t s);
void launch_reduce(const double *partials, int n, int stride, int count, double *out, hipStream_t s);
// observables.hip: unnormalised sums UU, DD, C (NS x NS each, NS = obs_ns_max)
// and the norm of psi^2 into out[3 * NS * NS + 1]; part holds
// obs_partial_count blocks of that size.  max_blocks bounds the accumulating
// workgroups (three on a CU fill its registers).
constexpr int kObsDefaultBlocks = 768;
int obs_ns_max(int sites);
int obs_partial_count(int ns, int64_t dim_up, int64_t dim_dn, int max_blocks = kObsDefaultBlocks);
void launch_observables(const double *psi, const uint32_t *states_up, const uint32_t *states_dn, int ns,
                        int64_t dim_up, int64_t dim_dn, double *part, double *out, int max_blocks, hipStream_t s);
// The allocation-free form: a static device array of kObsScratchBytes per
// device (its address taken once per device), and the largest workgroup count
// whose partial sums fit it.
constexpr size_t kObsScratchBytes = (size_t)16 << 20;
constexpr int kObsMaxDevices = 64;
double *obs_scratch(int device);
int obs_noalloc_blocks(int ns, int64_t dim_up, int64_t dim_dn);

// propagate.hip: the Krylov propagation step (see the file's header for the
// slot layout and the device scalars sc[4j..4j+3] = {s_j, 0, a_j, b_{j+1}})
enum PropMode { PROP_START = 0, PROP_DOT = 1, PROP_NORM = 2 };
int launch_prop_load(const double *re, const double *im, double *slot, int64_t npad, int64_t dim_up, int64_t dim_dn,
                     int64_t ld, double *partials, hipStream_t s);
int launch_prop_update(double *y, const double *w, const double *wp, const double *sc, int j, int64_t n,
                       double *partials, hipStream_t s);
int launch_prop_combine(double *basis, int nv, int64_t slot_stride, int64_t npad, const double *gam, double *re,
                        double *im, int64_t dim_up, int64_t dim_dn, int64_t ld, double *partials, hipStream_t s);
void launch_prop_reduce(const double *partials, int n, int mode, double *sc, int j, hipStream_t s);

// Most lower eigenvectors one deflated Lanczos run projects out.
constexpr int kMaxDeflate = 15;
// number of partial sums the two deflation kernels write per vector
int defl_blocks(int64_t dim_up);
template <typename T>
int launch_defl_dots(T *q, const T *v, const double *coef, const double *psi, int nd, int64_t dim, int64_t dim_up,
                     int64_t dim_dn, int64_t ld, double *partials, hipStream_t s);
template <typename T>
int launch_defl_update(T *q, const double *psi, const double *D, int nd, int64_t dim, int64_t dim_up, int64_t dim_dn,
                       int64_t ld, double *partials, hipStream_t s);
// nd: lower vectors of a fused deflated step (RED_FUSED)
void launch_reduce_step(const double *partials, int n, int mode, double *S, double *hist, int j, hipStream_t s,
                        int nd = 0);
void launch_init_scalars(double *S, hipStream_t s);
int stream_blocks(int64_t n);

}  // namespace hub
