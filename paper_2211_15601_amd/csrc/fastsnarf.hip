// C ABI of the Fast-SNARF articulation library (see include/fastsnarf.h): argument checks,
// context-owned device buffers and kernel launches.  gfx950 only.
#include "../../include/fastsnarf.h"
#include "../../include/fastsnarf_bench.h"
#include "fs_kernels.hpp"

#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

using namespace fs;

struct fs_ctx {
    fs_grid_desc desc;
    fs_params prm;
    hipStream_t stream;
    int device;
    GridP G;
    CorrP C;
    bool have_T;
    // device buffers owned by the context
    float *T;          // [P][V][12]
    float *Bdev;       // [P][nb][12] copy of the bone transforms of the last precompute
    float *Binv;       // [P][nb][12]
    uint8_t *Bok;      // [P][nb]
    float *GT;         // [P][V][12] gradient w.r.t. the transform grid (allocated on first fs_grad)
    // correspondence grid (voxel init)
    float *Y;          // [P][V][3]
    unsigned *bb_ord;  // [P][6][blocks of k_precompute]: per-block extents of the node images
    float *bbox;       // [P][6]
    int *head;         // [2][P*ncell] chunks of a correspondence cell, and the first of those that its table does not hold (k_corr_chunks)
    int2 *table;       // [P*ncell][CHUNKS] place and length of a cell's chunks
    int2 *link;        // [P][bricks][BRICK] next chunk and length, of those places where a chunk of a list starts
    float4 *sample;    // [P][bricks][BRICK] the nodes of a brick sorted by correspondence cell: {image[3], node index}
    int32_t *cand;     // [P][ncell][ck]
    uint8_t *ccnt;     // [P][ncell] number of candidates of a correspondence cell
    float4 *cinit;     // [P][ncell][ck][4] initial state of every candidate (k_corr_init)
    unsigned *cursor;  // work cursor of the solve kernel
    int *cells;        // [P*ncells] converged lanes per grid cell while a call counts them, zero between calls (behind the look-back words)
    int *gplace;       // [cell_words] where the cells' records begin in the list of a backward from arrays (place_cells)
    int *gplace_solve; // [cell_words] the same for the positions of the last fs_solve that gave them
    long long slots_N; // N of that fs_solve (0: none)
    int slots_K;
    bool slots_list;   // that solve drew its pairs from the candidate list: pairs without a candidate have no record
    int *gpos;         // [K*N] position of a lane inside its cell's list (grows on demand)
    float *grec;       // [K*N][8] cell-sorted {x*, lambda, cell} records (grows on demand)
    size_t gcap;       // lanes gpos / grec can hold
    float *gpart;      // [P][gb_blocks][nb*12] partial sums of dL/dB, one per block of k_grad_outputs
    int gb_blocks;
    float4 *srec;      // per-pair result records of the solve kernel (grows on demand)
    size_t srec_cap;   // float4 entries srec can hold
    u64 *look;         // look-back words of the kernels that scan in one pass, zero between kernels
    size_t look_words; // words look holds: enough for every call the context accepts
    size_t dd_look_at; // where those of k_dedupe_one begin
    bool look_dirty;   // a launch has failed: the words may have been used and not cleared
    int *dd_sums;      // [DD_TILES] tile sums of fs_dedupe (behind the cursor's words)
    uint8_t *vcnt;     // [N] candidates per point
    int *vgcell;       // [N] pose * ncell + correspondence cell of every point
    int2 *vlist;       // [K*N] pairs that have a candidate: {point, cell << 3 | k}
    size_t vcap, vgcell_cap;       // points vcnt / vlist, vgcell can hold
    int *vhist;        // [buckets][blocks] + 1: counts, then places, of the counting sort that orders the list by place
    size_t vhist_cap;
    int n_cus, occ_blocks_per_cu, occ_ws_blocks_per_cu, occ_vx_blocks_per_cu, chunk, refill_min, blocks_per_cu, point_major, lds_grid;
    bool lds_big;      // the grid is larger than 60 KiB and fits the LDS of a CU as one block of 12 waves
    int sort_list;     // order the list of (point, candidate) pairs by place (large voxel-mode batches)
    int xcd_ranges;    // with an ordered list: one range of it, and one cursor, per XCD
    int spin_limit;    // polls for room in the block's queue before the producer wave of a solve block gives up
    int pre_serial;    // number of the last fs_precompute (may_skip_corners)
    int *gave_up;      // pinned host word, mapped into the device: a wave that gave up sets it
    int *gave_up_dev;  // the device's address of it
    // optional timing of the Broyden kernel alone (events on the context's stream)
    bool timing;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> *timed;
    // caller pointers the runtime has already confirmed as memory of this device (direct-mapped by address)
    const void *ptr_seen[128];
    char err[256];
};

static __device__ __align__(256) int scratch[DD_TILES];     // see scratch_on_device()

namespace {

fs_status fail(fs_ctx *c, fs_status s, const char *fmt, ...)
{
    if (c) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(c->err, sizeof c->err, fmt, ap);
        va_end(ap);
    }
    return s;
}

// Null, alignment and "is memory of this context's device".  The last needs a lookup in the runtime (about a
// microsecond; a step makes some thirty such checks and a small step lasts 150 us), so a pointer that passed it
// once is remembered per context: a training or serving loop passes the same buffers again and again.  A
// remembered pointer whose memory the caller has freed since is the caller's error, as it would be one
// instruction after a fresh check.
bool device_ptr_ok(fs_ctx *c, const void *p, bool nullable)
{
    if (!p) return nullable;
    const uintptr_t u = reinterpret_cast<uintptr_t>(p);
    if ((u & 15u) != 0) return false;
    const size_t h = (size_t)((u >> 4) ^ (u >> 11) ^ (u >> 20)) & 127u;
    if (c->ptr_seen[h] == p) return true;
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (a.type != hipMemoryTypeDevice && a.type != hipMemoryTypeManaged) return false;
    if (a.device != c->device) return false;
    c->ptr_seen[h] = p;
    return true;
}

#define FS_CHECK_PTR(ctx, p, nullable)                                                            \
    do {                                                                                          \
        if (!device_ptr_ok((ctx), (p), (nullable)))                                               \
            return fail((ctx), FS_E_ARG, "%s: " #p " must be a 16-byte aligned device pointer%s", \
                        __func__, (nullable) ? " or NULL" : "");                                  \
    } while (0)

fs_status launch_status(fs_ctx *c, const char *what)
{
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) return FS_OK;
    c->look_dirty = true;        // the kernel that clears the look-back words may be the one that did not run
    return fail(c, FS_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

// A wave of the solve kernel that waited too long for its block's work queue has left early: the results
// of that call are incomplete.  Seen by the first call that comes after the kernel has run; the context
// stays in error from then on.
fs_status check_gave_up(fs_ctx *c, const char *what)
{
    if (c->gave_up && *static_cast<volatile int *>(c->gave_up))
        return fail(c, FS_E_DEVICE, "%s: an earlier fs_solve did not finish (a wave of its kernel gave up waiting for its block's work queue); create a new context", what);
    return FS_OK;
}

template <class Tp>
bool dev_alloc(Tp **p, size_t count)
{
    *p = nullptr;
    if (count == 0) return true;
    if (hipMalloc(reinterpret_cast<void **>(p), count * sizeof(Tp)) != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return false;
    }
    return true;
}

bool params_ok(const fs_params *p, char *why, size_t n)
{
    if (!(p->tol > 0.0f) || !(p->div_thresh > p->tol) || !std::isfinite(p->div_thresh)) {
        snprintf(why, n, "need 0 < tol < div_thresh < inf");
        return false;
    }
    if (p->max_iters < 0 || p->max_iters > 255) { snprintf(why, n, "max_iters must be in 0..255"); return false; }
    if (p->grad_mode != FS_GRAD_BROYDEN_J && p->grad_mode != FS_GRAD_EXACT_J) {
        snprintf(why, n, "bad grad_mode");
        return false;
    }
    return true;
}

int grid1d(long long n, int block) { return (int)((n + block - 1) / block); }

// The bricks of nodes that blocks of k_corr_chunks take: 2^lz nodes along z, 2^ly along y, the rest of BRICK along x; 8 x 8 x 16 nodes, longer along the others
// where an axis is shorter, so that bricks have room for at most four times the nodes of a large grid (P V < 2^31 / 12: places stay below 2^31).
struct Bricks {
    int lz, ly, nx, ny, nz;
    explicit Bricks(const GridP &G)
    {
        auto bits = [](int n) { int b = 0; while (b < 10 && 1 << b < n) ++b; return b; };
        lz = std::min(4, bits(G.nz));
        ly = std::min(3, bits(G.ny));
        const int lx = std::min(10 - lz - ly, bits(G.nx));
        ly = std::min(10 - lz - lx, std::max(ly, bits(G.ny)));
        lz = 10 - ly - lx;
        static_assert(BRICK == 1 << 10, "bits of a brick");
        nx = grid1d(G.nx, 1 << lx);
        ny = grid1d(G.ny, 1 << ly);
        nz = grid1d(G.nz, 1 << lz);
    }
    size_t count() const { return (size_t)nx * ny * nz; }
};

void free_all(fs_ctx *c)
{
    void *ptrs[] = {c->T, c->Bdev, c->Binv, c->Bok, c->GT, c->Y, c->bb_ord, c->bbox,
                    c->head, c->table, c->link, c->sample, c->cand, c->cursor, c->gplace, c->gplace_solve, c->gpos, c->grec, c->look, c->srec, c->gpart, c->vlist, c->cinit, c->vcnt, c->vgcell, c->vhist, c->ccnt};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
}

int scan_per_thread(int n) { return n <= (1 << 19) ? 4 : 16; }
int scan_blocks(int n) { return grid1d(n, 1024 * scan_per_thread(n)); }
// thousand points that a block of k_voxel_list takes
// (kernel us for 2 / 4 / 8 thousand: 0.3 M points 9 / 10 / 16, 1 M 17 / 13 / 16, 2 M 30 / 24 / 22, 4.2 M 76 / 65 / 62)
int list_per_thread(long long N) { return N <= (1 << 19) ? 2 : (N <= (1 << 21) ? 4 : 8); }
constexpr int DD_ONE_BLOCKS = 1024;                       // of k_dedupe_one at most
constexpr long long SORT_MAX_COUNTS = 1ll << 24;          // (buckets x blocks) of the sort that orders the list by place

// The look-back words are made and cleared with the context, for the largest call it accepts: 8 bytes per 8192 points of
// K * N < 2^31, 2 MiB at most.  The counts of converged lanes per cell, 4 bytes for every 48 of the transform grid, are behind them: they are zero
// between calls as well.  Growing them on demand, with a launch that clears them, breaks where the stream records a graph:
// the launch does not run, and calls before the graph's first replay find words of any value.
long long all_cells(const fs_ctx *c) { return (long long)c->G.P * (c->G.nx - 1) * (c->G.ny - 1) * (c->G.nz - 1); }
bool look_create(fs_ctx *c)
{
    long long blocks = 0;
    if (c->prm.init_mode == FS_INIT_VOXEL) {
        const long long N = ((1ll << 31) - 1) / c->C.ck;
        blocks = std::max({blocks, (long long)scan_blocks((int)SORT_MAX_COUNTS),
                           (long long)grid1d(N, 1024 * list_per_thread(N)), 1ll << 9});
    }
    c->look_words = (size_t)blocks + LOOK_HEAD;
    c->dd_look_at = c->look_words + LOOK_HEAD;                  // k_dedupe_one has words of its own behind them
    c->look_words = c->dd_look_at + LOOK_HEAD + DD_ONE_BLOCKS;
    c->look_words += c->look_words & 1;                         // the counts are read 16 bytes at a time
    const size_t cells_at = c->look_words;
    c->look_words += ((size_t)all_cells(c) + 1) / 2;
    c->look_dirty = false;
    if (!dev_alloc(&c->look, c->look_words)) return false;
    c->cells = reinterpret_cast<int *>(c->look + cells_at);
    return hipMemset(c->look, 0, c->look_words * sizeof(u64)) == hipSuccess;
}

// Before the first launch of a call that counts on words that are zero: clears them if a launch has failed since they were used.
fs_status look_ready(fs_ctx *c, const char *what)
{
    if (!c->look_dirty) return FS_OK;
    if (hipStreamSynchronize(c->stream) != hipSuccess || hipMemset(c->look, 0, c->look_words * sizeof(u64)) != hipSuccess ||
        hipStreamSynchronize(nullptr) != hipSuccess)
        return launch_status(c, what);
    k_fill_zero_i32<<<1, 64, 0, c->stream>>>(2, reinterpret_cast<int *>(c->cursor + CUR_ALL));        // CUR_LIST as well
    k_fill_zero_i32<<<1, 64, 0, c->stream>>>(N_XCD, reinterpret_cast<int *>(c->cursor + CUR_XCD));
    c->look_dirty = false;
    return launch_status(c, what);
}

// exclusive scan of a[0..n), n > 0, in place on the context's stream, a[n] = total; returns what
// the kernel after it has to clear of the look-back words
int scan_exclusive(fs_ctx *c, int n, int *a)
{
    const int m = scan_blocks(n);
    if (scan_per_thread(n) == 4) k_scan<4><<<m, 1024, 0, c->stream>>>(n, a, c->look);
    else k_scan<16><<<m, 1024, 0, c->stream>>>(n, a, c->look);
    return m;
}

// ---- scratch memory of fs_dedupe_noalloc: a file-scope device array instead of a context-owned allocation ----
// The sums of the at most DD_TILES tiles of points (whatever their number; the limit of points is the entry point's own, kept
// from when the array held a sum per fixed number of points); every GPU the library runs on holds its own 8 KiB copy of the array
// until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress: the device address is
// looked up once per device (with that device current) and kept in g_scratch_ptr.
constexpr long long FS_NOALLOC_MAX_N = 1ll << 24;
constexpr int FS_MAX_DEVICES = 64;
int *g_scratch_ptr[FS_MAX_DEVICES];       // device address of `scratch` on device i, nullptr until looked up
std::mutex g_scratch_mutex;

// address of `scratch` on the context's device (which must be the current one); nullptr on failure
int *scratch_on_device(fs_ctx *c)
{
    if (c->device < 0 || c->device >= FS_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[c->device]) {
        int cur = -1;
        if (hipGetDevice(&cur) != hipSuccess || cur != c->device) {
            (void)hipGetLastError();
            return nullptr;
        }
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[c->device] = static_cast<int *>(p);
    }
    return g_scratch_ptr[c->device];
}

// largest transform grid (all poses) kept in LDS by the solve: a block may ask for 64 KiB in all, and k_solve has 4 KiB of
// its own (the parked cell-position requests of its four waves)
constexpr size_t FS_LDS_GRID_MAX = 60 * 1024;
// ... by one block of 12 waves per CU: the CU's 160 KiB less the 12 KiB of parked requests of those waves
constexpr int FS_LDS_BIG_WAVES = 12;
constexpr size_t FS_LDS_GRID_MAX_BIG = 148 * 1024;
constexpr size_t L2_BYTES = 4u << 20;       // of an XCD

// where the places of the cells go
bool need_places(fs_ctx *c, int **p) { return *p || dev_alloc(p, (size_t)cell_words(all_cells(c))); }

// Kernels of the solve by the size of a batch (pairs = K * N; all three give the same bits).  What bounds a small batch is
// max_iters times the latency of a step, which is the shorter the more lanes share a pair (16 lanes 0.35 us, 4 0.5, one 1.0 to 1.2);
// what bounds a large one is instruction issue and the vector cache, where one lane per pair and refilled waves win.
// Measured, us, k_solve_quad / k_solve_once / k_solve_ws (k_solve where the grid is in LDS).  Solve and dedupe, 24 states per point, 64x64x16 nodes: 24 k pairs 35 / 42 / 46; 48 k 40 / 42 /
// 51; 72 k 48 / 49 / 59; 120 k 62 / 51 / 68; 156 k 72 / 61 / 75; 192 k 80 / 63 / 71; 228 k 89 / 83 / 75; 288 k 103 / 90 / 84; 128x128x32 nodes: 98 k 62 / 63 / 66; 192 k 94 / 86 / 77.  The lines
// are where the chip is full: three quad waves per SIMD; all pairs of k_solve_once resident at once (3 waves per SIMD of 64).
// With positions a wave takes several states of a point (pair_of), those of a point without a root all run to the last step, and
// k_solve_once keeps them in single lanes for longer; a step of training, 64x64x16: 48 k pairs 84 / 90 / 95, 98 k 102 / 104 / 109, 156 k 118 / 118 / 127,
// 192 k 128 / 124 / 124, 228 k 140 / 143 / 132.  On a grid in LDS a step in single lanes is shorter: 16x16x4, 48 k pairs 66 / 70 / 97, 98 k 87 / 76 / 108, 192 k 114 / 89 / 121, 228 k
// 128 / 120 / 128.
// With voxel-based candidates the share of pairs that have one is not known here (rays 1/7, scans 6/10), k_solve_ws needs
// its list of them first and most quads of a sparse batch end at once.  Solve and dedupe, 64x64x16: rays, 74 k pairs 27 / 32 / 41, 150 k 29 / 34 / 43, 285 k 36 / 38 / 53, 390 k 42 / 40 / 56, 600 k
// 54 / 48 / 61, 900 k 72 / 60 / 66; scans, 30 k 24 / 27 / 37, 74 k 31 / 27 / 42, 150 k 41 / 33 / 46, 285 k 56 / 47 / 50, 390 k 68 / 55 / 54, 600 k 92 / 75 / 59; 128x128x32: rays, 285 k 45 / 46 / 64, 600 k
// 61 / 63 / 75; scans, 150 k 48 / 46 / 54, 285 k 68 / 68 / 60.  Both lines are compromises between the two: the upper one, 4.5 waves per SIMD of which 3 are resident, where scans begin to
// lose more than rays gain.
enum { SOLVE_QUAD, SOLVE_ONCE, SOLVE_LARGE };
int solve_kind(const fs_ctx *c, long long pairs, bool candidates, bool positions, bool lds)
{
    const long long quad = (candidates ? 320 : (positions && !lds ? 512 : 192)) * (long long)c->n_cus, once = (candidates ? 1152 : 768) * (long long)c->n_cus;
    return pairs <= quad ? SOLVE_QUAD : (pairs <= once ? SOLVE_ONCE : SOLVE_LARGE);
}

// Do [a, a + na) and [b, b + nb) share a byte?  (nullptr: an array that is not there)
bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return a && b && x < y + nb && y < x + na;
}

// Should the kernels of small batches copy the grid (it fits the LDS) into every block's LDS?  A block of one wave moves
// 0.09 us per KiB before its first step, and a step from LDS is 0.1 to 0.2 us shorter than one through the caches, so a wave
// can afford to move some 60 KiB where most trajectories are long (one state per bone), 24 with candidates, which
// need few steps.  Measured, whole fs_solve in us, LDS / caches (50 steps, 24 states or 3 candidates per point):
//   states per bone:  48 KiB, 100 points 32 / 38, 500 36 / 38;  96 KiB, 37 points (a wave per block) 37 / 32, 800 (5) 40 / 42;
//                     146 KiB, 1 point 25 / 13, 100 (1) 44 / 35, 300 (2) 42 / 36, 800 (5) 39 / 39, 4096 (6) 46 / 52
//   candidates:       48 KiB, 37 points (1) 29 / 24, 4096 (3) 31 / 29;  96 KiB, 500 (1) 36 / 27, 8000 (6) 40 / 37;
//                     146 KiB, 1 point 21 / 6, 500 (1) 42 / 29, 4096 (3) 36 / 31, 28000 (6) 48 / 46
bool small_in_lds(const fs_ctx *c, size_t grid_bytes, int waves_per_block)
{
    const size_t per_wave = c->prm.init_mode == FS_INIT_VOXEL ? 24 * 1024 : 60 * 1024;
    return grid_bytes <= per_wave * waves_per_block;
}

int lanes_K(const fs_ctx *c) { return c->prm.init_mode == FS_INIT_BONE ? c->desc.n_bones : c->prm.corr_k; }

}  // namespace

extern "C" {

const char *fs_version(void) { return "fastsnarf-mi355x 0.1 (gfx950)"; }

const char *fs_last_error(const fs_ctx *ctx) { return ctx ? ctx->err : "null context"; }

fs_status fs_create(const fs_grid_desc *desc, const fs_params *params, void *hip_stream, fs_ctx **out)
{
    if (out) *out = nullptr;
    if (!desc || !params || !out) return FS_E_ARG;
    if (desc->nx < 2 || desc->ny < 2 || desc->nz < 2 || desc->n_bones < 1 || desc->n_bones > FS_MAX_BONES ||
        desc->n_poses < 1 || desc->n_poses > FS_MAX_POSES)
        return FS_E_SHAPE;
    const long long V = (long long)desc->nx * desc->ny * desc->nz;
    if ((long long)desc->n_poses * V * 12 >= (1ll << 31)) return FS_E_SHAPE;   /* grid offsets are 32-bit */
    if (desc->n_poses * desc->n_bones > 1024) return FS_E_UNSUPPORTED;   /* bone tables are staged in 48 KiB of LDS */
    for (int a = 0; a < 3; ++a)
        if (!(desc->hi[a] > desc->lo[a]) || !std::isfinite(desc->hi[a]) || !std::isfinite(desc->lo[a])) return FS_E_ARG;
    char why[128];
    if (!params_ok(params, why, sizeof why)) return FS_E_ARG;
    if (params->init_mode != FS_INIT_BONE && params->init_mode != FS_INIT_VOXEL) return FS_E_ARG;
    if (params->init_mode == FS_INIT_VOXEL) {
        if (params->corr_nx < 1 || params->corr_ny < 1 || params->corr_nz < 1 || params->corr_k < 1 ||
            params->corr_k > FS_MAX_CORR_K)
            return FS_E_SHAPE;
        if ((long long)params->corr_nx * params->corr_ny * params->corr_nz * desc->n_poses >= (1ll << 24)) return FS_E_SHAPE;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return FS_E_DEVICE;
    }
    fs_ctx *c = new (std::nothrow) fs_ctx;
    if (!c) return FS_E_ALLOC;
    std::memset(c, 0, sizeof *c);
    c->desc = *desc;
    c->prm = *params;
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->device = dev;
    GridP &G = c->G;
    G.nx = desc->nx; G.ny = desc->ny; G.nz = desc->nz; G.nb = desc->n_bones; G.P = desc->n_poses;
    G.sy = desc->nz * 12;
    G.sx = desc->ny * desc->nz * 12;
    G.V = V;
    G.mag_ny = div_magic((unsigned)desc->ny);
    G.mag_nz = div_magic((unsigned)desc->nz);
    G.mag_V = div_magic((unsigned)V);          // n_poses * V * 12 < 2^31
    const int n[3] = {desc->nx, desc->ny, desc->nz};
    for (int a = 0; a < 3; ++a) {
        G.lo[a] = desc->lo[a];
        G.hi[a] = desc->hi[a];
        G.inv_h[a] = (float)(n[a] - 1) / (desc->hi[a] - desc->lo[a]);
        G.h[a] = (desc->hi[a] - desc->lo[a]) / (float)(n[a] - 1);
        G.m[a] = (float)(n[a] - 1);
    }
    const size_t P = desc->n_poses, nb = desc->n_bones;
    bool ok = dev_alloc(&c->T, P * V * 12) && dev_alloc(&c->Bdev, P * nb * 12) && dev_alloc(&c->Binv, P * nb * 12) &&
              dev_alloc(&c->Bok, P * nb) && dev_alloc(&c->cursor, CUR_WORDS + DD_TILES);
    if (ok) c->dd_sums = reinterpret_cast<int *>(c->cursor + CUR_WORDS);
    if (ok) ok = hipMemset(c->cursor, 0, CUR_WORDS * sizeof(unsigned)) == hipSuccess;
    {
        int per_cu = 0, cus = 0;
        int per_cu_ws = 0;
        // resident blocks of the LDS-grid kernel with the LDS this context's grid needs (the grid's size never changes)
        const size_t gb = (size_t)desc->n_poses * V * 48;
        if (gb > FS_LDS_GRID_MAX && gb <= FS_LDS_GRID_MAX_BIG) {
            // the device must grant one block that much LDS; else the grid is read through the caches
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_solve<true, true, FS_LDS_BIG_WAVES>, 64 * FS_LDS_BIG_WAVES, gb) != hipSuccess) per_cu = 0;
            c->lds_big = per_cu >= 1;
            (void)hipGetLastError();
            if (c->lds_big) {       // more dynamic LDS than the default limit of a block: say so for every variant
                const void *fns[] = {(const void *)k_solve<true, true, FS_LDS_BIG_WAVES>, (const void *)k_solve<true, false, FS_LDS_BIG_WAVES>,
                                     (const void *)k_solve<false, true, FS_LDS_BIG_WAVES>, (const void *)k_solve<false, false, FS_LDS_BIG_WAVES>,
                                     (const void *)k_solve_quad<0, true>, (const void *)k_solve_quad<1, true>, (const void *)k_solve_quad<2, true>,
                                     (const void *)k_solve_once<0, true>, (const void *)k_solve_once<1, true>, (const void *)k_solve_once<2, true>};
                for (const void *f : fns)
                    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)gb) != hipSuccess) {
                        (void)hipGetLastError();
                        c->lds_big = false;
                    }
            }
            per_cu = 1;
        } else if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_solve<true, true>, 256, gb <= FS_LDS_GRID_MAX ? gb : 0) != hipSuccess || per_cu < 1) per_cu = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_ws, k_solve_ws<true, true, FS_WS_CONSUMERS, true>, 64 * (FS_WS_CONSUMERS + 1), 0) != hipSuccess || per_cu_ws < 1) per_cu_ws = 2;
        c->occ_ws_blocks_per_cu = per_cu_ws;
        int per_cu_vx = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_vx, k_solve_ws<true, true, FS_VX_CONSUMERS, false>, 64 * (FS_VX_CONSUMERS + 1), 0) != hipSuccess || per_cu_vx < 1) per_cu_vx = 2;
        c->occ_vx_blocks_per_cu = per_cu_vx;
        c->spin_limit = 1 << 22;   /* x about 0.2 us per poll */
        c->blocks_per_cu = 0;      /* 0: chosen per call */
        c->point_major = -1;       /* -1: chosen per call */
        c->lds_grid = 1;
        c->sort_list = 0;
        c->xcd_ranges = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
        (void)hipGetLastError();
        c->n_cus = cus;
        c->occ_blocks_per_cu = per_cu;
        c->chunk = 128;
        c->refill_min = 0;         /* 0: chosen per call */
    }
    if (ok && params->init_mode == FS_INIT_VOXEL) {
        CorrP &C = c->C;
        C.cx = params->corr_nx; C.cy = params->corr_ny; C.cz = params->corr_nz; C.ck = params->corr_k;
        C.ncell = C.cx * C.cy * C.cz;
        ok = dev_alloc(&c->Y, P * V * 3) && dev_alloc(&c->bb_ord, P * 6 * (size_t)grid1d(V, 256)) && dev_alloc(&c->bbox, P * 6) &&
             dev_alloc(&c->head, 2 * P * C.ncell) && dev_alloc(&c->table, P * C.ncell * CHUNKS) && dev_alloc(&c->link, P * Bricks(G).count() * BRICK) && dev_alloc(&c->sample, P * Bricks(G).count() * BRICK) &&
             dev_alloc(&c->cand, P * (size_t)C.ncell * C.ck) && dev_alloc(&c->ccnt, P * (size_t)C.ncell) &&
             dev_alloc(&c->cinit, P * (size_t)C.ncell * C.ck * 4);
    }
    if (ok) ok = look_create(c) && hipStreamSynchronize(nullptr) == hipSuccess;      // cleared before the first call, whichever stream that is on
    if (ok) {
        ok = hipHostMalloc(reinterpret_cast<void **>(&c->gave_up), sizeof(int), hipHostMallocMapped) == hipSuccess;
        if (ok) {
            *c->gave_up = 0;
            ok = hipHostGetDevicePointer(reinterpret_cast<void **>(&c->gave_up_dev), c->gave_up, 0) == hipSuccess;
        }
        if (!ok) (void)hipGetLastError();
    }
    if (!ok) {
        free_all(c);
        if (c->gave_up) (void)hipHostFree(c->gave_up);
        delete c;
        return FS_E_ALLOC;
    }
    *out = c;
    return FS_OK;
}

fs_status fs_destroy(fs_ctx *ctx)
{
    if (!ctx) return FS_OK;
    (void)hipStreamSynchronize(ctx->stream);
    if (ctx->timed) {
        for (auto &e : *ctx->timed) {
            (void)hipEventDestroy(e.first);
            (void)hipEventDestroy(e.second);
        }
        delete ctx->timed;
    }
    free_all(ctx);
    if (ctx->gave_up) (void)hipHostFree(ctx->gave_up);
    delete ctx;
    return FS_OK;
}

fs_status fs_set_params(fs_ctx *ctx, const fs_params *params)
{
    if (!ctx) return FS_E_ARG;
    if (!params) return fail(ctx, FS_E_ARG, "fs_set_params: params is NULL");
    char why[128];
    if (!params_ok(params, why, sizeof why)) return fail(ctx, FS_E_ARG, "fs_set_params: %s", why);
    ctx->prm.tol = params->tol;
    ctx->prm.div_thresh = params->div_thresh;
    ctx->prm.max_iters = params->max_iters;
    ctx->prm.grad_mode = params->grad_mode;
    return FS_OK;
}

fs_status fs_set_tuning(fs_ctx *ctx, int32_t chunk, int32_t refill_min, int32_t blocks_per_cu, int32_t point_major, int32_t lds_grid)
{
    if (!ctx) return FS_E_ARG;
    if ((chunk != 0 && (chunk < 8 || chunk > 4096)) || (refill_min != 0 && (refill_min < 1 || refill_min > 64)) ||
        blocks_per_cu < 0 || blocks_per_cu > 32 || point_major < -1 || point_major > 1 || lds_grid < -1 || lds_grid > 1)
        return fail(ctx, FS_E_ARG, "fs_set_tuning: value out of range");
    if (chunk) ctx->chunk = chunk;
    if (refill_min) ctx->refill_min = refill_min;
    if (blocks_per_cu) ctx->blocks_per_cu = blocks_per_cu;
    if (point_major >= 0) ctx->point_major = point_major;
    if (lds_grid >= 0) ctx->lds_grid = lds_grid;
    return FS_OK;
}

fs_status fs_set_list_order(fs_ctx *ctx, int32_t by_place)
{
    if (!ctx) return FS_E_ARG;
    if (by_place < 0 || by_place > 2) return fail(ctx, FS_E_ARG, "fs_set_list_order: by_place must be 0, 1 or 2");
    ctx->sort_list = by_place != 0;
    ctx->xcd_ranges = by_place == 2;
    return FS_OK;
}

fs_status fs_set_spin_limit(fs_ctx *ctx, int32_t polls)
{
    if (!ctx) return FS_E_ARG;
    if (polls < 0) return fail(ctx, FS_E_ARG, "fs_set_spin_limit: polls must be >= 0");
    ctx->spin_limit = polls;
    return FS_OK;
}

fs_status fs_precompute(fs_ctx *ctx, const float *d_W, const float *d_B)
{
    if (!ctx) return FS_E_ARG;
    { fs_status gs = check_gave_up(ctx, "fs_precompute"); if (gs != FS_OK) return gs; }
    FS_CHECK_PTR(ctx, d_W, false);
    FS_CHECK_PTR(ctx, d_B, false);
    const GridP &G = ctx->G;
    hipStream_t st = ctx->stream;
    const bool voxel = ctx->prm.init_mode == FS_INIT_VOXEL;
    const int ncp = voxel ? G.P * ctx->C.ncell : 0, vblocks = grid1d(G.V, 256);
    { fs_status ls = look_ready(ctx, "fs_precompute"); if (ls != FS_OK) return ls; }
    ++ctx->pre_serial;
    // poses per pass over the weights: see k_precompute
    const bool wide = (long long)vblocks * ((G.P + 3) / 4) >= 4ll * ctx->n_cus;
#define FS_LAUNCH_PRE(NP, FEW)                                                                                         \
    k_precompute<NP, FEW><<<(vblocks + (FEW) + N_XCD - 1) / N_XCD * N_XCD * ((G.P + (NP) - 1) / (NP)), 256, 0, st>>>(       \
        G, d_W, d_B, ctx->T, ctx->Bdev, ctx->Binv, ctx->Bok, reinterpret_cast<int *>(ctx->cursor + CUR_GRID),          \
        ctx->pre_serial, voxel ? ctx->Y : nullptr, ctx->bb_ord, ctx->head, 2 * ncp, vblocks, (G.P + (NP) - 1) / (NP))
    if (wide) FS_LAUNCH_PRE(4, false);
    else if ((long long)vblocks * G.P <= 2ll * ctx->n_cus) FS_LAUNCH_PRE(1, true);
    else FS_LAUNCH_PRE(1, false);
#undef FS_LAUNCH_PRE
    if (voxel) {
        const CorrP &C = ctx->C;
        const bool own_box = vblocks <= EXTENT_OWN;
        if (!own_box) k_corr_bbox<<<G.P * 6, 1024, 0, st>>>(vblocks, ctx->bb_ord, ctx->bbox);
        const Bricks b(G);
        k_corr_chunks<<<dim3((unsigned)b.count(), G.P), BRICK, 0, st>>>(G, C, ctx->Y, ctx->bb_ord, vblocks, own_box, ctx->bbox, b.lz, b.ly, b.ny, b.nz,
                                                                        ctx->head, ctx->table, ctx->link, ctx->sample);
        k_corr_select<<<dim3(grid1d(C.ncell, 4), G.P), 256, 0, st>>>(G, C, ctx->bbox, ctx->head, ctx->table, ctx->link, ctx->sample, ctx->cand, ctx->ccnt);
        k_corr_init<<<grid1d((long long)ncp * C.ck, 256), 256, 0, st>>>(G, C, ctx->T, ctx->cand, ctx->cinit);
    }
    fs_status s = launch_status(ctx, "fs_precompute");
    ctx->have_T = s == FS_OK;
    return s;
}

fs_status fs_init(fs_ctx *ctx, const float *d_xq, const int32_t *d_pose, int64_t N, float *d_x0, float *d_Jinv0,
                  uint8_t *d_valid0)
{
    if (!ctx) return FS_E_ARG;
    { fs_status gs = check_gave_up(ctx, "fs_init"); if (gs != FS_OK) return gs; }
    if (!ctx->have_T) return fail(ctx, FS_E_STATE, "fs_init: call fs_precompute first");
    const int K = lanes_K(ctx);
    if (N < 0 || (long long)N * K >= (1ll << 31)) return fail(ctx, FS_E_SHAPE, "fs_init: need 0 <= N and K*N < 2^31");
    if (N == 0) return FS_OK;
    if (ctx->desc.n_poses > 1 && !d_pose) return fail(ctx, FS_E_ARG, "fs_init: d_pose is required when n_poses > 1");
    FS_CHECK_PTR(ctx, d_xq, false);
    FS_CHECK_PTR(ctx, d_pose, true);
    FS_CHECK_PTR(ctx, d_x0, false);
    FS_CHECK_PTR(ctx, d_Jinv0, false);
    FS_CHECK_PTR(ctx, d_valid0, false);
    const long long total = (long long)N * K;
    if (ctx->prm.init_mode == FS_INIT_BONE)
        k_init_bone<<<grid1d(total, 256), 256, 0, ctx->stream>>>(ctx->G, ctx->T, ctx->Binv, ctx->Bok, d_xq, d_pose, N,
                                                                 d_x0, d_Jinv0, d_valid0, reinterpret_cast<const int *>(ctx->cursor + CUR_GRID));
    else
        k_init_voxel<<<grid1d(total, 256), 256, 0, ctx->stream>>>(ctx->G, ctx->C, ctx->bbox, ctx->cinit, d_xq, d_pose, N,
                                                                  d_x0, d_Jinv0, d_valid0);
    return launch_status(ctx, "fs_init");
}

fs_status fs_solve(fs_ctx *ctx, const float *d_xq, const int32_t *d_pose, int64_t N, int32_t K, const float *d_x0,
                   const float *d_Jinv0, const uint8_t *d_valid0, float *d_xc, uint8_t *d_conv, float *d_Jinv,
                   uint8_t *d_iters, int32_t *d_slot)
{
    if (!ctx) return FS_E_ARG;
    { fs_status gs = check_gave_up(ctx, "fs_solve"); if (gs != FS_OK) return gs; }
    if (!ctx->have_T) return fail(ctx, FS_E_STATE, "fs_solve: call fs_precompute first");
    if (K != lanes_K(ctx)) return fail(ctx, FS_E_SHAPE, "fs_solve: K = %d but the init mode produces %d lanes per point", K, lanes_K(ctx));
    if (N < 0 || (long long)N * K >= (1ll << 31)) return fail(ctx, FS_E_SHAPE, "fs_solve: need 0 <= N and K*N < 2^31");
    if (N == 0) return FS_OK;
    if (ctx->desc.n_poses > 1 && !d_pose) return fail(ctx, FS_E_ARG, "fs_solve: d_pose is required when n_poses > 1");
    FS_CHECK_PTR(ctx, d_xq, false);
    FS_CHECK_PTR(ctx, d_pose, true);
    const bool fused = d_x0 == nullptr;
    if (fused && (d_Jinv0 || d_valid0))
        return fail(ctx, FS_E_ARG, "fs_solve: d_x0, d_Jinv0 and d_valid0 must be all NULL (fused initial states) or all set");
    if (!fused) {
        FS_CHECK_PTR(ctx, d_x0, false);
        FS_CHECK_PTR(ctx, d_Jinv0, false);
        FS_CHECK_PTR(ctx, d_valid0, false);
    }
    FS_CHECK_PTR(ctx, d_xc, false);
    FS_CHECK_PTR(ctx, d_conv, false);
    FS_CHECK_PTR(ctx, d_Jinv, true);
    FS_CHECK_PTR(ctx, d_iters, true);
    FS_CHECK_PTR(ctx, d_slot, true);
    SolveP S;
    S.N = N;
    S.total = (long long)N * K;
    S.max_iters = ctx->prm.max_iters;
    S.tol2 = ctx->prm.tol * ctx->prm.tol;
    S.div2 = ctx->prm.div_thresh * ctx->prm.div_thresh;
    S.K = K;
    S.mag_N = div_magic((unsigned)N);
    S.mag_K = div_magic((unsigned)K);
    S.chunk = ctx->chunk;
    S.spin_limit = ctx->spin_limit;
    const long long chunks = (S.total + S.chunk - 1) / S.chunk;
    const size_t grid_bytes = (size_t)ctx->G.P * ctx->G.V * 48;
    const bool lds_big = ctx->lds_grid && ctx->lds_big && grid_bytes > FS_LDS_GRID_MAX && grid_bytes <= FS_LDS_GRID_MAX_BIG;
    const bool lds = (ctx->lds_grid && grid_bytes <= FS_LDS_GRID_MAX) || lds_big;
    // Launch shape.  Grid in LDS (k_solve): latency / ALU bound, every wave the registers allow, refill at 32 idle
    // lanes.  Grid read through the caches (k_solve_ws, bound by the vector-memory path): blocks of one producer and
    // several consumers, two or three per CU.
    const bool voxel_list = fused && ctx->prm.init_mode == FS_INIT_VOXEL;     // the solve draws from the list of pairs that have a candidate
    // fused voxel-based candidates: the producer only looks initial states up (k_corr_init computed them once per pose)
    const bool vx = !lds && voxel_list;
    const int wpb = lds_big ? FS_LDS_BIG_WAVES : (lds ? 4 : 1);       // waves of a block that draw chunks from the cursor
    const bool bone = ctx->prm.init_mode == FS_INIT_BONE;
    // A third block per CU hides latency, and misses the L2 more often.  fs_solve, us, two / three blocks:
    //   states per bone, 24, 12 k / 40 k / 200 k points: 3 MB grid, 200 k 634 / 580, with positions 838 / 713;  4.5 MB 76 / 75, 165 / 160, 673 / 616, with positions 97 / 97, 199 / 181, 814 / 706;  10.6 MB 81 / 81, 175 / 174,
    //   707 / 672, with positions 102 / 102, 206 / 191, 845 / 752;  13.5 MB 82 / 84, 182 / 183, 725 / 704;  21 MB 87 / 86, 192 / 197, 766 / 785;  24 MB 200 k 785 / 821;  7 MB in 4
    //   poses 88 / 88, 190 / 191, 773 / 712;  25 MB in 8 97 / 100, 214 / 218, 835 / 797
    //   candidates, 1 M points, roots only: 3 MB rays 87 / 90, scans 124 / 130;  7 MB 104 / 114, 173 / 181;  25 MB 132 / 137, 228 / 239;  with positions 3 MB 99 / 99, 166 / 156;  7 MB 117 / 125,
    //   220 / 209;  25 MB 149 / 149, 284 / 282;  25 MB in 8 poses, 4.2 M points 1378 / 1427;  0.1 M of scans, 3 MB, 44 / 48, with positions 53 / 56
    // Two is what fs_set_tuning promises for candidates, which gain in one form and lose in the others, and beyond 4 MiB, where three lost before the waves of a block shared one
    // queue; with this kernel large batches lose from some 16 MB on only.
    const int auto_blocks = lds || (bone && grid_bytes <= L2_BYTES) ? 3 : 2;
    const int want_blocks = ctx->blocks_per_cu ? (lds ? std::max(ctx->blocks_per_cu, 3) : ctx->blocks_per_cu) : auto_blocks;
    const int occ = lds ? ctx->occ_blocks_per_cu : (vx ? ctx->occ_vx_blocks_per_cu : ctx->occ_ws_blocks_per_cu);
    const int per_cu = lds_big ? 1 : std::max(1, std::min(want_blocks, occ));
    // consumers of k_solve_ws refill from their queue at 8 idle lanes (8 ... 24: within 1 % on grids the L2 holds; 32 and
    // more lose 3 ... 40 %); with candidates on grids beyond it at 24 (1.34 instead of 1.37 ms on the 8-pose batch; 48: 1.38)
    S.refill_min = ctx->refill_min ? ctx->refill_min : (lds ? 32 : (grid_bytes > (32u << 20) && !bone ? 24 : 8));
    S.prefetch = grid_bytes > (32u << 20);
    // Order of the pairs: tiles of points (tile_pair) or all states of a point side by side.  On a grid beyond the L2 neighbouring lanes should read
    // one point's surroundings: in tiles the lines fetched for a point are gone when its next states come.  That counts once many pairs meet
    // a large grid; small batches gain more from the tiles' outputs, given states are read whole lines at a time in tiles, and with positions
    // lanes share an atomic only with the same point's.  Whole calls, us, tiles / side by side, 24 states per point but where stated:
    //   roots only  9.3 MB grid, 20 k points 153 / 159, 60 k 308 / 304, 200 k 838 / 803;  24 MB 20 k 183 / 187, 60 k 374 / 359, 200 k 1050 / 945, 60 k of 64
    //               states 1122 / 900;  4.5 MB 60 k 284 / 290, 200 k 762 / 756;  25 MB in 8 poses, points in any order, 14 k 128 / 149, 200 k 1220 / 1088
    //   positions   120 k points in two poses of 24 MB 1072 / 996;  24 MB 20 k 287 / 288, 60 k 563 / 542, 200 k 1490 / 1370
    //   given       24 MB 20 k 353 / 376, 200 k 2049 / 2174
    // The line of the first is pairs times bytes of the grid = 1.5e13 (60 k points of 24 states: 10 MB).
    const bool beyond = grid_bytes > L2_BYTES;
    S.point_major = ctx->point_major >= 0 ? 2 * ctx->point_major : (beyond && (d_slot || (fused && (double)S.total * (double)grid_bytes > 1.5e13)) ? 2 : 1);
    // Eighths of the chunks dealt out without asking the cursor.  Whole calls, us, with 0 / 4 / 6 / 7:
    //   one state per bone, read through the caches: 64x64x16 nodes, 200 k points 732 / 709 / 723 / 739, 65 k 411 / 397 / 399 / 406, 20 k on 45x39x11 209 / 203 /
    //   201 / 201;  24 MB, 0 and 4 alone, 200 k 942 / 945, 60 k 358 / 356
    //   grid in LDS, 0 / 4 / 6: 34 KiB, 20 k 119 / 119 / 119, 60 k 221 / 221 / 203, 200 k 543 / 478 / 448;  135 KiB, 60 k 219 / 220 / 204
    //   candidates: 64x64x16 nodes, 2 M ray samples 303 / 292 / 286 / 286;  0 / 4 / 6: 11 MB, 2 M ray samples 296 / 281 / 275, 1 M of scans 323 / 297 / 289, 25 MB in
    //   8 poses 339 / 333 / 335;  given states, 0.3 M ray samples 248 / 233 / 224
    // On grids beyond 32 MiB all blocks should read the same stretch of the points: 8 poses of 128x128x32 nodes 2438 / 2447 / 2460 / 2488.
    S.dealt = S.prefetch ? 0 : (bone && !lds ? 4 : 6);
    const int blocks = (int)std::min<long long>(grid1d(chunks, wpb), (long long)per_cu * ctx->n_cus);
    InitP I;
    I.mode = ctx->prm.init_mode;
    I.Binv = ctx->Binv;
    I.Bok = ctx->Bok;
    I.C = ctx->C;
    I.bbox = ctx->bbox;
    I.cand = ctx->cand;
    I.ccnt = ctx->ccnt;
    I.cinit = ctx->cinit;
    const bool with_J = d_Jinv != nullptr || d_slot != nullptr;     // with d_slot alone J~ stays in the result records
    // On request (fs_set_list_order) batches of at least four tiles of the counting sort are ordered by place (pose, then
    // column of correspondence cells), whatever kernel their size would take otherwise: only k_solve and k_solve_ws draw
    // from a list.  Smaller ones, or correspondence grids with more columns than the sort's LDS counters hold, keep the order
    // of the points.
    const int nb = ctx->G.P * ctx->C.cx * ctx->C.cy;
    const long long sblk = (N + SORT_TILE - 1) / SORT_TILE;
    const bool sorted = voxel_list && ctx->sort_list && N >= 4 * SORT_TILE && nb <= SORT_MAX_BUCKETS && (long long)nb * sblk < SORT_MAX_COUNTS;
    // The kernels of small batches write the caller's outputs while other waves still read the inputs; the others leave
    // records, which are unpacked when the solve has ended: a solve in place (roots over the query points) takes those.
    bool in_place = false;
    {
        const size_t n = (size_t)N, kn = (size_t)S.total;
        const std::pair<const void *, size_t> in[] = {{d_xq, 12 * n}, {d_pose, 4 * n}, {d_x0, 12 * kn}, {d_Jinv0, 36 * kn}, {d_valid0, kn}};
        const std::pair<const void *, size_t> out[] = {{d_xc, 12 * kn}, {d_conv, kn}, {d_Jinv, 36 * kn}, {d_iters, kn}, {d_slot, 4 * kn}};
        for (const auto &i : in)
            for (const auto &o : out) in_place = in_place || overlap(i.first, i.second, o.first, o.second);
    }
    const int kind = sorted || in_place ? SOLVE_LARGE : solve_kind(ctx, S.total, voxel_list, d_slot != nullptr, lds);
    const bool quad = kind == SOLVE_QUAD;
    const size_t need = kind != SOLVE_LARGE ? (d_slot ? (size_t)S.total * 4 : 0) : (size_t)S.total * (with_J ? 4 : 1);
    ctx->slots_N = 0;            // from here on the records of the solve before are lost, also when this call fails
    if (need > ctx->srec_cap) {
        (void)hipStreamSynchronize(ctx->stream);
        if (ctx->srec) (void)hipFree(ctx->srec);
        ctx->srec = nullptr;
        ctx->srec_cap = 0;
        if (!dev_alloc(&ctx->srec, need)) return fail(ctx, FS_E_ALLOC, "fs_solve: out of device memory for %zu result records", (size_t)S.total);
        ctx->srec_cap = need;
    }
    hipStream_t st = ctx->stream;
    const int ncell = (ctx->G.nx - 1) * (ctx->G.ny - 1) * (ctx->G.nz - 1);
    const long long ncp = all_cells(ctx);              // P * V * 12 < 2^31
    if (d_slot && !need_places(ctx, &ctx->gplace_solve)) return fail(ctx, FS_E_ALLOC, "fs_solve: out of device memory");
    { fs_status ls = look_ready(ctx, "fs_solve"); if (ls != FS_OK) return ls; }
    if (kind != SOLVE_LARGE) {
        int *counts = d_slot ? ctx->cells : nullptr;
        hipEvent_t ev0 = nullptr, ev1 = nullptr;
        if (ctx->timing && hipEventCreate(&ev0) == hipSuccess && hipEventCreate(&ev1) == hipSuccess) (void)hipEventRecord(ev0, st);
        // grid in LDS: about one block per CU, as many waves in it as the batch gives it; else blocks of four waves
        long long waves = 0;
        int per_block = 0;
        auto split = [&](int per) {            // into waves of `per` pairs
            S.per = per;
            S.ki = d_slot && K >= 8 ? std::min(8, per) : 1;
            const int pts = per / S.ki;        // points per wave
            waves = ((N + pts - 1) / pts) * ((K + S.ki - 1) / S.ki);
            per_block = (int)std::min<long long>(quad ? 16 : FS_LDS_BIG_WAVES, std::max<long long>(1, (waves + ctx->n_cus - 1) / ctx->n_cus));
        };
        split(quad ? QUADS : WAVE);
        const bool staged = lds && small_in_lds(ctx, grid_bytes, per_block);
        // Waves of four pairs, which take rows of 16 lanes at once: while there is one of them per SIMD, three where pairs wait for each other otherwise
        // (candidates: most have none; positions: states of one point).  Whole calls, us, 16 pairs / 4: 24 states, roots only, 0.9 k pairs
        // 30 / 29, 4.8 k 32 / 33, 12 k 32 / 35;  a step 2.4 k 79 / 71, 8 k 83 / 78, 12 k 66 / 62, 19 k 65 / 71;  ray samples 4.5 k 23 / 21, 13 k 22.7 / 20.6, 27 k 23.3 / 23.1,
        // scans 9 k 29.7 / 30.4, 18 k 30 / 33.
        // (Where the copy of the grid is dear, blocks keep the number of waves that small_in_lds was asked about.)
        const bool many = voxel_list ? !staged : (d_slot && !(staged && lds_big));
        if (quad && S.total <= (many ? 48ll : 16ll) * ctx->n_cus) split(HEXES);
        const int threads = staged ? WAVE * per_block : 256;
        const dim3 qg(grid1d(waves * 64, threads));
        const int *state = reinterpret_cast<const int *>(ctx->cursor + CUR_GRID);
#define FS_LAUNCH_QUAD(IM, L)                                                                                          \
    do {                                                                                                               \
        if (quad)                                                                                                      \
            k_solve_quad<IM, L><<<qg, threads, (L) ? grid_bytes : 0, st>>>(                                            \
                ctx->G, S, I, ctx->T, d_xq, d_pose, d_x0, d_Jinv0, d_valid0, d_xc, d_conv, d_Jinv, d_iters, d_slot,    \
                d_slot ? ctx->srec : nullptr, counts, ncell, ctx->cursor + CUR_TOTAL);                                 \
        else                                                                                                           \
            k_solve_once<IM, L><<<qg, threads, (L) ? grid_bytes : 0, st>>>(                                            \
                ctx->G, S, I, ctx->T, d_xq, d_pose, d_x0, d_Jinv0, d_valid0, d_xc, d_conv, d_Jinv, d_iters, d_slot,    \
                d_slot ? ctx->srec : nullptr, counts, ncell, state, ctx->cursor + CUR_TOTAL);                          \
    } while (0)
        const int im = !fused ? 2 : (voxel_list ? 1 : 0);
        if (staged) {
            if (im == 0) FS_LAUNCH_QUAD(0, true);
            else if (im == 1) FS_LAUNCH_QUAD(1, true);
            else FS_LAUNCH_QUAD(2, true);
        } else {
            if (im == 0) FS_LAUNCH_QUAD(0, false);
            else if (im == 1) FS_LAUNCH_QUAD(1, false);
            else FS_LAUNCH_QUAD(2, false);
        }
#undef FS_LAUNCH_QUAD
        if (ev0 && ev1) {
            (void)hipEventRecord(ev1, st);
            ctx->timed->emplace_back(ev0, ev1);
        }
        if (d_slot) k_place_cells<<<grid1d(ncp, CELL_TILE), 256, 0, st>>>((int)ncp, ctx->cells, ctx->gplace_solve, ctx->cursor + CUR_TOTAL);
        fs_status qs = launch_status(ctx, "fs_solve");
        if (qs == FS_OK && d_slot) {
            ctx->slots_N = N;
            ctx->slots_K = K;
            ctx->slots_list = false;
        }
        return qs;
    }
    const int2 *list = nullptr;
    const int *list_len = nullptr;
    S.xcd_ranges = 0;
    int *const cell_count = d_slot ? ctx->cells : nullptr;
    int look_blocks = 0;         // look-back words that the last kernel of this call has to clear
    if (voxel_list) {
        const size_t need_h = (size_t)nb * sblk + 1;
        if ((size_t)N > ctx->vcap) {
            (void)hipStreamSynchronize(st);
            for (void *q : {(void *)ctx->vlist, (void *)ctx->vcnt})
                if (q) (void)hipFree(q);
            ctx->vlist = nullptr;
            ctx->vcnt = nullptr;
            ctx->vcap = 0;
            if (!dev_alloc(&ctx->vlist, (size_t)N * K) || !dev_alloc(&ctx->vcnt, (size_t)N))
                return fail(ctx, FS_E_ALLOC, "fs_solve: out of device memory for the pair list");
            ctx->vcap = (size_t)N;
        }
        if (sorted && ((size_t)N > ctx->vgcell_cap || need_h > ctx->vhist_cap)) {
            (void)hipStreamSynchronize(st);
            for (void *q : {(void *)ctx->vgcell, (void *)ctx->vhist})
                if (q) (void)hipFree(q);
            ctx->vgcell = ctx->vhist = nullptr;
            ctx->vgcell_cap = ctx->vhist_cap = 0;
            if (!dev_alloc(&ctx->vgcell, (size_t)N) || !dev_alloc(&ctx->vhist, need_h))
                return fail(ctx, FS_E_ALLOC, "fs_solve: out of device memory for the pair list");
            ctx->vgcell_cap = (size_t)N;
            ctx->vhist_cap = need_h;
        }
        const size_t boxes = sizeof(float) * 6 * ctx->G.P;
        if (sorted) {
            k_voxel_count<<<grid1d(N, 256), 256, boxes, st>>>(ctx->G, I, N, d_xq, d_pose, ctx->vcnt, ctx->vgcell);
            k_sort_hist<<<(unsigned)sblk, 1024, nb * sizeof(int), st>>>(N, ctx->C.cz, nb, ctx->vgcell, ctx->vcnt, ctx->vhist);
            const int scanned = scan_exclusive(ctx, (int)((long long)nb * sblk), ctx->vhist);
            k_sort_scatter<<<(unsigned)sblk, 1024, nb * sizeof(int), st>>>(N, ctx->C.cz, nb, ctx->vgcell, ctx->vcnt, ctx->vhist, ctx->vlist, ctx->look, scanned);
            list_len = ctx->vhist + (long long)nb * sblk;
            S.xcd_ranges = (!lds && ctx->xcd_ranges) ? 1 : 0;
        } else {
#define FS_LAUNCH_LIST(U)                                                                                              \
    k_voxel_list<U><<<grid1d(N, 1024 * (U)), 1024, boxes, st>>>(ctx->G, I, N, K, d_xq, d_pose, ctx->vcnt, ctx->vlist,  \
                                                                ctx->cursor, ctx->look, ordered)
            // k_voxel_list, us, in the points' order / in the order of the blocks: 0.3 M points of rays or scans 8.7 / 7.6, 1 M 13.4 / 10.9, 2 M 22.9 / 16.4
            const bool ordered = grid_bytes > L2_BYTES;
            const int U = list_per_thread(N);
            look_blocks = ordered ? grid1d(N, 1024 * U) : 0;
            if (U == 2) FS_LAUNCH_LIST(2);
            else if (U == 4) FS_LAUNCH_LIST(4);
            else FS_LAUNCH_LIST(8);
#undef FS_LAUNCH_LIST
            list_len = reinterpret_cast<const int *>(ctx->cursor + CUR_LIST);
        }
        list = ctx->vlist;
    }
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (ctx->timing && hipEventCreate(&ev0) == hipSuccess && hipEventCreate(&ev1) == hipSuccess) (void)hipEventRecord(ev0, st);
    if (lds) {
#define FS_LAUNCH_SOLVE(F, J, NW)                                                                                      \
    k_solve<F, J, NW><<<dim3(blocks), dim3(NW * WAVE), grid_bytes, st>>>(ctx->G, S, I, ctx->T, d_xq, d_pose, d_x0,     \
                                                                         d_Jinv0, d_valid0, ctx->srec, ctx->cursor,    \
                                                                         list, list_len, cell_count, ncell)
        if (lds_big) {
            if (fused && with_J) FS_LAUNCH_SOLVE(true, true, FS_LDS_BIG_WAVES);
            else if (fused) FS_LAUNCH_SOLVE(true, false, FS_LDS_BIG_WAVES);
            else if (with_J) FS_LAUNCH_SOLVE(false, true, FS_LDS_BIG_WAVES);
            else FS_LAUNCH_SOLVE(false, false, FS_LDS_BIG_WAVES);
        } else {
            if (fused && with_J) FS_LAUNCH_SOLVE(true, true, 4);
            else if (fused) FS_LAUNCH_SOLVE(true, false, 4);
            else if (with_J) FS_LAUNCH_SOLVE(false, true, 4);
            else FS_LAUNCH_SOLVE(false, false, 4);
        }
#undef FS_LAUNCH_SOLVE
    } else {
#define FS_LAUNCH_SOLVE(F, J, NC, Z)                                                                                   \
    k_solve_ws<F, J, NC, Z><<<dim3(blocks), dim3((NC + 1) * WAVE), 0, st>>>(                                           \
        ctx->G, S, I, ctx->T, d_xq, d_pose, d_x0, d_Jinv0, d_valid0, ctx->srec, ctx->cursor, list, list_len, cell_count,  \
        ncell, ctx->gave_up_dev, reinterpret_cast<const int *>(ctx->cursor + CUR_GRID))
        // Z = true: contexts with one state per bone.  Many of those lanes start outside the box (51 % of the
        // evaluations on the SMPL-scale scene have a clamped coordinate): the consumers skip the corner records of
        // weight zero (kernel -8 %).  Z = false: voxel-based candidates, which start inside it, where the bookkeeping
        // costs more than it saves (+15 %); with fused initial states the producer reads them from the table
        const bool skip = ctx->prm.init_mode == FS_INIT_BONE;
        if (skip) {
            if (fused && with_J) FS_LAUNCH_SOLVE(true, true, FS_WS_CONSUMERS, true);
            else if (fused) FS_LAUNCH_SOLVE(true, false, FS_WS_CONSUMERS, true);
            else if (with_J) FS_LAUNCH_SOLVE(false, true, FS_WS_CONSUMERS, true);
            else FS_LAUNCH_SOLVE(false, false, FS_WS_CONSUMERS, true);
        } else {
            if (fused && with_J) FS_LAUNCH_SOLVE(true, true, FS_VX_CONSUMERS, false);
            else if (fused) FS_LAUNCH_SOLVE(true, false, FS_VX_CONSUMERS, false);
            else if (with_J) FS_LAUNCH_SOLVE(false, true, FS_WS_CONSUMERS, false);
            else FS_LAUNCH_SOLVE(false, false, FS_WS_CONSUMERS, false);
        }
#undef FS_LAUNCH_SOLVE
    }
    if (ev0 && ev1) {
        (void)hipEventRecord(ev1, st);
        ctx->timed->emplace_back(ev0, ev1);
    }
    // one thread per pair: x = point, y = initial state; rows of blocks before those place the cells
    const int tiles = d_slot ? grid1d(ncp, CELL_TILE) : 0, bx = grid1d(N, 256), rows = (tiles + bx - 1) / bx;
    const dim3 ub(bx, rows + K);
#define FS_LAUNCH_UNPACK(J, Z)                                                                                         \
    k_solve_unpack<J, Z><<<ub, 256, 0, st>>>(N, S.total, (Z) ? ctx->vcnt : nullptr, ctx->srec, d_xc, d_conv, d_Jinv, d_iters, d_slot, ctx->look, \
                                             look_blocks, ctx->cursor, rows, tiles, (int)ncp, ctx->cells, ctx->gplace_solve)
    if (with_J && voxel_list) FS_LAUNCH_UNPACK(true, true);
    else if (with_J) FS_LAUNCH_UNPACK(true, false);
    else if (voxel_list) FS_LAUNCH_UNPACK(false, true);
    else FS_LAUNCH_UNPACK(false, false);
#undef FS_LAUNCH_UNPACK
    fs_status lst = launch_status(ctx, "fs_solve");
    if (lst == FS_OK && d_slot) {
        ctx->slots_N = N;
        ctx->slots_K = K;
        ctx->slots_list = list != nullptr;
    }
    return lst;
}

fs_status fs_grad(fs_ctx *ctx, const float *d_W, const float *d_xc, const float *d_Jinv, const uint8_t *d_conv,
                  const float *d_gxc, const int32_t *d_pose, int64_t N, int32_t K, const int32_t *d_slot, float *d_gW,
                  float *d_gB, float *d_gxq)
{
    if (!ctx) return FS_E_ARG;
    { fs_status gs = check_gave_up(ctx, "fs_grad"); if (gs != FS_OK) return gs; }
    if (!ctx->have_T) return fail(ctx, FS_E_STATE, "fs_grad: call fs_precompute first");
    if (K < 1 || K > FS_MAX_BONES) return fail(ctx, FS_E_SHAPE, "fs_grad: K out of range");
    if (N < 0 || (long long)N * K >= (1ll << 31)) return fail(ctx, FS_E_SHAPE, "fs_grad: need 0 <= N and K*N < 2^31");
    if (ctx->desc.n_poses > 1 && !d_pose && N > 0) return fail(ctx, FS_E_ARG, "fs_grad: d_pose is required when n_poses > 1");
    const int mode = ctx->prm.grad_mode;
    FS_CHECK_PTR(ctx, d_W, false);
    FS_CHECK_PTR(ctx, d_gW, false);
    FS_CHECK_PTR(ctx, d_gB, false);
    FS_CHECK_PTR(ctx, d_gxq, true);
    if (N > 0) {
        FS_CHECK_PTR(ctx, d_xc, false);
        FS_CHECK_PTR(ctx, d_Jinv, mode == FS_GRAD_EXACT_J || d_slot != nullptr);
        FS_CHECK_PTR(ctx, d_conv, false);
        FS_CHECK_PTR(ctx, d_gxc, false);
        FS_CHECK_PTR(ctx, d_pose, true);
    }
    FS_CHECK_PTR(ctx, d_slot, true);
    if (d_slot && (ctx->slots_N != N || ctx->slots_K != K || N == 0))
        return fail(ctx, FS_E_STATE, "fs_grad: d_slot must come from the last fs_solve on this context with the same N and K");
    const bool from_rec = d_slot != nullptr;
    const GridP &G = ctx->G;
    const int ncell = (G.nx - 1) * (G.ny - 1) * (G.nz - 1);
    const long long ncp = (long long)G.P * ncell;
    if (!ctx->GT && !dev_alloc(&ctx->GT, (size_t)G.P * G.V * 12)) return fail(ctx, FS_E_ALLOC, "fs_grad: out of device memory");
    if (!d_slot && !need_places(ctx, &ctx->gplace)) return fail(ctx, FS_E_ALLOC, "fs_grad: out of device memory");
    if (!ctx->gpart) {
        // 16 nodes per wave and pass, so 128 nodes are two passes of a block; no more blocks than are resident with six slots
        // (8 poses of 128x128x32 nodes, us: 512 blocks 82, 768 103, 1024 89; one pose of 65 k nodes: 256 blocks 8.6, 512 6.6)
        ctx->gb_blocks = (int)std::min<long long>(grid1d(G.V, 128), 2ll * ctx->n_cus);
        if (!dev_alloc(&ctx->gpart, (size_t)G.P * ctx->gb_blocks * G.nb * 12)) return fail(ctx, FS_E_ALLOC, "fs_grad: out of device memory");
    }
    const size_t lanes = (size_t)N * K;
    if (lanes > ctx->gcap) {
        (void)hipStreamSynchronize(ctx->stream);
        if (ctx->gpos) (void)hipFree(ctx->gpos);
        if (ctx->grec) (void)hipFree(ctx->grec);
        ctx->gpos = nullptr; ctx->grec = nullptr; ctx->gcap = 0;
        if (!dev_alloc(&ctx->gpos, lanes) || !dev_alloc(&ctx->grec, std::max<size_t>(lanes, PIECE_MIN) * GREC))
            return fail(ctx, FS_E_ALLOC, "fs_grad: out of device memory for %zu lanes", lanes);
        ctx->gcap = lanes;
    }
    { fs_status ls = look_ready(ctx, "fs_grad"); if (ls != FS_OK) return ls; }
    hipStream_t st = ctx->stream;
    // With d_slot the solve has counted its converged lanes per cell, given each its position and placed the cells; all of that is
    // left as it is, so the backward can be repeated
    const int *const pos = d_slot ? d_slot : ctx->gpos, *const places = d_slot ? ctx->gplace_solve : ctx->gplace;
    unsigned *const records = ctx->cursor + CUR_TOTAL + (d_slot ? 0 : 1);
    if (!d_slot) {
        if (N > 0) {
            const int ki = K >= 8 ? 8 : 1;
            const long long waves = ((N + WAVE / ki - 1) / (WAVE / ki)) * ((K + ki - 1) / ki);
            k_grad_count<<<grid1d(waves * WAVE, 256), 256, 0, st>>>(G, d_xc, d_conv, d_pose, N, K, ki, ncell, ctx->cells, ctx->gpos, records);
        }
        k_place_cells<<<grid1d(ncp, CELL_TILE), 256, 0, st>>>((int)ncp, ctx->cells, ctx->gplace, records);
    }
    if (N > 0) {
        // small batches: several threads share a point's lanes so that the chip has enough threads in flight
        const int groups = N >= (1 << 19) ? 1 : (K >= 8 ? 8 : (K >= 4 ? 4 : (K >= 2 ? 2 : 1)));
        const dim3 rg(grid1d(N, 256 / groups));
        float4 *grec4 = reinterpret_cast<float4 *>(ctx->grec);
        const int *state = reinterpret_cast<const int *>(ctx->cursor + CUR_GRID);
#define FS_LAUNCH_RECORDS(R, ...)                                                                                     \
    k_grad_records<R, __VA_ARGS__><<<rg, 256, 0, st>>>(G, ctx->T, d_xc, d_Jinv, d_conv, d_gxc, d_pose, N, K, ncell, places, pos, \
                                                       grec4, d_gxq, groups, (R) ? ctx->srec : nullptr,               \
                                                       ((R) && ctx->slots_list) ? ctx->vcnt : nullptr, state)
#define FS_LAUNCH_EXACT(J)                                                                                            \
    do {                                                                                                              \
        if (from_rec) FS_LAUNCH_RECORDS(true, J);                                                                     \
        else FS_LAUNCH_RECORDS(false, J);                                                                             \
    } while (0)
        // from_rec: the solve's own result records are still in the context: one 64-byte read per pair
        // The exact Jacobian: many roots of bone states lie beyond the box, where half the corners or more are left out; candidates' roots
        // seldom do.  For those, on a grid that the L2 holds waves in flight count most, and beyond it that the two z-neighbours of
        // a corner, one or two cache lines, are asked for together.  fs_grad, us, all corners / halves / without weight zero: bones, 65 k points 135 / 130 /
        // 123, 200 k points on 128x128x32 nodes 502 / 469 / 437; candidates on 64x64x16 nodes, 0.5 M ray samples 54 / 57 / 66, 2 M 106 / 113 / 144, 0.5 M points of scans
        // 99 / 94 / 106; 2 M ray samples on 84x84x21 (7 MB) 170 / 171 / 202, on 128x128x32 288 / 278 / 305, 1 M of scans 457 / 398 / 380.
        if (mode == 0) {
            if (from_rec && groups == 1) FS_LAUNCH_RECORDS(true, JAC_BROYDEN, 3);     // large batches: three lanes of a point in flight, stage by stage
            else if (from_rec) FS_LAUNCH_RECORDS(true, JAC_BROYDEN);
            else FS_LAUNCH_RECORDS(false, JAC_BROYDEN);
        } else if (ctx->prm.init_mode == FS_INIT_BONE) FS_LAUNCH_EXACT(JAC_CLAMPED);
        else if ((size_t)G.P * G.V * 48 > L2_BYTES) FS_LAUNCH_EXACT(JAC_HALVES);
        else FS_LAUNCH_EXACT(JAC_CELL);
#undef FS_LAUNCH_EXACT
#undef FS_LAUNCH_RECORDS
    }
    if (N > 0) k_grad_pieces<<<grid1d((long long)lanes, PIECE_R), 64 * PIECE_WAVES, 0, st>>>(G, records, ctx->grec);
    // crowded grids: one thread per (node, adjacent cell); sparse ones: one thread per node, which walks the 4 cells at
    // its height and hands their share for the node above to the next SIMD lane
    const long long nodes = (long long)G.P * G.V;
    if ((long long)lanes >= 8 * nodes)
        k_grad_nodes_p<<<grid1d(nodes * 8, 256), 256, 0, st>>>(G, ncell, places, ctx->grec, ctx->GT);
    else
        k_grad_nodes_z<<<grid1d(nodes, 256), 256, 0, st>>>(G, ncell, places, ctx->grec, ctx->GT);
    const int nout = G.nb * 12;
#define FS_LAUNCH_OUT_S(MT, S) k_grad_outputs<MT, S><<<ctx->gb_blocks, 256, 0, st>>>(G, d_W, ctx->GT, ctx->Bdev, d_gW, ctx->gpart)
#define FS_LAUNCH_OUT(MT)                                                                                              \
    do {                                                                                                               \
        if (G.P == 1) FS_LAUNCH_OUT_S(MT, 1);                                                                          \
        else FS_LAUNCH_OUT_S(MT, 3);                                                                                   \
    } while (0)
    switch ((G.nb + 15) / 16) {
    case 1:
        if (G.P > 4) FS_LAUNCH_OUT_S(1, 6);
        else FS_LAUNCH_OUT(1);
        break;
    case 2:
        if (G.P > 4) FS_LAUNCH_OUT_S(2, 6);
        else FS_LAUNCH_OUT(2);
        break;
    case 3: FS_LAUNCH_OUT(3); break;
    default: FS_LAUNCH_OUT(4); break;
    }
#undef FS_LAUNCH_OUT
#undef FS_LAUNCH_OUT_S
    k_grad_bones_final<<<dim3(grid1d(nout, 16), G.P), 1024, 0, st>>>(ctx->gb_blocks, nout, ctx->gpart, d_gB);
    return launch_status(ctx, "fs_grad");
}

// k_dedupe_one where it is the shorter; false: not launched.  At most DD_FEW lanes: for few blocks, while look-back costs less than a launch (served ray
// samples with candidates, whole call, us, two launches / one: 37 points 15.7 / 13.4, 1024 20.7 / 18.5, 5000 22.2 / 21.2, 12 k 23.8 / 23.1, 25 k
// 24.9 / 24.5, 60 k 33.9 / 34.5).  More than 32 lanes: the other kernels hand on 32 bits per point and read the kept lanes again (64 states: 37 points
// 39 / 29, 3000 87 / 71, 32 k 345 / 326).  Between, two launches are as short or shorter (24 states, 37 points 29.8 / 29.8, 1500 38.9 / 41.1).
static bool launch_dedupe_one(fs_ctx *ctx, long long N, int K, float md2, const float *d_xc, const uint8_t *d_conv, uint8_t *d_keep,
                              int32_t *d_offsets, float *d_roots, int32_t *d_lane, long long cap)
{
    u64 *const look = ctx->look + ctx->dd_look_at;
    if (K <= DD_FEW && N <= 16 * 1024)
        k_dedupe_one<0><<<grid1d(N, 1024), 1024, 0, ctx->stream>>>(N, K, cap, md2, d_xc, d_conv, d_keep, d_offsets, d_roots, d_lane, look);
    else if (K > 32 && N <= 128ll * DD_ONE_BLOCKS)
        k_dedupe_one<8><<<grid1d(N, 128), 1024, 0, ctx->stream>>>(N, K, cap, md2, d_xc, d_conv, d_keep, d_offsets, d_roots, d_lane, look);
    else return false;
    return true;
}

// shared body of fs_dedupe and fs_dedupe_noalloc, which differ in where the tile sums live
static fs_status dedupe_impl(fs_ctx *ctx, const char *who, int *sums, const float *d_xc, const uint8_t *d_conv, int64_t N,
                             int32_t K, float min_dist, uint8_t *d_keep, int32_t *d_offsets, float *d_roots, int32_t *d_lane,
                             int64_t cap)
{
    if (K < 1 || K > FS_MAX_BONES) return fail(ctx, FS_E_SHAPE, "%s: K must be in 1..%d", who, (int)FS_MAX_BONES);
    if (N < 0 || (long long)N * K >= (1ll << 31)) return fail(ctx, FS_E_SHAPE, "%s: need 0 <= N and K*N < 2^31", who);
    if (sums != ctx->dd_sums && N > FS_NOALLOC_MAX_N)
        return fail(ctx, FS_E_SHAPE, "%s: N = %lld exceeds the %lld points that the call with fixed scratch memory takes; use fs_dedupe",
                    who, (long long)N, FS_NOALLOC_MAX_N);
    if (!(min_dist >= 0.0f) || !std::isfinite(min_dist)) return fail(ctx, FS_E_ARG, "%s: min_dist must be finite and >= 0", who);
    if (cap < 0) return fail(ctx, FS_E_SHAPE, "%s: cap must be >= 0", who);
    FS_CHECK_PTR(ctx, d_offsets, false);
    FS_CHECK_PTR(ctx, d_roots, true);
    FS_CHECK_PTR(ctx, d_lane, true);
    hipStream_t st = ctx->stream;
    if (N > 0) {
        FS_CHECK_PTR(ctx, d_xc, false);
        FS_CHECK_PTR(ctx, d_conv, false);
        FS_CHECK_PTR(ctx, d_keep, false);
        if (sums == ctx->dd_sums && launch_dedupe_one(ctx, N, K, min_dist * min_dist, d_xc, d_conv, d_keep, d_offsets, d_roots, d_lane, cap))
            return launch_status(ctx, who);
        const bool four = K <= DD_FEW && N >= 1 << 19;         // one point per thread / four, whole call, us: 66 k points 7.5 / 8.1, 262 k 9.1 / 9.7, 524 k 12.9 / 12.6, 1 M 24.9 / 20.5, 4.2 M 78.5 / 73.1
        int tile = K <= DD_FEW ? 256 : 32;          // what a block takes in one pass
        while ((N + tile - 1) / tile > DD_TILES) tile *= 2;
        const int tiles = grid1d(N, tile);
        const int threads = four ? std::min(256, tile / 4) : 256;
#define FS_LAUNCH_DEDUPE(KERNEL) KERNEL<<<tiles, threads, 0, st>>>(N, K, min_dist * min_dist, d_xc, d_conv, d_keep, d_offsets, tile, sums)
        if (four) FS_LAUNCH_DEDUPE(k_dedupe_few<4>);
        else if (K <= DD_FEW) FS_LAUNCH_DEDUPE(k_dedupe_few<1>);
        else if (K <= 8) FS_LAUNCH_DEDUPE(k_dedupe<1>);
        else if (K <= 16) FS_LAUNCH_DEDUPE(k_dedupe<2>);
        else if (K <= 24) FS_LAUNCH_DEDUPE(k_dedupe<3>);
        else if (K <= 32) FS_LAUNCH_DEDUPE(k_dedupe<4>);
        else FS_LAUNCH_DEDUPE(k_dedupe<8>);
#undef FS_LAUNCH_DEDUPE
        k_dedupe_pack<<<tiles, 256, 0, st>>>(N, K, cap, d_xc, d_keep, d_offsets, tile, sums, d_roots, d_lane);
    } else {
        k_fill_zero_i32<<<1, 64, 0, st>>>(1, d_offsets);
    }
    return launch_status(ctx, who);
}

fs_status fs_dedupe(fs_ctx *ctx, const float *d_xc, const uint8_t *d_conv, int64_t N, int32_t K, float min_dist,
                    uint8_t *d_keep, int32_t *d_offsets, float *d_roots, int32_t *d_lane, int64_t cap)
{
    if (!ctx) return FS_E_ARG;
    { fs_status gs = check_gave_up(ctx, "fs_dedupe"); if (gs != FS_OK) return gs; }
    { fs_status ls = look_ready(ctx, "fs_dedupe"); if (ls != FS_OK) return ls; }
    return dedupe_impl(ctx, "fs_dedupe", ctx->dd_sums, d_xc, d_conv, N, K, min_dist, d_keep, d_offsets, d_roots, d_lane, cap);
}

fs_status fs_dedupe_noalloc(fs_ctx *ctx, const float *d_xc, const uint8_t *d_conv, int64_t N, int32_t K, float min_dist,
                            uint8_t *d_keep, int32_t *d_offsets, float *d_roots, int32_t *d_lane, int64_t cap)
{
    if (!ctx) return FS_E_ARG;
    { fs_status gs = check_gave_up(ctx, "fs_dedupe_noalloc"); if (gs != FS_OK) return gs; }
    int *sums = scratch_on_device(ctx);
    if (!sums) return fail(ctx, FS_E_DEVICE, "fs_dedupe_noalloc: the address of the library's scratch array could not be obtained "
                                             "(the context's device must be the current one)");
    return dedupe_impl(ctx, "fs_dedupe_noalloc", sums, d_xc, d_conv, N, K, min_dist, d_keep, d_offsets, d_roots, d_lane, cap);
}

fs_status fs_set_timing(fs_ctx *ctx, int32_t enable)
{
    if (!ctx) return FS_E_ARG;
    if (enable && !ctx->timed) {
        ctx->timed = new (std::nothrow) std::vector<std::pair<hipEvent_t, hipEvent_t>>();
        if (!ctx->timed) return fail(ctx, FS_E_ALLOC, "fs_set_timing: out of host memory");
    }
    ctx->timing = enable != 0;
    return FS_OK;
}

fs_status fs_get_timing(fs_ctx *ctx, double *solve_kernel_ms, int32_t *launches)
{
    if (!ctx || !solve_kernel_ms || !launches) return FS_E_ARG;
    { fs_status gs = check_gave_up(ctx, "fs_get_timing"); if (gs != FS_OK) return gs; }
    *solve_kernel_ms = 0.0;
    *launches = 0;
    if (!ctx->timed) return FS_OK;
    if (hipStreamSynchronize(ctx->stream) != hipSuccess) return launch_status(ctx, "fs_get_timing");
    for (auto &e : *ctx->timed) {
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, e.first, e.second) == hipSuccess) {
            *solve_kernel_ms += ms;
            ++*launches;
        }
        (void)hipEventDestroy(e.first);
        (void)hipEventDestroy(e.second);
    }
    (void)hipGetLastError();
    ctx->timed->clear();
    return FS_OK;
}

fs_status fs_get_transforms(fs_ctx *ctx, float *d_T)
{
    if (!ctx) return FS_E_ARG;
    if (!ctx->have_T) return fail(ctx, FS_E_STATE, "fs_get_transforms: call fs_precompute first");
    FS_CHECK_PTR(ctx, d_T, false);
    if (hipMemcpyAsync(d_T, ctx->T, sizeof(float) * ctx->G.P * ctx->G.V * 12, hipMemcpyDeviceToDevice, ctx->stream) != hipSuccess)
        return launch_status(ctx, "fs_get_transforms");
    return FS_OK;
}

fs_status fs_get_corr(fs_ctx *ctx, float *d_bbox, int32_t *d_cand)
{
    if (!ctx) return FS_E_ARG;
    if (ctx->prm.init_mode != FS_INIT_VOXEL) return fail(ctx, FS_E_STATE, "fs_get_corr: context was not created with FS_INIT_VOXEL");
    if (!ctx->have_T) return fail(ctx, FS_E_STATE, "fs_get_corr: call fs_precompute first");
    FS_CHECK_PTR(ctx, d_bbox, false);
    FS_CHECK_PTR(ctx, d_cand, false);
    hipError_t e = hipMemcpyAsync(d_bbox, ctx->bbox, sizeof(float) * ctx->G.P * 6, hipMemcpyDeviceToDevice, ctx->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(d_cand, ctx->cand, sizeof(int32_t) * ctx->G.P * (size_t)ctx->C.ncell * ctx->C.ck,
                           hipMemcpyDeviceToDevice, ctx->stream);
    if (e != hipSuccess) return launch_status(ctx, "fs_get_corr");
    return FS_OK;
}

}  // extern "C"
