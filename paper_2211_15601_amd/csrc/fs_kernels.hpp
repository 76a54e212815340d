// HIP kernels of the articulation path for gfx950 (wave64).
#pragma once
#include "fs_field.hpp"

namespace fs {

constexpr int WAVE = 64, N_XCD = 8;

// Corner records of weight zero may be left out while no product of an entry with a position is infinite (0 * inf is not 0):
// entries and positions below this number, whose products add up to less than 2^123.
constexpr float SKIP_MAX = 0x1p60f;

// pose index of point n, forced into [0, P) so that a bad index in the caller's array cannot send
// a kernel outside the transform grids
__device__ __forceinline__ int pose_of(const int32_t *__restrict__ pose, long long n, int P)
{
    if (!pose) return 0;
    const int p = pose[n];
    return p < 0 ? 0 : (p >= P ? P - 1 : p);
}
constexpr int FS_MAX_CORR_K_DEV = 8, FS_BONES_MAX = 64;

// number of lanes of the wave with `on`, as a scalar (the compiler compares a 64-bit population count on the vector unit)
__device__ __forceinline__ int lanes_on(bool on) { return __builtin_amdgcn_readfirstlane(__popcll(__ballot(on))); }

// Two words about the grid that stands, both written by k_precompute: the number of the call that made it, and the number of the last call
// whose grid had an entry that is not finite or not below SKIP_MAX.  Where they are equal, records of weight zero are not skipped.
// Both are on the device because a recorded graph keeps the numbers it was recorded with, whatever calls came between its
// replays: a replay of a recorded fs_precompute writes its own number, and whoever reads asks about the grid that is there.  (A recorded call
// that has once made such a grid is taken to make one at every later replay: right, and slower.)
enum { GRID_NUMBER = 0, GRID_REFUSED = 1 };
__device__ __forceinline__ bool may_skip_corners(const int *__restrict__ state)
{
    return __builtin_amdgcn_readfirstlane(state[GRID_NUMBER]) != __builtin_amdgcn_readfirstlane(state[GRID_REFUSED]);
}

// ------------------------------------------------------------------------------------------------
// Pre-computed LBS (Eq. (13)): one thread per node, all poses.  The bone transforms are read with
// wave-uniform addresses, i.e. through the scalar cache into SGPR operands of the multiply-adds.
// Reads W once (96 B / node for 24 bones), writes 48 B per node and pose.
// ------------------------------------------------------------------------------------------------
// Every lane of a wave holds one row of NF floats (NF = 12: a 48-byte record; NF = 3: a point) of a tile whose rows are
// contiguous in memory (row r of the wave's tile at dst + r * NF).  Stored straight from registers, a row goes out as
// 16-byte pieces at a 48-byte stride: partial writes of cache lines, for which the L2 first fetches the line (on the
// 8-pose 128x128x32 grid k_precompute fetched 386 MB to read 50 MB of weights).  Through LDS the tile leaves as whole,
// consecutive 16-byte pieces from consecutive lanes.  nrows = valid rows of the wave's tile (wave-uniform; <= 0: none).
// s_tile: 64 * NF floats of LDS that belong to this wave alone, so no barrier between waves is needed; all 64 lanes
// must call.
template <int NF>
__device__ __forceinline__ void wave_store_rows(float *__restrict__ dst, const float (&v)[NF], int nrows, float *s_tile)
{
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // s_tile may still be read from the call before
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int e = 0; e < NF; ++e) s_tile[lane * NF + e] = v[e];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int n4 = nrows * NF / 4, tail = nrows * NF - n4 * 4;
    if ((reinterpret_cast<uintptr_t>(dst) & 15u) == 0) {
        for (int i = lane; i < n4; i += 64)
            reinterpret_cast<float4 *>(dst)[i] = reinterpret_cast<const float4 *>(s_tile)[i];
        if (lane < tail) dst[n4 * 4 + lane] = s_tile[n4 * 4 + lane];
    } else {
        for (int i = lane; i < nrows * NF; i += 64) dst[i] = s_tile[i];
    }
}

__device__ __forceinline__ void bone_inverse(int i, const float *__restrict__ B, float *__restrict__ Bcopy,
                                             float *__restrict__ Binv, uint8_t *__restrict__ ok);

// monotone float <-> uint mapping so that min / max can use integer atomics (exact, order-free)
__device__ __forceinline__ unsigned f2ord(float f)
{
    const unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ord2f(unsigned o)
{
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// smallest v of the 64 lanes in lane 31, complement of the largest in lane 63; all lanes must call.  Lanes without a value: lo = hi = ~0.
// (lo = v, hi = ~v: one exchange of the wave's halves leaves 32 lanes to each of the two.)
__device__ __forceinline__ unsigned wave_extent(unsigned lo, unsigned hi)
{
    const auto s = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
    unsigned v = min((unsigned)s[0], (unsigned)s[1]);
#define FS_EXTENT_STEP(ctrl, rows) v = min(v, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)v, (ctrl), (rows), 0xf, false))
    FS_EXTENT_STEP(0x111, 0xf);         // row_shr 1, 2, 4, 8: within rows of 16 lanes
    FS_EXTENT_STEP(0x112, 0xf);
    FS_EXTENT_STEP(0x114, 0xf);
    FS_EXTENT_STEP(0x118, 0xf);
    FS_EXTENT_STEP(0x142, 0xa);         // row_bcast 15 into rows 1 and 3
#undef FS_EXTENT_STEP
    return v;
}

// n_poses*n_bones threads also invert a bone's linear part for Eq. (8) and keep a copy of the bone transforms for the backward.
// Y (may be null; voxel-based initial states): the image y_v = T_v x_v of every node is written as well -- the
// correspondence grid is built on those, and the transforms are in registers here anyway (a pass of its own would
// read all of T again).  So are the extents of a block's images (bb_part[p][entry][block], ordered-integer images of the
// floats: min x, y, z, max x, y, z), and the counters of the correspondence cells are cleared on the way.  (A kernel
// each for the extents and the counters: two launches, 16 us together on the 8-pose grid.)
// NP: poses that share one pass over a node's weights.  Large grids, bound by memory: four (8-pose 128x128x32 grid: 1 -> 109 us,
// 2 -> 86, 4 -> 87; all groups of a node on one XCD: 110 -> 87).  Grids of fewer than four blocks of 256 nodes per CU: one,
// so that there are waves to hide the latency of weights and transforms (4 poses of 61x47x13 nodes: 4 -> 27 us, 2 -> 16, 1 -> 10).
// FEW: no more than two blocks of one pose per CU.  A wave has no other to hide behind: the bones come from LDS and the next eight weights are on
// their way while eight are worked in, so that it waits for memory once, not for scalar operands and weights every four bones (64x64x16 nodes: 24 bones
// 10.2 -> 7.5 us, a frame with 64 bones 54 -> 48).  With more blocks LDS is the slower source (four poses 14.4, from LDS 15.9).
template <int NP, bool FEW>
__global__ __launch_bounds__(256) void k_precompute(GridP G, const float *__restrict__ W,
                                                    const float *__restrict__ B, float *__restrict__ T,
                                                    float *__restrict__ Bcopy, float *__restrict__ Binv,
                                                    uint8_t *__restrict__ Bok, int *__restrict__ state,
                                                    int serial, float *__restrict__ Y, unsigned *__restrict__ bb_part,
                                                    int *__restrict__ ccount, int ncount, int vblocks, int groups)
{
    // block -> (nodes, group of poses): blocks go to the 8 XCDs in turn, the groups of the same nodes to the same XCD one
    // after the other, so that its L2 has the weights
    const int t = (int)blockIdx.x / N_XCD, bt = t / groups, group = t - bt * groups, blk = bt * N_XCD + (int)blockIdx.x % N_XCD;
    if (FEW && blk == vblocks && group == 0)          // a block without nodes, which would be the last to end if it had some, inverts the bones
        for (int i = threadIdx.x; i < G.P * G.nb; i += blockDim.x) bone_inverse(i, B, Bcopy, Binv, Bok);
    if (blk >= vblocks) return;
    __shared__ __attribute__((aligned(16))) float s_tiles[4][64 * 12];
    __shared__ unsigned s_ext[NP][4][6];
    const int wib = threadIdx.x >> 6;
    float *s_tile = s_tiles[wib];
    const long long v = (long long)blk * blockDim.x + threadIdx.x, v0 = v - (threadIdx.x & 63);   // v0: the wave's first node
    if (group == 0) {
        if (v == 0) state[GRID_NUMBER] = serial;
        if (!FEW)
            for (long long i = v; i < (long long)G.P * G.nb; i += (long long)vblocks * blockDim.x)
                bone_inverse((int)i, B, Bcopy, Binv, Bok);
        if (Y)
            for (long long i = v; i < ncount; i += (long long)vblocks * blockDim.x) ccount[i] = 0;
    }
    const bool live = v < G.V;                   // the last wave: its other lanes stay for the wave-wide stores
    const int nrows = (int)min(64ll, G.V - v0);
    const float *w = W + (live ? v : 0) * G.nb;
    const bool vec = (G.nb & 3) == 0;        // weight rows are 16-byte aligned: read them four at a time
    float xv[3] = {0.0f, 0.0f, 0.0f};
    if (Y && live) node_pos(G, v, xv);
    // per pose the sum runs over the bones in order, first term a product, the rest fused multiply-adds
    const int p0 = group * NP, np = min(NP, G.P - p0);
    float acc[NP][12];
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int e = 0; e < 12; ++e) acc[q][e] = 0.0f;
    if constexpr (FEW) {
        static_assert(NP == 1, "one pose's bones are staged");
        __shared__ float4 s_bone[FS_BONES_MAX * 3];
        const float4 *Bp = reinterpret_cast<const float4 *>(B + (long long)p0 * G.nb * 12);
        for (int i = threadIdx.x; i < G.nb * 3; i += 256) s_bone[i] = Bp[i];
        float wn[8];
        auto weights = [&](int b0) {
#pragma unroll
            for (int j = 0; j < 8; j += 4) {
                float4 w4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (vec) {
                    if (b0 + j < G.nb) w4 = *reinterpret_cast<const float4 *>(w + b0 + j);
                } else {
                    if (b0 + j < G.nb) w4.x = w[b0 + j];
                    if (b0 + j + 1 < G.nb) w4.y = w[b0 + j + 1];
                    if (b0 + j + 2 < G.nb) w4.z = w[b0 + j + 2];
                    if (b0 + j + 3 < G.nb) w4.w = w[b0 + j + 3];
                }
                wn[j] = w4.x; wn[j + 1] = w4.y; wn[j + 2] = w4.z; wn[j + 3] = w4.w;
            }
        };
        weights(0);
        __syncthreads();
        for (int b0 = 0; b0 < G.nb; b0 += 8) {
            float wv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) wv[j] = wn[j];
            weights(b0 + 8);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (b0 + j < G.nb) {
                    const float4 r0 = s_bone[(b0 + j) * 3], r1 = s_bone[(b0 + j) * 3 + 1], r2 = s_bone[(b0 + j) * 3 + 2];
                    const float bone[12] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w, r2.x, r2.y, r2.z, r2.w};
#pragma unroll
                    for (int e = 0; e < 12; ++e) acc[0][e] = b0 + j == 0 ? wv[0] * bone[e] : FS_FMA(wv[j], bone[e], acc[0][e]);
                }
            }
        }
    } else if (live) {
        for (int b0 = 0; b0 < G.nb; b0 += 4) {
            float wv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (vec) {
                const float4 w4 = *reinterpret_cast<const float4 *>(w + b0);
                wv[0] = w4.x; wv[1] = w4.y; wv[2] = w4.z; wv[3] = w4.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (b0 + j < G.nb) wv[j] = w[b0 + j];
            }
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                if (q < np) {
                    const float *Bp = B + (long long)(p0 + q) * G.nb * 12;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (b0 + j < G.nb) {
                            if (b0 == 0 && j == 0) {
#pragma unroll
                                for (int e = 0; e < 12; ++e) acc[q][e] = wv[0] * Bp[e];
                            } else {
#pragma unroll
                                for (int e = 0; e < 12; ++e) acc[q][e] = FS_FMA(wv[j], Bp[(b0 + j) * 12 + e], acc[q][e]);
                            }
                        }
                    }
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        if (q < np) {                        // wave-uniform
            if (live) {
                float big = 0.0f;
#pragma unroll
                for (int e = 0; e < 12; ++e) big = __builtin_fmaxf(big, __builtin_fabsf(acc[q][e]) < SKIP_MAX ? 0.0f : 1.0f);
                if (big != 0.0f) state[GRID_REFUSED] = serial;
            }
            wave_store_rows<12>(T + ((long long)(p0 + q) * G.V + v0) * 12, acc[q], nrows, s_tile);
            if (Y) {
                float y[3] = {0.0f, 0.0f, 0.0f};
                if (live) apply12(acc[q], xv, y);
                wave_store_rows<3>(Y + ((long long)(p0 + q) * G.V + v0) * 3, y, nrows, s_tile);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const unsigned o = f2ord(y[a]);
                    const unsigned r = wave_extent(live ? o : ~0u, live ? ~o : ~0u);
                    if ((threadIdx.x & 63) == 31) s_ext[q][wib][a] = r;
                    if ((threadIdx.x & 63) == 63) s_ext[q][wib][3 + a] = ~r;
                }
            }
        }
    }
    if (!Y) return;
    __syncthreads();
    if (threadIdx.x < 6 * np) {
        const int q = threadIdx.x / 6, e = threadIdx.x - 6 * q;
        const unsigned a = s_ext[q][0][e], b = s_ext[q][1][e], c = s_ext[q][2][e], d = s_ext[q][3][e];
        bb_part[((long long)(p0 + q) * 6 + e) * vblocks + blk] = e < 3 ? min(min(a, b), min(c, d)) : max(max(a, b), max(c, d));
    }
}

// Inverse of one bone's linear part for Eq. (8): Binv [P][nb][12] = 9 inverse entries + t, ok flag.
__device__ __forceinline__ void bone_inverse(int i, const float *__restrict__ B, float *__restrict__ Bcopy,
                                             float *__restrict__ Binv, uint8_t *__restrict__ ok)
{
    const float *b = B + i * 12;
    for (int e = 0; e < 12; ++e) Bcopy[i * 12 + e] = b[e];
    const float R[9] = {b[0], b[1], b[2], b[4], b[5], b[6], b[8], b[9], b[10]};
    float Ri[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    const bool good = inv3(R, Ri);
    for (int e = 0; e < 9; ++e) Binv[i * 12 + e] = Ri[e];
    Binv[i * 12 + 9] = b[3];
    Binv[i * 12 + 10] = b[7];
    Binv[i * 12 + 11] = b[11];
    ok[i] = good ? 1 : 0;
}

// Corners that can have a non-zero weight: along a clamped axis only the side the point was clamped to
// (fraction 0: offset 0, fraction 1: offset 1).  An axis that merely happens to have fraction 0 keeps both sides.
__device__ __forceinline__ int corners_needed(const Cell &c)
{
    const int mx = c.cl[0] ? (c.f[0] == 0.0f ? 0x55 : 0xAA) : 0xFF;
    const int my = c.cl[1] ? (c.f[1] == 0.0f ? 0x33 : 0xCC) : 0xFF;
    const int mz = c.cl[2] ? (c.f[2] == 0.0f ? 0x0F : 0xF0) : 0xFF;
    return mx & my & mz;
}

// Jacobian (and field) of a fresh pair from the corners in `need` (zeros in place of the others): the arithmetic of
// jacobian_from_corners, but the corners are fetched in two halves, the z-pairs of one x, y side and then of the other: with all eight
// records in registers the producer of k_solve_ws, not its consumers, would decide how many waves a SIMD holds (197 registers with J~ and 179
// without, where three waves leave 168 to each).  Returns whether an entry of the blend or of the Jacobian is an exact zero.
__device__ __forceinline__ bool prepare_jacobian(const float *__restrict__ Tcell, const GridP &G, const Cell &c, int need, const float (&x)[3],
                                                 float (&d)[3], float (&J)[9])
{
    float om[8], T[12], dc[8][3], q[2][4][12];          // q[h]: corners 2h, 2h + 4, 2h + 1, 2h + 5
    corner_weights(c, om);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 2 * h + (i >> 1) + 4 * (i & 1);
#pragma unroll
            for (int e = 0; e < 12; ++e) q[h][i][e] = 0.0f;
            if ((need >> k) & 1) load12(Tcell + corner_off(G, k), q[h][i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) apply12(q[h][i], x, dc[2 * h + (i >> 1) + 4 * (i & 1)]);
#pragma unroll
        for (int i = 0; i < 4; i += 2)
#pragma unroll
            for (int e = 0; e < 12; ++e) T[e] = h + i == 0 ? om[0] * q[0][0][e] : FS_FMA(om[2 * h + (i >> 1)], q[h][i][e], T[e]);
        // nothing is moved across: the lower corners of this half have been added when the other half is asked for
#pragma unroll
        for (int e = 0; e < 12; ++e) asm volatile("" : "+v"(T[e]));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 2 * h + (i >> 1) + 4 * (i & 1);
            asm volatile("" : "+v"(dc[k][0]), "+v"(dc[k][1]), "+v"(dc[k][2]) : : "memory");
        }
    }
#pragma unroll
    for (int k = 4; k < 8; ++k)
#pragma unroll
        for (int e = 0; e < 12; ++e) T[e] = FS_FMA(om[k], q[(k - 4) >> 1][((k & 1) << 1) + 1][e], T[e]);
    apply12(T, x, d);
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int j = 0; j < 3; ++j) J[r * 3 + j] = T[r * 4 + j];
#pragma unroll
    for (int k = 0; k < 8; ++k) add_weight_derivative(G, c, k, dc[k], J);
    float m = __builtin_fabsf(T[0]);
#pragma unroll
    for (int e = 1; e < 12; ++e) m = __builtin_fminf(m, __builtin_fabsf(T[e]));
#pragma unroll
    for (int e = 0; e < 9; ++e) m = __builtin_fminf(m, __builtin_fabsf(J[e]));
    return m == 0.0f;
}

// field_dJ without the corners of weight zero, whose records contribute nothing (the derivative of their weight vanishes along the
// clamped axis by definition and carries the zero factor along the others): zeros in their place, and if an entry of the blend or of
// the Jacobian comes out as an exact zero, again with all eight.  may_skip: the grid's entries are below SKIP_MAX.
// Bound: the gathers.  (fs_init, us, all eight / these: 30 k points x 17 bones on 32x32x8 nodes 27 / 20, 65 k x 24 on 64x64x16 85 / 50, 20 k x 24 on
// 128x128x32 48 / 32.)
__device__ __forceinline__ void field_dJ_clamped(const float *__restrict__ Tp, const GridP &G, const Cell &c, bool may_skip, const float (&x)[3],
                                                 float (&d)[3], float (&J)[9])
{
    const bool near = __builtin_fabsf(x[0]) < SKIP_MAX && __builtin_fabsf(x[1]) < SKIP_MAX && __builtin_fabsf(x[2]) < SKIP_MAX;
    int need = may_skip && near ? corners_needed(c) : 0xFF;
    while (prepare_jacobian(Tp + c.base, G, c, need, x, d, J) && need != 0xFF) need = 0xFF;
}

// ------------------------------------------------------------------------------------------------
// Initial states.  One thread per lane q = k*N + n.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void write_init(long long q, long long N, int k, long long n, const float x0[3],
                                           const float Ji[9], bool ok, float *__restrict__ o_x0,
                                           float *__restrict__ o_J, uint8_t *__restrict__ o_v)
{
#pragma unroll
    for (int r = 0; r < 3; ++r) o_x0[((long long)k * 3 + r) * N + n] = x0[r];
#pragma unroll
    for (int e = 0; e < 9; ++e) o_J[((long long)k * 9 + e) * N + n] = ok ? Ji[e] : 0.0f;
    o_v[q] = ok ? 1 : 0;
}

__global__ __launch_bounds__(256) void k_init_bone(GridP G, const float *__restrict__ T,
                                                   const float *__restrict__ Binv, const uint8_t *__restrict__ Bok,
                                                   const float *__restrict__ xq, const int32_t *__restrict__ pose,
                                                   long long N, float *__restrict__ o_x0, float *__restrict__ o_J,
                                                   uint8_t *__restrict__ o_v, const int *__restrict__ state)
{
    const bool may_skip = may_skip_corners(state);
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N * G.nb) return;
    const int k = (int)(q / N);
    const long long n = q - (long long)k * N;
    const int p = pose_of(pose, n, G.P);
    const float *bi = Binv + ((long long)p * G.nb + k) * 12;
    float x0[3] = {0, 0, 0}, Ji[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    bool ok = Bok[p * G.nb + k] != 0;
    if (ok) {
        const float y[3] = {xq[n] - bi[9], xq[N + n] - bi[10], xq[2 * N + n] - bi[11]};
#pragma unroll
        for (int r = 0; r < 3; ++r)
            x0[r] = FS_FMA(bi[r * 3 + 0], y[0], FS_FMA(bi[r * 3 + 1], y[1], bi[r * 3 + 2] * y[2]));
        float d[3], J[9];
        field_dJ_clamped(T + (long long)p * G.V * 12, G, locate(G, x0), may_skip, x0, d, J);
        ok = inv3(J, Ji);
    }
    write_init(q, N, k, n, x0, Ji, ok, o_x0, o_J, o_v);
}

struct CorrP {
    int cx, cy, cz, ck;
    int ncell;
};

__device__ __forceinline__ int cell_coord(float y, float blo, float cs, int n)
{
    if (!(cs > 0.0f)) return 0;
    float t = (y - blo) / cs;
    if (!(t >= 0.0f)) t = 0.0f;
    if (t > (float)(n - 1)) t = (float)(n - 1);
    return (int)t;
}

__device__ __forceinline__ int cell_index(const CorrP &C, const float *__restrict__ bb, const float y[3])
{
    const float cs0 = (bb[3] - bb[0]) / (float)C.cx;
    const float cs1 = (bb[4] - bb[1]) / (float)C.cy;
    const float cs2 = (bb[5] - bb[2]) / (float)C.cz;
    return (cell_coord(y[0], bb[0], cs0, C.cx) * C.cy + cell_coord(y[1], bb[1], cs1, C.cy)) * C.cz +
           cell_coord(y[2], bb[2], cs2, C.cz);
}

__global__ __launch_bounds__(256) void k_init_voxel(GridP G, CorrP C, const float *__restrict__ bbox,
                                                    const float4 *__restrict__ cinit, const float *__restrict__ xq,
                                                    const int32_t *__restrict__ pose, long long N,
                                                    float *__restrict__ o_x0, float *__restrict__ o_J,
                                                    uint8_t *__restrict__ o_v)
{
    // the candidate's initial state was computed once per pose (k_corr_init)
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N * C.ck) return;
    const int k = (int)(q / N);
    const long long n = q - (long long)k * N;
    const int p = pose_of(pose, n, G.P);
    const float y[3] = {xq[n], xq[N + n], xq[2 * N + n]};
    const int cell = cell_index(C, bbox + p * 6, y);
    const float4 *ci = cinit + (((long long)p * C.ncell + cell) * C.ck + k) * 4;
    const float4 a = ci[0], b = ci[1], c = ci[2], d = ci[3];
    const float x0[3] = {a.x, a.y, a.z};
    const float Ji[9] = {b.w, c.x, c.y, c.z, c.w, d.x, d.y, d.z, d.w};
    write_init(q, N, k, n, x0, Ji, (__float_as_int(a.w) & 1) != 0, o_x0, o_J, o_v);
}

// ------------------------------------------------------------------------------------------------
// Correspondence grid build (voxel-based initialisation).
// ------------------------------------------------------------------------------------------------
// Bounding box of the images of all nodes of a pose, without atomics: k_precompute leaves the extent of every block's
// share, one wave per entry reduces the blocks' values (all lanes of the wave; the answer in every lane).  (With atomicMin / atomicMax on the 6
// words of a pose -- all in one cache line -- the atomics were the cost: about 3 ns each, 37 of 40 us on the 8-pose grid
// with 256 blocks per pose, 145 us with 1024.)
__device__ __forceinline__ unsigned reduce_extent(const unsigned *__restrict__ bb_part, int nblk, int p, int e, int first, int step)
{
    const unsigned *q = bb_part + ((long long)p * 6 + e) * nblk;
    const bool is_min = e < 3;
    unsigned r = is_min ? 0xffffffffu : 0u;
    for (int b = first; b < nblk; b += step) r = is_min ? min(r, q[b]) : max(r, q[b]);
#pragma unroll
    for (int sft = 32; sft >= 1; sft >>= 1) {
        const unsigned o = (unsigned)__shfl_xor((int)r, sft);
        r = is_min ? min(r, o) : max(r, o);
    }
    return r;
}

// one block per pose and entry; only for grids of more than EXTENT_OWN blocks
__global__ __launch_bounds__(1024) void k_corr_bbox(int nblk, const unsigned *__restrict__ bb_part, float *__restrict__ bbox)
{
    __shared__ unsigned s_part[16];
    const int p = blockIdx.x / 6, e = blockIdx.x - 6 * p;
    const unsigned r = reduce_extent(bb_part, nblk, p, e, threadIdx.x, 1024);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned t = s_part[0];
        for (int i = 1; i < 16; ++i) t = e < 3 ? min(t, s_part[i]) : max(t, s_part[i]);
        bbox[blockIdx.x] = ord2f(t);
    }
}

// The nodes by the cell of their image, as lists of chunks.  A block of 1024 threads takes a brick of nodes (8 x 8 x 16; images of
// neighbours are neighbours, a brick falls into a few dozen cells), counts per cell in an LDS hash table, and leaves the brick's nodes
// {image[3], node index} sorted by cell in the brick's own part of `sample`: a chunk per cell, {place, length}.  The first CHUNKS of a cell are
// entered in a table of the cell's, by one atomic on how many there are; the others make a list behind that, each put in front by an exchange.
// head[gc]: number of chunks, head[cells + gc]: place of the list's first + 1, or 0 (both cleared by k_precompute); link[place]: {place + 1 of the next
// or 0, length}.  Nothing is added up over blocks, so that no scan and no second pass over the nodes follows.  (Positions by an atomic per cell and
// brick, a scan, a kernel that moves the nodes, and lists that are read once per candidate: 21 us with k_corr_select on 65 k nodes and two launches
// more, 129 on the 8-pose grid; now 14 and 113.)
constexpr int CHUNKS = 8;
// own_box: the block reduces the extents itself (up to EXTENT_OWN blocks of k_precompute; block 0 of a pose keeps the box).
constexpr int EXTENT_OWN = 512;
constexpr int BRICK = 1024, HASH = 2 * BRICK;
__global__ __launch_bounds__(BRICK) void k_corr_chunks(GridP G, CorrP C, const float *__restrict__ Y, const unsigned *__restrict__ bb_part,
                                                       int nblk, bool own_box, float *__restrict__ bbox, int lz, int ly, int nby, int nbz,
                                                       int *__restrict__ head, int2 *__restrict__ table, int2 *__restrict__ link,
                                                       float4 *__restrict__ sample)
{
    __shared__ int s_key[HASH], s_cnt[HASH], s_tot[BRICK / 64];
    __shared__ float s_box[6];
    const int p = blockIdx.y, wib = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < HASH; i += BRICK) {
        s_key[i] = -1;
        s_cnt[i] = 0;
    }
    if (wib < 6) {
        const float r = own_box ? ord2f(reduce_extent(bb_part, nblk, p, wib, lane, 64)) : bbox[p * 6 + wib];
        if (lane == 0) {
            s_box[wib] = r;
            if (own_box && blockIdx.x == 0) bbox[p * 6 + wib] = r;
        }
    }
    __syncthreads();
    // brick of 2^lz nodes along z, 2^ly along y, the rest along x
    const int bz = (int)blockIdx.x % nbz, bt = (int)blockIdx.x / nbz, by = bt % nby, bx = bt / nby, t = (int)threadIdx.x;
    const int iz = (bz << lz) + (t & ((1 << lz) - 1)), iy = (by << ly) + ((t >> lz) & ((1 << ly) - 1));
    const int ix = bx * (BRICK >> (lz + ly)) + (t >> (lz + ly));
    const bool valid = ix < G.nx && iy < G.ny && iz < G.nz;
    const long long i = (long long)p * G.V + ((long long)ix * G.ny + iy) * G.nz + iz;
    int h = 0, rank = 0;
    float y[3] = {0.0f, 0.0f, 0.0f};
    if (valid) {
#pragma unroll
        for (int r = 0; r < 3; ++r) y[r] = Y[i * 3 + r];
        const int c = cell_index(C, s_box, y);
        // at most BRICK keys in a table of twice the size: the search ends
        h = (int)(((unsigned)c * 2654435761u) >> 21);
        static_assert(HASH == 1 << 11, "hash bits");
        while (true) {
            int k = __hip_atomic_load(&s_key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (k == -1) {
                k = atomicCAS(&s_key[h], -1, c);
                if (k == -1) k = c;
            }
            if (k == c) break;
            h = (h + 1) & (HASH - 1);
        }
        rank = atomicAdd(&s_cnt[h], 1);
    }
    __syncthreads();
    // counts -> where the chunks start, two entries per thread
    static_assert(HASH == 2 * BRICK, "entries per thread");
    const int e0 = 2 * (int)threadIdx.x, n0 = s_cnt[e0], n1 = s_cnt[e0 + 1];
    int inc = n0 + n1;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane == 63) s_tot[wib] = inc;
    __syncthreads();
    int at0 = inc - n0 - n1;
    for (int b = 0; b < wib; ++b) at0 += s_tot[b];
    const int base = (int)(blockIdx.y * gridDim.x + blockIdx.x) * BRICK;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int n = q == 0 ? n0 : n1, at = q == 0 ? at0 : at0 + n0;
        s_cnt[e0 + q] = at;
        if (n > 0) {
            const int gc = p * C.ncell + s_key[e0 + q], slot = atomicAdd(head + gc, 1);
            if (slot < CHUNKS) table[(long long)gc * CHUNKS + slot] = make_int2(base + at, n);
            else link[base + at] = make_int2(atomicExch(head + G.P * C.ncell + gc, base + at + 1), n);
        }
    }
    __syncthreads();
    if (valid) sample[base + s_cnt[h] + rank] = make_float4(y[0], y[1], y[2], __int_as_float((int)(i - (long long)p * G.V)));
}

// ---- prefix sums over blocks in one pass (decoupled look-back) ------------------------------------------------------
// Every block takes a ticket (its place in the order), publishes the sum of its part, and adds up what the blocks before
// it have published until it meets one that knows the sum of everything up to itself.  A block waits only for blocks with
// lower tickets, which are running already and publish their own sums before they wait for anything: every wait ends.
// look[0]: tickets given out; look[LOOK_HEAD + t]: {state, value} of ticket t.  All words are zero when the kernel starts: the
// kernel that follows it in the same call clears what it used (look_clear), so that nothing about a call is kept on the
// host and a captured graph replays.  (A count of finished blocks, whose last one clears, is a second atomic per block.)
// Tickets are atomics on one address, served one after the other, hence a few hundred blocks at most for all but the
// largest inputs.
typedef unsigned long long u64;
constexpr u64 LOOK_SUM = 1ull << 32, LOOK_PREFIX = 2ull << 32;
constexpr int LOOK_HEAD = 16;        // the ticket counter has a cache line of its own

__device__ __forceinline__ u64 look_load(u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void look_store(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// the block's ticket (all threads; one barrier)
__device__ __forceinline__ int look_ticket(u64 *__restrict__ look)
{
    __shared__ int s_ticket;
    if (threadIdx.x == 0) s_ticket = (int)atomicAdd(reinterpret_cast<unsigned *>(look), 1u);
    __syncthreads();
    return s_ticket;
}
// sum of the blocks before ticket t, whose own sum is `mine`; by one whole wave
__device__ __forceinline__ int look_back(u64 *__restrict__ look, int t, int mine, int lane)
{
    u64 *st = look + LOOK_HEAD;
    if (lane == 0) look_store(st + t, (t == 0 ? LOOK_PREFIX : LOOK_SUM) | (unsigned)mine);
    int before = 0;
    for (int at = t; at > 0; at -= 64) {          // lane l looks at ticket at - 1 - l
        const int i = at - 1 - lane;
        u64 w;
        unsigned long long prefix, unknown;
        int first;
        do {
            w = i >= 0 ? look_load(st + i) : LOOK_PREFIX;
            prefix = __ballot((w >> 32) == 2ull);
            unknown = __ballot((w >> 32) == 0ull);
            first = prefix ? __ffsll((long long)prefix) - 1 : 63;       // nearest block that knows everything up to itself
            if (unknown & ((2ull << first) - 1ull)) __builtin_amdgcn_s_sleep(1);
        } while (unknown & ((2ull << first) - 1ull));
        int v = lane <= first ? (int)(unsigned)w : 0;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
        before += v;
        if (prefix) break;
    }
    if (lane == 0 && t > 0) look_store(st + t, LOOK_PREFIX | (unsigned)(before + mine));
    return before;
}
// by a kernel that runs after: the words that one of `blocks` blocks used (0: none)
__device__ __forceinline__ void look_clear(u64 *__restrict__ look, int blocks)
{
    if (blocks == 0) return;
    const long long stride = (long long)gridDim.x * gridDim.y * blockDim.x;
    for (long long i = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; i < LOOK_HEAD + blocks; i += stride) look[i] = 0ull;
}
// By a whole wave of every block of a kernel that no other follows in its call, after its look_back: the last block clears the words.  done: one word,
// LOOK_HEAD before the ticket.
__device__ __forceinline__ void look_finish(u64 *__restrict__ look, int blocks, int lane)
{
    unsigned *done = reinterpret_cast<unsigned *>(look - LOOK_HEAD);
    int last = 0;
    if (lane == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this block's own words have been written
        last = (int)atomicAdd(done, 1u) == blocks - 1;
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    if (lane == 0) *done = 0u;
    for (int i = lane; i < LOOK_HEAD + blocks; i += 64) look[i] = 0ull;
}

// sums of the block's waves (up to 16 U of them per thread group) -> exclusive prefix within the block in s_tot[0 .. n),
// return value (first wave only): the block's sum
__device__ __forceinline__ int scan_totals(int *s_tot, int n, int lane)
{
    int run = 0;
    for (int b = 0; b < n; b += 64) {
        const int t = b + lane < n ? s_tot[b + lane] : 0;
        int inc = t;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(inc, d);
            if (lane >= d) inc += o;
        }
        if (b + lane < n) s_tot[b + lane] = run + inc - t;
        run += __shfl(inc, 63);
    }
    return run;
}

// Exclusive prefix sum of a[0..n) in place, a[n] = total; a 16-byte aligned.  PER (a multiple of 4) entries per
// thread, 1024 threads.  Bound: memory, and the launch.  (Tile sums and a second pass over the tiles, two launches: 21 us
// on 4.2 M entries, 9 us on 65 k; now 13 and 5.)
template <int PER>
__global__ __launch_bounds__(1024) void k_scan(int n, int *__restrict__ a, u64 *__restrict__ look)
{
    __shared__ int s_tot[16 * (PER / 4)], s_before;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int t = look_ticket(look);
    const long long base = (long long)t * (1024 * PER) + threadIdx.x * 4;
    int4 e[PER / 4];
    int sum[PER / 4], at[PER / 4];
#pragma unroll
    for (int b = 0; b < PER / 4; ++b) {
        const long long i = base + b * 4096;
        e[b] = make_int4(0, 0, 0, 0);
        if (i + 3 < n) e[b] = *reinterpret_cast<const int4 *>(a + i);
        else if (i < n) {
            e[b].x = a[i];
            if (i + 1 < n) e[b].y = a[i + 1];
            if (i + 2 < n) e[b].z = a[i + 2];
        }
        sum[b] = e[b].x + e[b].y + e[b].z + e[b].w;
        int inc = sum[b];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(inc, d);
            if (lane >= d) inc += o;
        }
        at[b] = inc - sum[b];
        if (lane == 63) s_tot[b * 16 + wid] = inc;
    }
    __syncthreads();
    if (wid == 0) {
        const int mine = scan_totals(s_tot, 16 * (PER / 4), lane);
        const int before = look_back(look, t, mine, lane);
        if (lane == 0) {
            s_before = before;
            if (t == (int)gridDim.x - 1) a[n] = before + mine;
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < PER / 4; ++b) {
        const long long i = base + b * 4096;
        int4 o;
        o.x = s_before + s_tot[b * 16 + wid] + at[b];
        o.y = o.x + e[b].x;
        o.z = o.y + e[b].y;
        o.w = o.z + e[b].z;
        if (i + 3 < n) *reinterpret_cast<int4 *>(a + i) = o;
        else if (i < n) {
            a[i] = o.x;
            if (i + 1 < n) a[i + 1] = o.y;
            if (i + 2 < n) a[i + 2] = o.z;
        }
    }
}

// smallest value of the 64 lanes; all lanes must call
__device__ __forceinline__ u64 wave_min(u64 v)
{
#define FS_MIN_STEP(ctrl, rows)                                                                                        \
    do {                                                                                                               \
        const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(-1, (int)(unsigned)v, (ctrl), (rows), 0xf, false);   \
        const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(-1, (int)(unsigned)(v >> 32), (ctrl), (rows), 0xf, false); \
        const u64 o = (u64)hi << 32 | lo;                                                                              \
        v = o < v ? o : v;                                                                                             \
    } while (0)
    FS_MIN_STEP(0x111, 0xf);            // row_shr 1, 2, 4, 8: within rows of 16 lanes
    FS_MIN_STEP(0x112, 0xf);
    FS_MIN_STEP(0x114, 0xf);
    FS_MIN_STEP(0x118, 0xf);
    FS_MIN_STEP(0x142, 0xa);            // row_bcast 15 into rows 1 and 3, row_bcast 31 into rows 2 and 3
    FS_MIN_STEP(0x143, 0xc);
#undef FS_MIN_STEP
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63), hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
    return (u64)hi << 32 | lo;
}

// One wave per cell.  Candidate j is the sample with the smallest (distance^2 of its image to the
// cell centre, node index) among those farther than r_sep (canonical distance) from candidates
// 0..j-1: the same set, in the same order, as visiting the samples by increasing key and accepting
// greedily.  The keys of a cell's first SELECT_MAX samples are held in registers: made once, and a sample that is too close to a
// candidate is out for good.  Those behind them are read once per candidate.
// Bound: latency (chunks -> samples) with few cells, instruction issue with many, so the places of the samples are written into LDS chunk by chunk
// (compared in registers with where each chunk starts: 95 us for 65,536 cells instead of 79; now, with crowded cells apart, 64), empty cells end at once, and the wave's minimum runs on DPP
// moves (with lane shuffles through the LDS 12 us more).  16 keys per lane instead of 8: 10 instead of 6.9 us for 8192 cells.
constexpr int SELECT_REGS = 8, SELECT_MAX = 64 * SELECT_REGS;
__global__ __launch_bounds__(256) void k_corr_select(GridP G, CorrP C, const float *__restrict__ bbox, const int *__restrict__ head,
                                                     const int2 *__restrict__ table, const int2 *__restrict__ link, const float4 *__restrict__ sample, int32_t *__restrict__ cand,
                                                     uint8_t *__restrict__ ccnt)
{
    // accepted candidates' positions, per wave: the same for all lanes and indexed by a loop counter -- in registers
    // that indexing turns into chains of selects, from LDS it is one broadcast read per candidate
    __shared__ float4 s_acc[4][FS_MAX_CORR_K_DEV];
    __shared__ int s_from[4][SELECT_MAX];
    const int lane = threadIdx.x & 63, wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int p = blockIdx.y, c = blockIdx.x * 4 + wib;
    if (c >= C.ncell) return;
    const long long gc = (long long)p * C.ncell + c;
    const float *bb = bbox + p * 6;
    const int chunks = __builtin_amdgcn_readfirstlane(head[gc]), rest = __builtin_amdgcn_readfirstlane(head[G.P * C.ncell + gc]);
    int2 entry = make_int2(0, 0);
    if (lane < CHUNKS) entry = table[gc * CHUNKS + lane];
    int32_t *out = cand + gc * C.ck;
    if (chunks == 0) {
        if (lane < C.ck) out[lane] = -1;
        if (lane == 0) ccnt[gc] = 0;
        return;
    }
    const int ciz = c % C.cz, ciy = (c / C.cz) % C.cy, cix = c / (C.cz * C.cy);
    const float cs0 = (bb[3] - bb[0]) / (float)C.cx;
    const float cs1 = (bb[4] - bb[1]) / (float)C.cy;
    const float cs2 = (bb[5] - bb[2]) / (float)C.cz;
    const float ctr[3] = {FS_FMA((float)cix + 0.5f, cs0, bb[0]), FS_FMA((float)ciy + 0.5f, cs1, bb[1]),
                          FS_FMA((float)ciz + 0.5f, cs2, bb[2])};
    const float rs2 = 6.25f * FS_FMA(G.h[2], G.h[2], FS_FMA(G.h[1], G.h[1], G.h[0] * G.h[0]));
    int na = 0;
    // {distance^2 (its bits order like the number, which is not negative), node}; a distance that is no number never wins
    auto key_of = [&](const float4 sm) {
        const float dx = sm.x - ctr[0], dy = sm.y - ctr[1], dz = sm.z - ctr[2];
        const float key = FS_FMA(dz, dz, FS_FMA(dy, dy, dx * dx));
        return key == key ? (u64)__float_as_uint(key) << 32 | (unsigned)__float_as_int(sm.w) : ~0ull;
    };
    auto apart = [&](const float (&x)[3], const float (&ac)[3]) {
        const float ex = x[0] - ac[0], ey = x[1] - ac[1], ez = x[2] - ac[2];
        return FS_FMA(ez, ez, FS_FMA(ey, ey, ex * ex)) > rs2;
    };
    // the chunks, until `on` wants no more
    auto walk = [&](auto on) {
        bool more = true;
        for (int i = 0; i < min(chunks, CHUNKS) && more; ++i)
            more = on(__builtin_amdgcn_readlane(entry.x, i), __builtin_amdgcn_readlane(entry.y, i));
        for (int at = rest; at != 0 && more;) {
            const int2 l = link[at - 1];
            more = on(at - 1, __builtin_amdgcn_readfirstlane(l.y));
            at = __builtin_amdgcn_readfirstlane(l.x);
        }
    };
    // the places of the cell's samples, one after the other
    int n = 0;
    walk([&](int place, int len) {
        if (n + len <= SELECT_MAX)
            for (int i = lane; i < len; i += WAVE) s_from[wib][n + i] = place + i;
        n += len;
        return n <= SELECT_MAX;
    });
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (n <= SELECT_MAX) {
        u64 key[SELECT_REGS];
#pragma unroll
        for (int r0 = 0; r0 < SELECT_REGS; r0 += 4) {
#pragma unroll
            for (int r = r0; r < r0 + 4; ++r) key[r] = ~0ull;
            if (r0 * 64 < n) {
                float4 sm[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if ((r0 + r) * 64 + lane < n) sm[r] = sample[s_from[wib][(r0 + r) * 64 + lane]];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if ((r0 + r) * 64 + lane < n) key[r0 + r] = key_of(sm[r]);
            }
        }
        for (int j = 0; j < C.ck; ++j) {
            u64 best = key[0];
#pragma unroll
            for (int r = 1; r < SELECT_REGS; ++r)
                if (r * 64 < n && key[r] < best) best = key[r];
            best = wave_min(best);
            if (best == ~0ull) break;     // wave-uniform
            ++na;
            if (lane == 0) out[j] = (int)(unsigned)best;
            if (na == C.ck) break;
            float ac[3];
            node_pos(G, (unsigned)best, ac);
#pragma unroll
            for (int r = 0; r < SELECT_REGS; ++r)
                if (r * 64 < n && key[r] != ~0ull) {
                    float x[3];
                    node_pos(G, (unsigned)key[r], x);
                    if (!apart(x, ac)) key[r] = ~0ull;
                }
        }
    } else {
        // Crowded cell: the first SELECT_MAX samples as above, those behind them, the chunks from number `from` on and of that one what lies behind `skip`, once per
        // candidate.  Bound: latency of the chain of chunks and samples.  (fs_precompute on 64x64x16 nodes, us, with everything read once per candidate, a sample per
        // lane at a time: 4x4x2 cells of 8 candidates 536, now 298; 16x16x4 cells 73, now 44; eight poses of 128x128x32 nodes, 8x8x8 cells of 3 467, now 324.)
        int from = 0, skip = 0;
        n = 0;
        walk([&](int place, int len) {
            skip = min(len, SELECT_MAX - n);
            for (int i = lane; i < skip; i += WAVE) s_from[wib][n + i] = place + i;
            n += skip;
            if (skip < len) return false;
            ++from;
            return true;
        });
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        u64 key[SELECT_REGS];
#pragma unroll
        for (int r = 0; r < SELECT_REGS; ++r) key[r] = key_of(sample[s_from[wib][r * 64 + lane]]);
        for (int j = 0; j < C.ck; ++j) {
            u64 best = key[0];
#pragma unroll
            for (int r = 1; r < SELECT_REGS; ++r)
                if (key[r] < best) best = key[r];
            int seen = 0;
            walk([&](int place, int len) {
                const int first = seen < from ? len : (seen == from ? skip : 0);
                ++seen;
                for (int s0 = first + lane; s0 < len; s0 += 4 * WAVE) {        // four samples on their way together
                    float4 q[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (s0 + u * WAVE < len) q[u] = sample[place + s0 + u * WAVE];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const u64 k = s0 + u * WAVE < len ? key_of(q[u]) : ~0ull;
                        if (k < best) {
                            float x[3];
                            node_pos(G, (unsigned)k, x);
                            bool far = true;
                            for (int a = 0; a < na; ++a) {
                                const float4 ac = s_acc[wib][a];
                                const float acc[3] = {ac.x, ac.y, ac.z};
                                if (!apart(x, acc)) far = false;
                            }
                            if (far) best = k;
                        }
                    }
                }
                return true;
            });
            best = wave_min(best);
            if (best == ~0ull) break;     // wave-uniform
            float xa[3];
            node_pos(G, (unsigned)best, xa);
            if (lane == 0) s_acc[wib][na] = make_float4(xa[0], xa[1], xa[2], 0.0f);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            ++na;
            if (lane == 0) out[j] = (int)(unsigned)best;
#pragma unroll
            for (int r = 0; r < SELECT_REGS; ++r)
                if (key[r] != ~0ull) {
                    float x[3];
                    node_pos(G, (unsigned)key[r], x);
                    if (!apart(x, xa)) key[r] = ~0ull;
                }
        }
    }
    if (lane == 0) {
        for (int j = na; j < C.ck; ++j) out[j] = -1;
        ccnt[gc] = (uint8_t)na;              // candidates of this cell (they are packed at the front)
    }
}

// Initial state of every candidate of the correspondence grid, once per fs_precompute instead of once per pair: a
// candidate is a grid node, so its x0, its image d(x0) and J~0 = (dd/dx at x0)^-1 depend on the pose alone, not on
// the query point.  Entry (4 float4) of candidate k of cell gc, at [(gc * ck + k) * 4]:
// {x0[3], flags | d(x0)[3], J~0[0] | J~0[1..4] | J~0[5..8]}, flags (integer bits) = 0: no such candidate,
// 1: usable, 2: Jacobian singular (J~0 = 0), plus the lower corner node of x0's grid cell << 2.
// Same arithmetic as a lane computing it for itself (node_pos, the 8 corner records of x0's cell,
// jacobian_from_corners, inv3).  (By the selecting wave's first lanes, which know the candidate: 136 instead of 30 registers
// there, 15.7 instead of 8.6 + 4.8 us for 8192 cells, 180 instead of 84 + 24 for 65,536.)
__global__ __launch_bounds__(256) void k_corr_init(GridP G, CorrP C, const float *__restrict__ T,
                                                   const int32_t *__restrict__ cand, float4 *__restrict__ cinit)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)G.P * C.ncell * C.ck) return;
    const int p = (int)(i / ((long long)C.ncell * C.ck));
    const int v = cand[i];
    float x0[3] = {0, 0, 0}, d[3] = {0, 0, 0}, Ji[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    int flags = 0;
    if (v >= 0) {
        node_pos(G, v, x0);
        const float *Tp = T + (long long)p * G.V * 12;
        const Cell c0 = locate(G, x0);
        float q[8][12], Jac[9];
#pragma unroll
        for (int c = 0; c < 8; ++c) load12(Tp + c0.base + corner_off(G, c), q[c]);
        jacobian_from_corners(G, c0, q, x0, d, Jac);
        const bool ok = inv3(Jac, Ji);
        if (!ok) {
#pragma unroll
            for (int e = 0; e < 9; ++e) Ji[e] = 0.0f;
        }
        flags = (ok ? 1 : 2) | (c0.base / 12 << 2);
    }
    float4 *o = cinit + i * 4;
    o[0] = make_float4(x0[0], x0[1], x0[2], __int_as_float(flags));
    o[1] = make_float4(d[0], d[1], d[2], Ji[0]);
    o[2] = make_float4(Ji[1], Ji[2], Ji[3], Ji[4]);
    o[3] = make_float4(Ji[5], Ji[6], Ji[7], Ji[8]);
}

// ------------------------------------------------------------------------------------------------
// Broyden solve.  Lanes are persistent: a wave draws chunks of consecutive lanes q = k*N + n from a
// global cursor and hands a new one to each SIMD lane that has finished, so that a wave does not
// idle behind its slowest trajectory and the grid drains only once, at the very end.  Every loop
// iteration evaluates the field once per active lane: for a freshly loaded lane at x0, otherwise
// at x + dx followed by the rank-one update of J~.
// ------------------------------------------------------------------------------------------------
struct SolveP {
    long long N;
    long long total;     // K * N
    int chunk;           // lanes drawn from the global cursor at a time
    int refill_min;      // refill when at least this many SIMD lanes are idle
    int max_iters;
    float tol2, div2;
    int K;
    int point_major;     // order in which pairs are handed out: 0 state by state, 1 (k_solve_ws) in tiles of points, 2 point by point
    int ki;              // kernels of small batches: initial states per wave (pair_of)
    int spin_limit;      // producer / consumer kernel: polls of a work queue before a wave gives up
    int xcd_ranges;      // producer / consumer kernel: the list is cut into 8 ranges, one per XCD, each with its own cursor
    int dealt;           // eighths of the chunks that are dealt out without the cursor (Chunks)
    int prefetch;        // producer / consumer kernel: consumers ask for the next cell's records at the end of a pass
    unsigned mag_N, mag_K;      // div_magic of N and K
    int per;             // k_solve_quad: pairs per wave, QUADS or HEXES
};

// What the fused variant needs to compute initial states itself (same arithmetic as k_init_*).
struct InitP {
    int mode;                 // 0: one state per bone (Eq. (8)); 1: candidates of the correspondence grid
    const float *Binv;        // [P][nb][12]
    const uint8_t *Bok;       // [P][nb]
    CorrP C;
    const float *bbox;        // [P][6]
    const int32_t *cand;      // [P][ncell][ck]
    const uint8_t *ccnt;      // [P][ncell]: number of candidates of the cell
    const float4 *cinit;      // [P][ncell][ck][4]: initial state of every candidate (k_corr_init)
};

// Result record of one pair.  WITH_J: 16 floats {x*[3], flags | pos, J~[0..2] | J~[3..6] | J~[7], J~[8], pad[2]}, else 4 floats
// {x*[3], flags}; flags = conv | iters << 8 (as an integer bit pattern).  `pos` (the lane's position in its grid cell's
// list, for the backward) is not written here but later, by flush_slots, for converged lanes only: this store leaves
// that word alone, so the two never write the same address.  x*, flags and pos share the record's first 32-byte sector.
template <bool WITH_J>
__device__ __forceinline__ void write_record(float4 *__restrict__ rec, long long pq, const float x[3], const float J[9],
                                             int flags)
{
    if (WITH_J) {
        float4 *o = rec + pq * 4;
        o[0] = make_float4(x[0], x[1], x[2], __int_as_float(flags));
        float *j = reinterpret_cast<float *>(o) + 5;
        j[0] = J[0];
        j[1] = J[1];
        j[2] = J[2];
        o[2] = make_float4(J[3], J[4], J[5], J[6]);
        o[3] = make_float4(J[7], J[8], 0.0f, 0.0f);
    } else {
        rec[pq] = make_float4(x[0], x[1], x[2], __int_as_float(flags));
    }
}
constexpr int REC_POS = 4;      // float index of `pos` inside a 16-float record

__device__ __forceinline__ void read_record_J(const float4 *__restrict__ r, float (&J)[9])
{
    const float4 b = r[1], c = r[2], d = r[3];
    J[0] = b.y; J[1] = b.z; J[2] = b.w; J[3] = c.x; J[4] = c.y; J[5] = c.z; J[6] = c.w; J[7] = d.x; J[8] = d.y;
}

// Words of the context's cursor array: CUR_ALL is the work cursor of the solve kernels; CUR_GRID: two words about the grid (GRID_NUMBER).
// CUR_XCD + j (j = 0 .. 7): the cursor of the j-th eighth of an ordered pair list, relative to the start of that eighth.
// CUR_LIST: length of the list of pairs that have a candidate (k_voxel_list).
// CUR_TOTAL, CUR_TOTAL + 1: converged lanes of the last solve that gave positions, and of the last backward from arrays (place_cells).
// The work cursors and CUR_LIST are zero between calls: the kernel that follows a solve kernel clears them (reset_cursors).  (A launch of its own before the solve
// kernel: 2 to 4 us.)
constexpr int CUR_ALL = 0, CUR_LIST = 1, CUR_GRID = 2, CUR_XCD = 4, CUR_TOTAL = 12, CUR_WORDS = 14;
__device__ __forceinline__ void reset_cursors(unsigned *__restrict__ cursor, int i)
{
    if (i == 0) cursor[CUR_ALL] = cursor[CUR_LIST] = 0u;
    if (i < N_XCD) cursor[CUR_XCD + i] = 0u;
}

// ---- where a grid cell's records lie in the list of the backward -------------------------------------------------------
// The counts of a solve's converged lanes (one per pose and grid cell) become places: every cell gets a stretch of the list.  The order of the stretches
// is free, so a block takes a tile of cells, adds its sum to the total with one atomic, and needs nothing from the other blocks.  Cells of a tile follow each
// other; place(c) is where cell c's stretch begins, place(c) + 1 holds its end, which is the next cell's begin or a word of the tile's own.
// The counts are zero between calls: they are cleared here, on the way.
// Bound: memory, 4 bytes read and 4 written per cell.  (Counts cleared by a launch before the solve, then an ordered scan in the backward:
// two launches, 2 to 4 and 4.5 us on 60 k cells.)
constexpr int CELL_TILE = 4096, CELL_STRIDE = CELL_TILE + 4;          // ends of tiles: a word, and three for alignment
__host__ __device__ inline long long cell_words(long long ncp) { return (ncp + CELL_TILE - 1) / CELL_TILE * CELL_STRIDE; }
__device__ __forceinline__ int place(int c) { return c + (int)((unsigned)c / CELL_TILE) * (CELL_STRIDE - CELL_TILE); }

// tile `t`, by a block of 256 threads
__device__ __forceinline__ void place_cells(int t, int ncp, int *__restrict__ counts, int *__restrict__ offset, unsigned *__restrict__ total)
{
    __shared__ int s_sum[16], s_base;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, c0 = t * CELL_TILE + (int)threadIdx.x * 4;
    int4 e[4];
    int at[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int c = c0 + b * 1024;
        e[b] = make_int4(0, 0, 0, 0);
        if (c + 3 < ncp) {
            e[b] = *reinterpret_cast<const int4 *>(counts + c);
        } else {
            if (c < ncp) e[b].x = counts[c];
            if (c + 1 < ncp) e[b].y = counts[c + 1];
            if (c + 2 < ncp) e[b].z = counts[c + 2];
        }
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int c = c0 + b * 1024, sum = e[b].x + e[b].y + e[b].z + e[b].w;
        if (sum != 0) {
            if (c + 3 < ncp) *reinterpret_cast<int4 *>(counts + c) = make_int4(0, 0, 0, 0);
            else
                for (int i = c; i < ncp; ++i) counts[i] = 0;
        }
        int inc = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(inc, d);
            if (lane >= d) inc += o;
        }
        at[b] = inc - sum;
        if (lane == 63) s_sum[b * 4 + wid] = inc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int v = s_sum[i];
            s_sum[i] = run;
            run += v;
        }
        s_base = (int)atomicAdd(total, (unsigned)run);
        offset[t * CELL_STRIDE + CELL_TILE] = s_base + run;
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        int4 o;
        o.x = s_base + s_sum[b * 4 + wid] + at[b];
        o.y = o.x + e[b].x;
        o.z = o.y + e[b].y;
        o.w = o.z + e[b].z;
        *reinterpret_cast<int4 *>(offset + t * CELL_STRIDE + (int)threadIdx.x * 4 + b * 1024) = o;
    }
}
__global__ __launch_bounds__(256) void k_place_cells(int ncp, int *__restrict__ counts, int *__restrict__ offset, unsigned *__restrict__ total)
{
    place_cells((int)blockIdx.x, ncp, counts, offset, total);
}

// Per pose the lower corner of the box of node images and the size of a correspondence cell (the arithmetic of cell_index)
// into LDS, by all threads of the block; corr_cell: pose * ncell + correspondence cell of a point.
// (With the six box entries and the three candidate slots read per point through the vector cache -- nine gathered loads
// of four bytes instead of one byte -- counting the candidates of the 8-pose batch took 77 instead of 43 us.)
__device__ __forceinline__ void corr_boxes(const GridP &G, const InitP &I, float *s_pose)
{
    for (int i = threadIdx.x; i < G.P * 3; i += blockDim.x) {
        const int p = i / 3, a = i - 3 * p;
        const float *bb = I.bbox + p * 6;
        const int na = a == 0 ? I.C.cx : (a == 1 ? I.C.cy : I.C.cz);
        s_pose[p * 6 + a] = bb[a];
        s_pose[p * 6 + 3 + a] = (bb[3 + a] - bb[a]) / (float)na;
    }
    __syncthreads();
}
__device__ __forceinline__ int corr_cell(const InitP &I, const float *s_pose, int p, const float y[3])
{
    const float *sp = s_pose + p * 6;
    return p * I.C.ncell + (cell_coord(y[0], sp[0], sp[3], I.C.cx) * I.C.cy + cell_coord(y[1], sp[1], sp[4], I.C.cy)) * I.C.cz +
           cell_coord(y[2], sp[2], sp[5], I.C.cz);
}

// Voxel-based initial states leave most lanes without a candidate (a ray sample in empty space has none): the list of the
// pairs that have one, {point n, (pose * ncell + correspondence cell) << 3 | k}, from which the solve draws.  A block takes 1024 U consecutive points, whose
// pairs follow each other.  ordered: so do the blocks' parts, in the order of the points; parts in the order in which blocks arrive would mix up to two million
// points, i.e. several poses' grids (Broyden kernel on the 8-pose batch 1447 instead of 1330 us).  Where an XCD's L2 holds all grids that does not
// matter (ordered = false): a block takes its part of the list with one atomic and waits for no other.
// Bound: the chain of tickets and memory (17 bytes read or written per point, 8 per pair).  (A counting pass, a scan of two launches,
// an expanding pass and a clearing pass: 28 us on 1 M ray samples, 42 us on 2 M, 85 us on the 8-pose batch; now 13, 24 and 62.)
template <int U>
__global__ __launch_bounds__(1024) void k_voxel_list(GridP G, InitP I, long long N, int K, const float *__restrict__ xq,
                                                     const int32_t *__restrict__ pose, uint8_t *__restrict__ cnt8,
                                                     int2 *__restrict__ list, unsigned *__restrict__ cursor,
                                                     u64 *__restrict__ look, bool ordered)
{
    extern __shared__ float s_pose[];            // [P][6]
    __shared__ int s_tot[16 * U], s_base;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, ticket = ordered ? look_ticket(look) : (int)blockIdx.x;
    const long long n0 = (long long)ticket * (1024 * U);
    float y[U][3];
    int p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const long long n = n0 + u * 1024 + threadIdx.x;
        p[u] = -1;
        y[u][0] = y[u][1] = y[u][2] = 0.0f;
        if (n < N) {
            p[u] = pose_of(pose, n, G.P);
#pragma unroll
            for (int r = 0; r < 3; ++r) y[u][r] = xq[r * N + n];
        }
    }
    corr_boxes(G, I, s_pose);
    int gc[U], m[U], at[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        gc[u] = m[u] = 0;
        if (p[u] >= 0) {
            gc[u] = corr_cell(I, s_pose, p[u], y[u]);
            m[u] = I.ccnt[gc[u]];
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (p[u] >= 0) cnt8[n0 + u * 1024 + threadIdx.x] = (uint8_t)m[u];
        int all = 0;
        at[u] = 0;
        for (int k = 0; k < K; ++k) {
            const unsigned long long b = __ballot(k < m[u]);
            at[u] += __popcll(b & ((1ull << lane) - 1ull));
            all += __popcll(b);
        }
        if (lane == 0) s_tot[u * 16 + wid] = all;
    }
    __syncthreads();
    if (wid == 0) {
        const int mine = scan_totals(s_tot, 16 * U, lane);
        const int before = ordered ? look_back(look, ticket, mine, lane) : 0;
        if (lane == 0) {
            s_base = ordered ? before : (int)atomicAdd(cursor + CUR_LIST, (unsigned)mine);
            if (ordered && ticket == (int)gridDim.x - 1) cursor[CUR_LIST] = (unsigned)(before + mine);
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int n = (int)(n0 + u * 1024 + threadIdx.x);
        const long long o = (long long)s_base + s_tot[u * 16 + wid] + at[u];
        for (int k = 0; k < m[u]; ++k)
            list[o + k] = make_int2(n, (gc[u] << 3) | k);
    }
}

// Candidates and cells of the points for a list that is to be ordered by place.
__global__ __launch_bounds__(256) void k_voxel_count(GridP G, InitP I, long long N, const float *__restrict__ xq,
                                                     const int32_t *__restrict__ pose, uint8_t *__restrict__ cnt8,
                                                     int *__restrict__ gcell)
{
    extern __shared__ float s_pose[];            // [P][6]
    corr_boxes(G, I, s_pose);
    const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    const float y[3] = {xq[n], xq[N + n], xq[2 * N + n]};
    const int gc = corr_cell(I, s_pose, pose_of(pose, n, G.P), y);
    cnt8[n] = I.ccnt[gc];
    gcell[n] = gc;
}

// The list of pairs, ordered by place: all pairs whose query point falls into the same column of correspondence cells
// (bucket = (pose * ncell + cell) / cz, i.e. the cell index without its fastest coordinate) are made neighbours, so
// that the lanes at work at any one time -- on every XCD, since all blocks draw from one cursor -- read the same
// stretch of one pose's transform grid and of the candidate table, and the caches serve what memory served before.
// A counting sort without global atomics: every block counts the candidates of its tile of SORT_TILE points per
// bucket in LDS and leaves the counts in hist[bucket][block]; an exclusive scan over that matrix (bucket-major)
// gives every (bucket, block) the place where its pairs start; the blocks then hand out places within that from LDS
// counters.  The order inside a bucket is the order in which the lanes of a block arrive: any order is a valid list.
constexpr int SORT_TILE = 16384;          // points per block
constexpr int SORT_MAX_BUCKETS = 16384;   // 64 KiB of LDS counters

__global__ __launch_bounds__(1024) void k_sort_hist(long long N, int cz, int nb, const int *__restrict__ gcell,
                                                    const uint8_t *__restrict__ cnt8, int *__restrict__ hist)
{
    extern __shared__ int s_cnt[];
    for (int i = threadIdx.x; i < nb; i += blockDim.x) s_cnt[i] = 0;
    __syncthreads();
    const long long n0 = (long long)blockIdx.x * SORT_TILE, n1 = min(N, n0 + SORT_TILE);
    for (long long n = n0 + threadIdx.x; n < n1; n += blockDim.x) {
        const int c = cnt8[n];
        if (c) atomicAdd(&s_cnt[gcell[n] / cz], c);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += blockDim.x) hist[(long long)i * gridDim.x + blockIdx.x] = s_cnt[i];
}

// list entry of a pair: {point n, (pose * ncell + correspondence cell) << 3 | k}
__global__ __launch_bounds__(1024) void k_sort_scatter(long long N, int cz, int nb, const int *__restrict__ gcell,
                                                       const uint8_t *__restrict__ cnt8, const int *__restrict__ start,
                                                       int2 *__restrict__ list, u64 *__restrict__ look, int look_blocks)
{
    look_clear(look, look_blocks);
    extern __shared__ int s_cnt[];
    for (int i = threadIdx.x; i < nb; i += blockDim.x) s_cnt[i] = start[(long long)i * gridDim.x + blockIdx.x];
    __syncthreads();
    const long long n0 = (long long)blockIdx.x * SORT_TILE, n1 = min(N, n0 + SORT_TILE);
    for (long long n = n0 + threadIdx.x; n < n1; n += blockDim.x) {
        const int c = cnt8[n];
        if (!c) continue;
        const int gc = gcell[n];
        const int at = atomicAdd(&s_cnt[gc / cz], c);
        for (int k = 0; k < c; ++k) list[at + k] = make_int2((int)n, (gc << 3) | k);
    }
}

// records -> caller's layout: one thread per pair q = k*N + n, consecutive threads consecutive n.
// NOCAND: the solve ran with fused voxel-based initial states and wrote no record for lanes whose
// cell holds no k-th candidate (cand_cnt[n] = candidates of point n, packed at the front);
// those get the answer of an invalid lane (x0 = 0, J~ = 0, not converged).
// o_slot (may be null): the positions of the converged lanes in their grid cells' lists, which the solve kernel
// left in the records, -1 for every other lane.
template <bool WITH_J, bool NOCAND>
__global__ __launch_bounds__(256) void k_solve_unpack(long long N, long long total, const uint8_t *__restrict__ cand_cnt,
                                                      const float4 *__restrict__ rec, float *__restrict__ o_x,
                                                      uint8_t *__restrict__ o_conv, float *__restrict__ o_J,
                                                      uint8_t *__restrict__ o_it, int32_t *__restrict__ o_slot,
                                                      u64 *__restrict__ look, int look_blocks, unsigned *__restrict__ cursor,
                                                      int rows, int tiles, int ncp, int *__restrict__ counts, int *__restrict__ offset)
{
    look_clear(look, look_blocks);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < N_XCD) reset_cursors(cursor, (int)threadIdx.x);
    // grid: points x initial states, behind `rows` rows of blocks that place the cells of the positions (place_cells; tiles = 0: none)
    if ((int)blockIdx.y < rows) {
        const int t = (int)(blockIdx.y * gridDim.x + blockIdx.x);
        if (t < tiles) place_cells(t, ncp, counts, offset, cursor + CUR_TOTAL);
        return;
    }
    const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x, k = (int)blockIdx.y - rows;
    if (n >= N) return;
    const long long pq = k * N + n;
    bool have = true;
    if (NOCAND) have = k < cand_cnt[n];
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
    if (have) a = WITH_J ? rec[pq * 4] : rec[pq];
    o_x[(k * 3 + 0) * N + n] = a.x;
    o_x[(k * 3 + 1) * N + n] = a.y;
    o_x[(k * 3 + 2) * N + n] = a.z;
    const int flags = __float_as_int(a.w);
    o_conv[pq] = (uint8_t)(flags & 1);
    if (o_it) o_it[pq] = (uint8_t)(flags >> 8);
    if (WITH_J && (o_slot || o_J) && have) b = rec[pq * 4 + 1];
    if (WITH_J && o_slot) o_slot[pq] = (flags & 1) ? __float_as_int(b.x) : -1;
    if (WITH_J && o_J) {
        float J[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        if (have) {
            const float4 c = rec[pq * 4 + 2], d = rec[pq * 4 + 3];
            J[0] = b.y; J[1] = b.z; J[2] = b.w; J[3] = c.x; J[4] = c.y; J[5] = c.z; J[6] = c.w; J[7] = d.x; J[8] = d.y;
        }
#pragma unroll
        for (int e = 0; e < 9; ++e) o_J[(k * 9 + e) * N + n] = J[e];
    }
}

// One position in its cell's list for every lane with `want` (wave-wide call; cell: pose * ncell + grid cell): the lanes of
// the wave that name the same cell are counted together and one of them adds the group to the cell's counter.  The
// answer is used by group_position(), so that several requests can be on their way before the first wait.
struct CellGroup {
    int leader, rank, base;
};
__device__ __forceinline__ CellGroup group_request(bool want, int cell, int lane, int *__restrict__ cell_count)
{
    CellGroup g;
    g.leader = lane;
    g.rank = 0;
    int members = 1;
    unsigned long long todo = __ballot(want);
    while (todo) {
        const int first = __ffsll((long long)todo) - 1;
        const int key = __builtin_amdgcn_readlane(cell, first);
        const unsigned long long same = __ballot(want && cell == key);
        if (want && cell == key) {
            g.leader = first;
            g.rank = __popcll(same & ((1ull << lane) - 1ull));
            members = __popcll(same);
        }
        todo &= ~same;
    }
    g.base = 0;
    if (want && g.leader == lane) g.base = atomicAdd(cell_count + cell, members);
    return g;
}
__device__ __forceinline__ int group_position(const CellGroup &g) { return __shfl(g.base, g.leader) + g.rank; }

// Chunks of work for one of the waves that draw them.  The first S.dealt eighths are dealt out in rounds, chunk w + i * drawers to
// drawer w; the cursor hands out the rest: it serves one drawer after the other, 9 ns each, and every drawer
// waits for its answer.
struct Chunks {
    long long round, shared, own;
};
__device__ __forceinline__ Chunks first_chunk(const SolveP &S, long long total, int drawer, int drawers, long long &next, long long &c1)
{
    Chunks c;
    c.round = (long long)drawers * S.chunk;
    c.shared = max(c.round, total / c.round * S.dealt / 8 * c.round);
    c.own = next = (long long)drawer * S.chunk;
    c1 = min(total, next + S.chunk);
    return c;
}
// false: there is none left (wave-wide call)
__device__ __forceinline__ bool next_chunk(Chunks &c, const SolveP &S, long long total, unsigned *__restrict__ cursor, int lane,
                                           long long &next, long long &c1)
{
    c.own += c.round;
    if (c.own < c.shared) {
        next = c.own;
    } else {
        unsigned b = 0;
        if (lane == 0) b = atomicAdd(cursor + CUR_ALL, (unsigned)S.chunk);
        next = c.shared + (long long)(unsigned)__builtin_amdgcn_readfirstlane((int)b);
        if (next >= total) {
            next = c1;
            return false;
        }
    }
    c1 = min(total, next + S.chunk);
    return true;
}

// The parked requests of one wave: entry i = {cell, pair}, one per SIMD lane.  Lanes of one point that reach
// the same root are neighbours in the wave and finish within a few passes of each other, so many entries name
// the same cell: those are counted together and one lane adds the group to the cell's counter.
constexpr int PEND = 128;       // requests a wave parks before it sends them
constexpr int PEND_SEND = 112;  // ... at least this many

__device__ __forceinline__ void flush_slots(int (&pend)[2][PEND], int npend, int lane, int *__restrict__ cell_count,
                                            float4 *__restrict__ rec)
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the LDS writes of the wave's other lanes
    __builtin_amdgcn_wave_barrier();
    // two rounds of 64 entries; the atomics of both are on their way before either answer is used
    bool valid[2];
    int pq[2];
    CellGroup g[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        valid[b] = 64 * b + lane < npend;
        const int c = valid[b] ? pend[0][64 * b + lane] : -1;
        pq[b] = valid[b] ? pend[1][64 * b + lane] : 0;
        g[b] = group_request(valid[b], c, lane, cell_count);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int at = group_position(g[b]);
        // into the pair's own result record (written a few passes ago, still in the L2), not into an array of its own
        if (valid[b]) reinterpret_cast<int *>(rec)[(long long)pq[b] * 16 + REC_POS] = at;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // before the entries are overwritten
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ void park_slots(bool want_slot, int slot_cell, int pair, int (&pend)[2][PEND], int &npend, int lane,
                                           int *__restrict__ cell_count, float4 *__restrict__ rec)
{
    const unsigned long long m = __ballot(want_slot);
    if (m) {
        if (npend + __popcll(m) > PEND) {
            flush_slots(pend, npend, lane, cell_count, rec);
            npend = 0;
        }
        if (want_slot) {
            const int at = npend + __popcll(m & ((1ull << lane) - 1ull));
            pend[0][at] = slot_cell;
            pend[1][at] = pair;
        }
        npend += __popcll(m);
    }
    if (npend >= PEND_SEND) {
        flush_slots(pend, npend, lane, cell_count, rec);
        npend = 0;
    }
}

// 1 / den for the lanes of the wave that are here
__device__ __forceinline__ float reciprocal(float den)
{
    float rinv = recip(den);
    if (__builtin_expect(__any(!is_normal(rinv)), 0)) {
        asm volatile("");                // a branch: the division is not to be computed in every step
        rinv = 1.0f / den;
    }
    return rinv;
}

// Rank-one update of J~ (good Broyden, inverse form) with u = dx - J~ dg, v = dx^T J~, den = v dg; none where den is 0 or not finite.
__device__ __forceinline__ void rank_one(float (&J)[9], const float (&u)[3], const float (&v)[3], float den)
{
    if (den != 0.0f && __builtin_fabsf(den) < __builtin_inff()) {
        const float rinv = reciprocal(den);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const float sc = u[r] * rinv;
#pragma unroll
            for (int c = 0; c < 3; ++c) J[r * 3 + c] = FS_FMA(sc, v[c], J[r * 3 + c]);
        }
    }
}

// the next step dx = -J~ g, and x moved by it
__device__ __forceinline__ void advance(const float (&J)[9], const float (&g)[3], float (&x)[3], float (&dx)[3])
{
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        dx[r] = -FS_FMA(J[r * 3 + 2], g[2], FS_FMA(J[r * 3 + 1], g[1], J[r * 3] * g[0]));
        x[r] = x[r] + dx[r];
    }
}

// What follows once the field's residual gn at the new x is known: the update of J~ and the test.  True: the pair has ended.
// A step begins with advance() rather than ending with it, so that x and J~ have one place each and the test has no branch: with the next
// step computed in a branch after the test, and loops that end at their head, the compiler copied the state to other registers and back
// in every pass (a pass of k_solve_once 311 vector instructions, now 233).
__device__ __forceinline__ bool finish_step(const SolveP &S, const float (&dx)[3], const float (&gn)[3], float (&g)[3], float (&J)[9],
                                            int &it, bool &conv)
{
    float dg[3], v[3], u[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) dg[r] = gn[r] - g[r];
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = FS_FMA(dx[2], J[6 + c], FS_FMA(dx[1], J[3 + c], dx[0] * J[c]));
#pragma unroll
    for (int r = 0; r < 3; ++r)
        u[r] = dx[r] - FS_FMA(J[r * 3 + 2], dg[2], FS_FMA(J[r * 3 + 1], dg[1], J[r * 3] * dg[0]));
    rank_one(J, u, v, FS_FMA(v[2], dg[2], FS_FMA(v[1], dg[1], v[0] * dg[0])));
    ++it;
#pragma unroll
    for (int r = 0; r < 3; ++r) g[r] = gn[r];
    const float r2 = FS_FMA(g[2], g[2], FS_FMA(g[1], g[1], g[0] * g[0]));
    conv = r2 < S.tol2;
    return conv || !(r2 < S.div2) || it >= S.max_iters;
}

// ---- four SIMD lanes per pair ---------------------------------------------------------------------------------------
// A pair whose trajectory is long is bound by the latency of a step: a chain of cell lookup, 8 corner records, blend,
// rank-one update.  With one lane per pair a step costs the wave some 320 vector instructions and 24 gathered loads
// whoever else is active.  Here the four lanes of a quad work on one pair: lane r = 0, 1, 2 looks up axis r, fetches row r
// of every corner record (8 loads of 16 bytes; the three lanes read 48 contiguous bytes) and blends that row, and
// computes what belongs to row r of the update (QuadState).  Lane 3 repeats lane 2.  The operations
// on every number, and their order, are those of one lane per pair, so the results are the same bits.
template <int R>
__device__ __forceinline__ float quad_get(float v)      // the value of lane R of the quad
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), R * 0x55, 0xf, 0xf, true));
}
template <int R>
__device__ __forceinline__ int quad_get(int v)
{
    return __builtin_amdgcn_mov_dpp(v, R * 0x55, 0xf, 0xf, true);
}
__device__ __forceinline__ float pick3(int row, float a, float b, float c) { return row == 0 ? a : (row == 1 ? b : c); }

// Chains of multiply-adds whose first factor comes from another lane.  The compiler gives a multiply that form and a multiply-add a
// move of its own, hence the assembly.  A DPP operand may be read two wait states after it was written: every block begins with those, and what
// a block returns is read by plain instructions or by another block.
#define FS_QUAD(n) " quad_perm:[" #n "," #n "," #n "," #n "] row_mask:0xf bank_mask:0xf\n\t"
#define FS_ROW(n) " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"
// fma(a of lane 2, b2, fma(a of lane 1, b1, a of lane 0 * b0)), lanes of the quad
__device__ __forceinline__ float quad_dot(float a, float b0, float b1, float b2)
{
    float o;
    asm("s_nop 1\n\t"
        "v_mul_f32_dpp %0, %1, %2" FS_QUAD(0)
        "v_fmac_f32_dpp %0, %1, %3" FS_QUAD(1)
        "v_fmac_f32_dpp %0, %1, %4" FS_QUAD(2)
        : "=&v"(o) : "v"(a), "v"(b0), "v"(b1), "v"(b2));
    return o;
}
// a[i] = fma(s of lane i, v, a[i]), lanes of the quad
__device__ __forceinline__ void quad_update(float s, float v, float (&a)[3])
{
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %3, %4" FS_QUAD(0)
        "v_fmac_f32_dpp %1, %3, %4" FS_QUAD(1)
        "v_fmac_f32_dpp %2, %3, %4" FS_QUAD(2)
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]) : "v"(s), "v"(v));
}
// a row of a transform applied to the point whose coordinates the quad's lanes hold: fma(T0, x0, fma(T1, x1, fma(T2, x2, T3)))
__device__ __forceinline__ float quad_map(const float (&T)[4], float x)
{
    float o = T[3];
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %4" FS_QUAD(2)
        "v_fmac_f32_dpp %0, %1, %3" FS_QUAD(1)
        "v_fmac_f32_dpp %0, %1, %2" FS_QUAD(0)
        : "+v"(o) : "v"(x), "v"(T[0]), "v"(T[1]), "v"(T[2]));
    return o;
}
// quad_dot of two numbers with the same factors
__device__ __forceinline__ void quad_dots(float a, float c, float b0, float b1, float b2, float &oa, float &oc)
{
    asm("s_nop 1\n\t"
        "v_mul_f32_dpp %0, %2, %4" FS_QUAD(0)
        "v_mul_f32_dpp %1, %3, %4" FS_QUAD(0)
        "v_fmac_f32_dpp %0, %2, %5" FS_QUAD(1)
        "v_fmac_f32_dpp %1, %3, %5" FS_QUAD(1)
        "v_fmac_f32_dpp %0, %2, %6" FS_QUAD(2)
        "v_fmac_f32_dpp %1, %3, %6" FS_QUAD(2)
        : "=&v"(oa), "=&v"(oc) : "v"(a), "v"(c), "v"(b0), "v"(b1), "v"(b2));
}
// fma(-a of lane 8, b2, fma(-a of lane 4, b1, -a of lane 0 * b0)), lanes of the row
__device__ __forceinline__ float row_dot_neg(float a, float b0, float b1, float b2)
{
    float o;
    asm volatile("s_nop 1\n\t"
        "v_mul_f32_dpp %0, -%1, %2" FS_ROW(0)
        "v_fmac_f32_dpp %0, -%1, %3" FS_ROW(4)
        "v_fmac_f32_dpp %0, -%1, %4" FS_ROW(8)
        : "=&v"(o) : "v"(a), "v"(b0), "v"(b1), "v"(b2));
    return o;
}
// the blend of corner_weights om (corner k in lane k of the row) and records q, one entry per lane, and the map of x by the blended
// row that the quad holds (blend_apply)
__device__ __forceinline__ float row_blend_apply(float om, const float (&q)[8], float x0, float x1, float x2)
{
    float e, d;
    asm volatile("s_nop 1\n\t"
        "v_mul_f32_dpp %0, %2, %3" FS_ROW(0)
        "v_fmac_f32_dpp %0, %2, %4" FS_ROW(1)
        "v_fmac_f32_dpp %0, %2, %5" FS_ROW(2)
        "v_fmac_f32_dpp %0, %2, %6" FS_ROW(3)
        "v_fmac_f32_dpp %0, %2, %7" FS_ROW(4)
        "v_fmac_f32_dpp %0, %2, %8" FS_ROW(5)
        "v_fmac_f32_dpp %0, %2, %9" FS_ROW(6)
        "v_fmac_f32_dpp %0, %2, %10" FS_ROW(7)
        "s_nop 1\n\t"
        "v_mov_b32_dpp %1, %0" FS_QUAD(3)
        "v_fmac_f32_dpp %1, %0, %13" FS_QUAD(2)
        "v_fmac_f32_dpp %1, %0, %12" FS_QUAD(1)
        "v_fmac_f32_dpp %1, %0, %11" FS_QUAD(0)
        : "=&v"(e), "=&v"(d)
        : "v"(om), "v"(q[0]), "v"(q[1]), "v"(q[2]), "v"(q[3]), "v"(q[4]), "v"(q[5]), "v"(q[6]), "v"(q[7]), "v"(x0), "v"(x1), "v"(x2));
    return d;
}
// a[i] = fma(s of lane 4i of the row, v, a[i])
__device__ __forceinline__ void row_update(float s, float v, float (&a)[3])
{
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %3, %4" FS_ROW(0)
        "v_fmac_f32_dpp %1, %3, %4" FS_ROW(4)
        "v_fmac_f32_dpp %2, %3, %4" FS_ROW(8)
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]) : "v"(s), "v"(v));
}
#undef FS_QUAD
#undef FS_ROW
// what a lane needs to look its axis up
struct QuadAxis {
    float lo, inv_h, m;
    int n, stride, row;
    float far_x, far_y;         // 1 where bit 0, 1 of the lane is clear, else 0: |far - f| is the weight of that side of an axis (quad_weights)
};
__device__ __forceinline__ QuadAxis quad_axis(const GridP &G, int row)
{
    QuadAxis A;
    A.row = row;
    A.lo = pick3(row, G.lo[0], G.lo[1], G.lo[2]);
    A.inv_h = pick3(row, G.inv_h[0], G.inv_h[1], G.inv_h[2]);
    A.m = pick3(row, G.m[0], G.m[1], G.m[2]);
    A.n = row == 0 ? G.nx : (row == 1 ? G.ny : G.nz);
    A.stride = row == 0 ? G.sx : (row == 1 ? G.sy : 12);
    A.far_x = (threadIdx.x & 1) ? 0.0f : 1.0f;
    A.far_y = (threadIdx.x & 2) ? 0.0f : 1.0f;
    return A;
}

// base of the cell of x, and the fraction along the lane's axis, from the coordinate along that axis
__device__ __forceinline__ int quad_place(const QuadAxis &A, float xr, float &f)
{
    int i0;
    bool cl;
    locate_axis(xr, A.lo, A.inv_h, A.m, A.n, i0, f, cl);
    const int b = i0 * A.stride;
    return quad_get<0>(b) + quad_get<1>(b) + quad_get<2>(b);
}
// corner_weights from the fractions that the quad's lanes hold: lane k the product of corner k's x and y weights.  Fractions lie in [0, 1], so
// |1 - f| and |0 - f| are the weights of an axis.
__device__ __forceinline__ void quad_weights(const QuadAxis &A, float f, float (&om)[8])
{
    const float wxy = __builtin_fabsf(A.far_x - quad_get<0>(f)) * __builtin_fabsf(A.far_y - quad_get<1>(f));
    const float z1 = quad_get<2>(f), z0 = 1.0f - z1;
    om[0] = quad_get<0>(wxy) * z0;
    om[1] = quad_get<1>(wxy) * z0;
    om[2] = quad_get<2>(wxy) * z0;
    om[3] = quad_get<3>(wxy) * z0;
    om[4] = quad_get<0>(wxy) * z1;
    om[5] = quad_get<1>(wxy) * z1;
    om[6] = quad_get<2>(wxy) * z1;
    om[7] = quad_get<3>(wxy) * z1;
}

// the lane's row of the 8 corner records
__device__ __forceinline__ void quad_load(const float *__restrict__ Tcell, const GridP &G, int row, float (&q)[8][4])
{
    const float *t = Tcell + row * 4;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int c = (i >> 1) + 4 * (i & 1);        // the two z-neighbours of an (x, y) corner one after the other
        const float4 v = *reinterpret_cast<const float4 *>(t + corner_off(G, c));
        q[c][0] = v.x; q[c][1] = v.y; q[c][2] = v.z; q[c][3] = v.w;
    }
}

// row r of the blended transform applied to x (blend_apply, one row)
__device__ __forceinline__ float quad_apply(const float (&T)[4], const float x[3])
{
    return FS_FMA(T[0], x[0], FS_FMA(T[1], x[1], FS_FMA(T[2], x[2], T[3])));
}
__device__ __forceinline__ void quad_blend(const float (&om)[8], const float (&q)[8][4], float (&T)[4])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) T[e] = om[0] * q[0][e];
#pragma unroll
    for (int k = 1; k < 8; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) T[e] = FS_FMA(om[k], q[k][e], T[e]);
}

// The state of a quad's pair: x along the lane's axis, g whole, the lane's row and column of J~.  What is one number per row (dx, u, v) is
// computed by its lane and fetched by the others; every number by the operations of finish_step.  (All of J~ and x in every lane:
// 145 vector instructions per step; with moves between lanes as instructions of their own 128; now 113.)
struct QuadState {
    float x, g[3], row[3], col[3];
};
__device__ __forceinline__ QuadState quad_state(int row, const float (&x)[3], const float (&g)[3], const float (&J)[9])
{
    QuadState q;
    q.x = pick3(row, x[0], x[1], x[2]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        q.g[c] = g[c];
        q.row[c] = pick3(row, J[c], J[3 + c], J[6 + c]);
        q.col[c] = pick3(row, J[3 * c], J[3 * c + 1], J[3 * c + 2]);
    }
    return q;
}
// the whole x and J~ in every lane
__device__ __forceinline__ void quad_unpack(const QuadState &q, float (&x)[3], float (&J)[9])
{
    x[0] = quad_get<0>(q.x);
    x[1] = quad_get<1>(q.x);
    x[2] = quad_get<2>(q.x);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        J[c] = quad_get<0>(q.row[c]);
        J[3 + c] = quad_get<1>(q.row[c]);
        J[6 + c] = quad_get<2>(q.row[c]);
    }
}

// One Broyden step of the pair of every active quad.  xpr: x' along the lane's axis, it: steps taken; q, held: the lane's row of the
// corner records and the base of the cell they belong to (-1: none).  True: the pair has ended.
__device__ __forceinline__ bool quad_step(const GridP &G, const SolveP &S, const QuadAxis &A, const float *__restrict__ Tp, float xpr,
                                          QuadState &s, int &it, float (&q)[8][4], int &held, bool &conv)
{
    const float dxr = -FS_FMA(s.row[2], s.g[2], FS_FMA(s.row[1], s.g[1], s.row[0] * s.g[0]));
    s.x = s.x + dxr;
    float f;
    const int base = quad_place(A, s.x, f);
    if (base != held) {
        quad_load(Tp + base, G, A.row, q);
        held = base;
    }
    const float vr = quad_dot(dxr, s.col[0], s.col[1], s.col[2]);
    float om[8], T[4];
    quad_weights(A, f, om);
    quad_blend(om, q, T);
    const float gr = quad_map(T, s.x) - xpr;
    const float gn[3] = {quad_get<0>(gr), quad_get<1>(gr), quad_get<2>(gr)};
    float dg[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) dg[r] = gn[r] - s.g[r];
    const float ur = dxr - FS_FMA(s.row[2], dg[2], FS_FMA(s.row[1], dg[1], s.row[0] * dg[0]));
    const float den = quad_dot(vr, dg[0], dg[1], dg[2]);
    if (den != 0.0f && __builtin_fabsf(den) < __builtin_inff()) {
        const float sc = ur * reciprocal(den);
        quad_update(vr, sc, s.row);
        quad_update(sc, vr, s.col);
    }
    ++it;
#pragma unroll
    for (int r = 0; r < 3; ++r) s.g[r] = gn[r];
    const float r2 = FS_FMA(gn[2], gn[2], FS_FMA(gn[1], gn[1], gn[0] * gn[0]));
    conv = r2 < S.tol2;
    return conv || !(r2 < S.div2) || it >= S.max_iters;
}

// ---- sixteen SIMD lanes per pair ------------------------------------------------------------------------------------
// The last pairs of a wave wait for one chain of instructions, each for the one before it: what a quad computes entry after entry is
// spread over a row of 16 lanes: 82 vector instructions and 8 loads of 4 bytes per step instead of a quad's 113 and 8 of 16 bytes.  (37 points of 24
// states, up to 50 steps: the call 37.7 -> 30.4 us; scans of 24 k points with candidates, most quads of a wave idle from the start, 57 -> 38; 8 k points of
// 24 states by k_solve_once, whose waves end this way, 75 -> 65.)  Lane 4r + c of a row holds entry (r, c) of the blended transform (8 loads of 4 bytes; a row
// reads the 48 bytes of a corner record) and of J~, and column c of J~; lane k the weight of corner k mod 8.  r = 3 repeats r = 2, and in J~ c = 3
// repeats c = 2.  Numbers move between lanes as DPP operands of the multiply-adds.  Operations and their order are those of finish_step.
template <int N>
__device__ __forceinline__ float row_get(float v)       // the value of lane N of the row
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + N, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ int row_get(int v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x150 + N, 0xf, 0xf, true);
}
constexpr int HEXES = 4;        // pairs a wave can hold this way

// Steps of the pairs of at most HEXES active quads until all have ended: a row of lanes takes each, and the quads get their pairs' ends back
// (s.x, s.row, it, conv).  Wave-wide call; xpr, s, it, pz: of the lane's quad (xpr, s.x and s.row: row A.row; s.col: its column).
__device__ __forceinline__ void hex_run(const GridP &G, const SolveP &S, const float *__restrict__ T, bool active, int lane, int quad_row,
                                        float xpr, QuadState &s, int &it, int pz, bool &conv)
{
    unsigned long long m = __ballot(active);
    if (m == 0) return;
    int src = 0, mine = 0;              // first lane of the quad this row takes from; the row that this lane's quad gave to
    bool on = false;
    for (int j = 0; m; ++j) {           // wave-uniform
        const int b = __ffsll((long long)m) - 1;
        m &= ~(0xfull << b);
        if ((lane >> 4) == j) {
            src = b;
            on = true;
        }
        if ((lane >> 2) == (b >> 2)) mine = 16 * j;
    }
    const int r4 = (lane >> 2) & 3, c4 = lane & 3;
    const QuadAxis A = quad_axis(G, min(r4, 2));
    const float *Te = T + (long long)__shfl(pz, src) * G.V * 12 + A.row * 4 + c4;
    const float hx = __shfl(xpr, src + r4);
    float x = __shfl(s.x, src + r4), g[3], col[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        g[c] = __shfl(s.g[c], src);
        col[c] = __shfl(s.col[c], src + c4);
    }
    float a = pick3(A.row, col[0], col[1], col[2]);         // J~ (r, c)
    int hit = __shfl(it, src);
    bool hconv = false;
    const float far_z = (lane & 4) ? 0.0f : 1.0f;
    if (on) {
        float q[8];
        int held = -1;
        bool done;
        do {
            const float t = quad_dot(a, g[0], g[1], g[2]);          // -dx
            x = x - t;
            int i0;
            float f;
            bool cl;
            locate_axis(x, A.lo, A.inv_h, A.m, A.n, i0, f, cl);
            const int b = i0 * A.stride, base = row_get<0>(b) + row_get<4>(b) + row_get<8>(b);
            if (base != held) {
                const float *c = Te + base;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int k = (i >> 1) + 4 * (i & 1);        // the two z-neighbours of an (x, y) corner one after the other
                    q[k] = c[corner_off(G, k)];
                }
                held = base;
            }
            const float om = (__builtin_fabsf(A.far_x - row_get<0>(f)) * __builtin_fabsf(A.far_y - row_get<4>(f))) * __builtin_fabsf(far_z - row_get<8>(f));
            const float x0 = row_get<0>(x), x1 = row_get<4>(x), x2 = row_get<8>(x);
            const float v = row_dot_neg(t, col[0], col[1], col[2]);
            const float gr = row_blend_apply(om, q, x0, x1, x2) - hx;
            const float gn[3] = {row_get<0>(gr), row_get<4>(gr), row_get<8>(gr)};
            const float dg[3] = {gn[0] - g[0], gn[1] - g[1], gn[2] - g[2]};
            float u, den;
            quad_dots(a, v, dg[0], dg[1], dg[2], u, den);
            u = -t - u;
            if (den != 0.0f && __builtin_fabsf(den) < __builtin_inff()) {
                const float sc = u * reciprocal(den);
                a = FS_FMA(sc, v, a);
                row_update(sc, v, col);
            }
            ++hit;
#pragma unroll
            for (int c = 0; c < 3; ++c) g[c] = gn[c];
            const float r2 = FS_FMA(g[2], g[2], FS_FMA(g[1], g[1], g[0] * g[0]));
            hconv = r2 < S.tol2;
            done = hconv || !(r2 < S.div2) || hit >= S.max_iters;
        } while (!done);
    }
    const int back = mine + 4 * quad_row;
    const float bx = __shfl(x, back), b0 = __shfl(a, back), b1 = __shfl(a, back + 1), b2 = __shfl(a, back + 2);
    const int bi = __shfl(hit << 1 | (hconv ? 1 : 0), mine);
    if (active) {
        s.x = bx;
        s.row[0] = b0;
        s.row[1] = b1;
        s.row[2] = b2;
        it = bi >> 1;
        conv = (bi & 1) != 0;
    }
}

// Steps of the pairs of the active quads until all have ended: in quads while more than HEXES are left, then in rows (wave-wide call)
__device__ __forceinline__ void quad_run(const GridP &G, const SolveP &S, const QuadAxis &A, const float *__restrict__ T, bool active, int lane,
                                         float xpr, QuadState &s, int &it, int pz, bool &conv)
{
    if (lanes_on(active) > 4 * HEXES) {
        const float *Tp = T + (long long)pz * G.V * 12;
        float q[8][4];
        int held = -1;
        do {
            if (active) active = !quad_step(G, S, A, Tp, xpr, s, it, q, held, conv);
        } while (lanes_on(active) > 4 * HEXES);
    }
    hex_run(G, S, T, active, lane, A.row, xpr, s, it, pz, conv);
}

// A wave whose last QUADS pairs (or fewer) are all that is left for it hands them from single lanes to quads: quad j
// takes the pair of the j-th active lane.  Returns the lane to take from, and whether the quad gets a pair.
constexpr int QUADS = 16;
__device__ __forceinline__ int quad_source(unsigned long long active, int lane, bool &gets)
{
    int src = 0;
    gets = false;
    for (int j = 0; active; ++j, active &= active - 1ull) {      // wave-uniform
        const int b = __ffsll((long long)active) - 1;
        if ((lane >> 2) == j) {
            src = b;
            gets = true;
        }
    }
    return src;
}

// Steps of the wave's last pairs (at most QUADS active lanes, none of them fresh) in quads until all have ended; then
// emit(ends, conv, x, J, it, n, k, p), one wave-wide call with `ends` in one lane of every quad that had a pair.
template <class Emit>
__device__ __forceinline__ void quad_tail(const GridP &G, const SolveP &S, const float *__restrict__ T, bool active, int lane,
                                          const float (&xp)[3], float (&x)[3], float (&g)[3], float (&J)[9], int it, int n, int k,
                                          int pz, Emit emit)
{
    const unsigned long long m = __ballot(active);
    if (m == 0) return;
    bool on;
    const int src = quad_source(m, lane, on);
    const QuadAxis A = quad_axis(G, min(lane & 3, 2));
    const float xpr = pick3(A.row, __shfl(xp[0], src), __shfl(xp[1], src), __shfl(xp[2], src));
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        x[r] = __shfl(x[r], src);
        g[r] = __shfl(g[r], src);
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) J[e] = __shfl(J[e], src);
    it = __shfl(it, src);
    n = __shfl(n, src);
    k = __shfl(k, src);
    pz = __shfl(pz, src);
    bool conv = false;
    QuadState state = quad_state(A.row, x, g, J);
    quad_run(G, S, A, T, on, lane, xpr, state, it, pz, conv);
    quad_unpack(state, x, J);
    emit(on && (lane & 3) == 0, conv, x, J, it, n, k, pz);
}

// Broyden solve for a transform grid (all poses) small enough to be held in LDS: every block copies it there
// first and all corner records are then read from LDS, where per-lane addresses cost far less than in the
// vector memory path.  Every wave does everything:
// FUSED = false: initial states are read from x0 / J0 / valid0.  FUSED = true: a lane computes its
// initial state when it picks up a pair (Sec. 3.1 "Custom CUDA Kernel": the kernel first computes the
// initialisation states); the corner records fetched for the Jacobian then also serve the first
// evaluation of the field, and the 53 bytes per pair of initial state never touch memory.
//
// Results leave the kernel as one contiguous record per pair (lanes finish at different times, so
// writing the caller's structure-of-arrays layout from here would touch 14 cache lines per pair with
// 4 bytes each); k_solve_unpack then moves the records into that layout with coalesced stores.
// (record layout: see write_record).
// NW = waves per block.  4: grids of up to 60 KiB, three blocks per CU, each with its own copy.  12: larger grids, up
// to what one block may hold of the CU's 160 KiB: one block per CU, the same 3 waves per SIMD, one copy.
template <bool FUSED, bool WITH_J, int NW = 4>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 3 : 1) void k_solve(GridP G, SolveP S, InitP I, const float *__restrict__ Tglobal,
                                               const float *__restrict__ xq, const int32_t *__restrict__ pose,
                                               const float *__restrict__ x0, const float *__restrict__ J0,
                                               const uint8_t *__restrict__ valid0, float4 *__restrict__ rec,
                                               unsigned *__restrict__ cursor, const int2 *__restrict__ list,
                                               const int *__restrict__ list_len, int *__restrict__ cell_count,
                                               int ncell)
{
    extern __shared__ float4 s_grid[];
    // converged lanes waiting for their position in their grid cell's list: {cell, pair} per wave
    __shared__ int s_pend[NW][2][PEND];
    {
        const int n4 = (int)((long long)G.P * G.V * 3);      // float4 per record: 3
        const float4 *src = reinterpret_cast<const float4 *>(Tglobal);
        for (int i = threadIdx.x; i < n4; i += blockDim.x) s_grid[i] = src[i];
        __syncthreads();
    }
    const float *T = reinterpret_cast<const float *>(s_grid);
    if (blockIdx.x == 0 && threadIdx.x == 0) cursor[CUR_TOTAL] = 0u;          // for place_cells, later in this call
    // with a list only the pairs list[0 .. *list_len) ({point, cell << 3 | k}) are solved
    const long long total = list ? (long long)*list_len : S.total;
    const int lane = threadIdx.x & 63;
    // wave-uniform: the wave's current chunk is [next, c1)
    long long next, c1;
    Chunks chunks = first_chunk(S, total, __builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6)), (int)gridDim.x * NW, next, c1);
    bool exhausted = false;          // wave-uniform: the global cursor has run past the end
    const long long N = S.N;

    bool active = false, fresh = false;
    long long n = 0;
    int k = 0, it = 0, pz = 0;
    const float *Tp = T;
    float xp[3] = {0, 0, 0}, x[3] = {0, 0, 0}, g[3] = {0, 0, 0};
    float J[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    float q[8][12];                  // corner records of the lane's current cell, kept across iterations
    long long held = -1;             // grid offset of the cell whose corners q holds (-1: none)
    int npend = 0;                   // wave-uniform: entries of s_pend in use
    const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));

    while (true) {
        unsigned long long idle = __ballot(!active);
        int nidle = __popcll(idle);
        // hand out pairs until fewer than refill_min lanes are idle: a pair whose initial state is
        // invalid is answered on the spot and its lane asks again
        while (!exhausted && nidle >= S.refill_min) {
            if (next >= c1) exhausted = !next_chunk(chunks, S, total, cursor, lane, next, c1);
            if (!exhausted) {
                const int rank = __popcll(idle & ((1ull << lane) - 1ull));
                const long long pq = next + rank;
                if (!active && pq < c1) {
                    // K * N < 2^31: 32-bit division
                    if (list) {
                        const int2 e = list[pq];
                        n = e.x;
                        k = e.y & 7;
                    } else if (S.point_major) {   // consecutive SIMD lanes: the K initial states of one point
                        n = (unsigned)pq / (unsigned)S.K;
                        k = (int)((unsigned)pq - (unsigned)n * (unsigned)S.K);
                    } else {                      // consecutive SIMD lanes: consecutive points, same initial state
                        k = (int)((unsigned)pq / (unsigned)N);
                        n = (unsigned)pq - (unsigned)k * (unsigned)N;
                    }
                    const int p = pose_of(pose, n, G.P);
                    pz = p;
                    Tp = T + (long long)p * G.V * 12;
                    it = 0;
                    held = -1;
                    bool ok, norec = false;     // norec: no record needed, k_solve_unpack knows the answer
#pragma unroll
                    for (int r = 0; r < 3; ++r) xp[r] = xq[r * N + n];
                    if (FUSED) {
#pragma unroll
                        for (int r = 0; r < 3; ++r) x[r] = 0.0f;
#pragma unroll
                        for (int e = 0; e < 9; ++e) J[e] = 0.0f;
                        if (I.mode == 0) {
                            const float *bi = I.Binv + ((long long)p * G.nb + k) * 12;
                            ok = I.Bok[p * G.nb + k] != 0;
                            if (ok) {
                                const float y[3] = {xp[0] - bi[9], xp[1] - bi[10], xp[2] - bi[11]};
#pragma unroll
                                for (int r = 0; r < 3; ++r)
                                    x[r] = FS_FMA(bi[r * 3 + 0], y[0], FS_FMA(bi[r * 3 + 1], y[1], bi[r * 3 + 2] * y[2]));
                            }
                        } else {
                            const int cidx = cell_index(I.C, I.bbox + p * 6, xp);
                            const int v = I.cand[((long long)p * I.C.ncell + cidx) * I.C.ck + k];
                            ok = v >= 0;
                            norec = !ok;
                            if (ok) node_pos(G, v, x);
                        }
                        if (ok) {
                            const Cell c0 = locate(G, x);
#pragma unroll
                            for (int c = 0; c < 8; ++c) load12(Tp + c0.base + corner_off(G, c), q[c]);
                            held = (long long)(Tp - T) + c0.base;
                            float d0[3], Jac[9];
                            jacobian_from_corners(G, c0, q, x, d0, Jac);
                            ok = inv3(Jac, J);
                            if (!ok) {
#pragma unroll
                                for (int e = 0; e < 9; ++e) J[e] = 0.0f;
                            }
                        }
                    } else {
#pragma unroll
                        for (int r = 0; r < 3; ++r) x[r] = x0[((long long)k * 3 + r) * N + n];
#pragma unroll
                        for (int e = 0; e < 9; ++e) J[e] = J0[((long long)k * 9 + e) * N + n];
                        ok = valid0[(long long)k * N + n] != 0;
                    }
                    if (ok) {
                        active = true;
                        fresh = true;
                    } else if (!norec) {
                        write_record<WITH_J>(rec, (long long)k * N + n, x, J, 0);
                    }
                }
                next += min((long long)nidle, c1 - next);
            }
            idle = __ballot(!active);
            nidle = __popcll(idle);
        }
        if (exhausted && 64 - nidle <= QUADS && !__any(active && fresh)) break;
        if (nidle == 64) continue;
        bool want_slot = false;
        int slot_cell = 0;
        if (active) {
            float dx[3], d[3], gn[3];
            if (!fresh) advance(J, g, x, dx);
            // steps shrink as a lane converges, so it often stays in the cell it was in: reload the
            // 8 corner records only when the cell changed
            const Cell cell = locate(G, x);
            const long long want = (long long)(Tp - T) + cell.base;
            if (want != held) {
#pragma unroll
                for (int c = 0; c < 8; ++c) load12(Tp + cell.base + corner_off(G, c), q[c]);
                held = want;
            }
            blend_apply(cell, q, x, d);
#pragma unroll
            for (int r = 0; r < 3; ++r) gn[r] = d[r] - xp[r];
            bool conv, ends;
            if (!fresh) ends = finish_step(S, dx, gn, g, J, it, conv);
            else {
                fresh = false;
#pragma unroll
                for (int r = 0; r < 3; ++r) g[r] = gn[r];
                const float r2 = FS_FMA(g[2], g[2], FS_FMA(g[1], g[1], g[0] * g[0]));
                conv = r2 < S.tol2;
                ends = conv || !(r2 < S.div2) || 0 >= S.max_iters;
            }
            if (ends) {
                write_record<WITH_J>(rec, (long long)k * N + n, x, J, (conv ? 1 : 0) | (it << 8));
                if (WITH_J && cell_count && conv) {
                    want_slot = true;
                    slot_cell = pz * ncell + cell_linear(G, cell);
                }
                active = false;
            }
        }
        // For the backward every converged lane needs its arrival position in the list of its grid cell: one
        // returning atomic on the cell's counter.  A wave would wait for that answer in every pass (a few of
        // its lanes finish in each), so the requests are parked in LDS and sent 112 or more at a time, one per cell and round of 64.
        if (WITH_J && cell_count) park_slots(want_slot, slot_cell, (int)((long long)k * N + n), s_pend[wib], npend, lane, cell_count, rec);
    }
    // the wave's last pairs, four lanes each
    quad_tail(G, S, T, active, lane, xp, x, g, J, it, (int)n, k, pz,
              [&](bool ends, bool conv, const float (&xe)[3], const float (&Je)[9], int ite, int ne, int ke, int pe) {
                  int cell = 0;
                  if (ends) {
                      write_record<WITH_J>(rec, (long long)ke * N + ne, xe, Je, (conv ? 1 : 0) | (ite << 8));
                      if (WITH_J && cell_count && conv) cell = pe * ncell + cell_linear(G, locate(G, xe));
                  }
                  if (WITH_J && cell_count)
                      park_slots(ends && conv, cell, (int)((long long)ke * N + ne), s_pend[wib], npend, lane, cell_count, rec);
              });
    if (WITH_J && cell_count && npend > 0) flush_slots(s_pend[wib], npend, lane, cell_count, rec);
}

// ------------------------------------------------------------------------------------------------
// Broyden solve (Eq. (7) with the rank-one update of J~, Algorithm 1 variant 2, per-iteration filter of
// Sec. 3.1 "Custom CUDA Kernel") with the work divided between the waves of a block.  One wave (the producer) prepares
// pairs 64 at a time, every SIMD lane busy: initial state, first evaluation of the field, first step; pairs
// that end there (invalid state, converged or diverged at x0) it answers itself.  The other waves (the
// consumers) iterate: idle lanes take prepared states {x', x, g, J~, pair} from the block's queue in LDS, and the loop
// holds nothing but the Broyden step.  Neither role ever holds the other's vector registers.
// Start and end cost what the middle does not show, so every wave works from the first to the last: a consumer prepares its first 64 pairs itself
// (its segment of the queue takes them from the one loop to the other), and the producer iterates when there is nothing left to prepare.
// The queue is one for the block, so that what is left when the producer ends goes to whoever has room.  (A queue of 128 per consumer, all filled by the
// producer: on 65 k points the consumers of a block had their first pairs after 5, 14 and 28 us, and the last of 277 us ended 75 after the producer.
// Whole fs_solve, us, that, and quads for a wave's last pairs / now: 0.29 M pairs of bone states 91 / 73, 0.48 M 108 / 97, 1.6 M 233 / 217, 4.8 M 591 / 576, with positions 699 / 706; candidates of
// 0.3 M ray samples 75 / 56, of 1 M 98 / 87, of 4.2 M points in eight poses 1118 / 1098, with positions 1317 / 1322; 8 candidates of 16x16x4 cells, 0.5 M points of scans 203 / 208, whose lanes have
// fewer neighbours in a wave.  A longer queue, 256 to 384 entries: within 1 %.)
// Entries are numbered as they come; one has its place modulo the queue's size.  tail: twice the entries written (by the producer), and one more when
// nothing will be added; claim: entries taken (by exchanges among the waves that iterate); freed: of each segment of 64, how many have been read since the
// start, the consumers' own pairs being the first round.  The producer writes into a segment when all of the round before has been read.
// Every wait ends: a producer that has polled S.spin_limit times in vain for room raises
// *give_up (host-visible) and prepares no more; it marks the tail as final in any case, and the waves, which wait for
// nothing else, finish what the queue holds and leave.
// ------------------------------------------------------------------------------------------------
constexpr int WS_SEGMENTS = 3, WS_RING = 64 * WS_SEGMENTS;     // one segment per consumer (16 KiB)
constexpr int FS_WS_CONSUMERS = 3;           // measured: a producer that computes Eq. (8) keeps up with three consumers, not with four
// A producer that only looks up voxel-based candidates could serve more consumers, but more iterating waves per CU
// only compete for the vector cache: measured on the multi-pose / training / ray batches, kernel ms with 2 blocks per
// CU: 3 consumers 1.73 / 0.175 / 0.120, 4 consumers 1.87 / 0.196 / 0.124, 5 consumers 1.92 / 0.213 / 0.138.
constexpr int FS_VX_CONSUMERS = 3;
constexpr int ST_XP = 0, ST_X = 3, ST_G = 6, ST_J = 9, ST_N = 18, ST_K = 19, ST_P = 20, ST_FIELDS = 21;

__device__ __forceinline__ int lds_load_acquire(const int *p)
{
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_store_release(int *p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---- result records of k_solve_ws leave through LDS ---------------------------------------------------------------
// A lane that finishes does not store its 64-byte record itself (four 16-byte stores to an address of its own: four
// vector-memory instructions in nearly every pass of the wave, each of which reaches memory as a partial write of a
// 32-byte sector).  The wave parks finished records in LDS, OUT_PEND per wave, together with the place of the
// converged ones; when OUT_PEND - 16 have gathered it asks for their positions in their cells' lists (one atomic per cell
// and round of 64, as flush_slots does), puts each position into its record, and writes the records out with four
// consecutive lanes per record: every record reaches memory once, whole, as 64 contiguous bytes.
// Without J~ a record is 16 bytes; those of eight neighbouring points in one state are one line.  (Stored by each lane as it finished: 200 k points
// of 24 states 705 us, now 682.)
template <int OUT_PEND, bool WITH_J>
struct OutQ {
    float4 rec[OUT_PEND][WITH_J ? 4 : 1];
    int place[WITH_J ? OUT_PEND : 1];      // where in the transform grids the cell of a converged lane that wants a position begins, else -1
    int pair[OUT_PEND];
};

// pose * ncell + grid cell, from where the cell's lower corner record lies in the grids of all poses (in floats)
__device__ __forceinline__ int cell_at(const GridP &G, int ncell, int place)
{
    const unsigned t = (unsigned)place / 12u, p = div_by(t, (unsigned)G.V, G.mag_V), v = t - p * (unsigned)G.V;
    const unsigned c = div_by(v, (unsigned)G.nz, G.mag_nz), ix = div_by(c, (unsigned)G.ny, G.mag_ny);       // c = ix * ny + iy
    return (int)(p * (unsigned)ncell + (c - ix) * (unsigned)(G.nz - 1) + v - c * (unsigned)G.nz);
}

template <int OUT_PEND, bool WITH_J>
__device__ __forceinline__ void out_flush(const GridP &G, OutQ<OUT_PEND, WITH_J> &q, int npend, int lane, int *__restrict__ cell_count, int ncell,
                                          float4 *__restrict__ rec)
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the LDS writes of the wave's other lanes
    __builtin_amdgcn_wave_barrier();
    if (WITH_J && cell_count) {
        // rounds of 64 entries; the atomics of all are on their way before an answer is used
        bool valid[OUT_PEND / 64];
        CellGroup g[OUT_PEND / 64];
#pragma unroll
        for (int b = 0; b < OUT_PEND / 64; ++b) {
            const int at = 64 * b + lane < npend ? q.place[64 * b + lane] : -1;
            valid[b] = at >= 0;
            const int c = valid[b] ? cell_at(G, ncell, at) : -1;
            g[b] = group_request(valid[b], c, lane, cell_count);
        }
#pragma unroll
        for (int b = 0; b < OUT_PEND / 64; ++b) {
            const int at = group_position(g[b]);
            if (valid[b]) reinterpret_cast<int *>(&q.rec[64 * b + lane][WITH_J ? 1 : 0])[0] = at;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    constexpr int Q = WITH_J ? 4 : 1;          // float4 per record
    for (int i = lane; i < npend * Q; i += 64) rec[(long long)q.pair[i / Q] * Q + i % Q] = q.rec[i / Q][i % Q];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // before the entries are overwritten
    __builtin_amdgcn_wave_barrier();
}

// park the record of every lane with `want` (wave-wide call); place < 0: no position wanted
template <int OUT_PEND, bool WITH_J>
__device__ __forceinline__ void out_park(const GridP &G, bool want, const float x[3], const float J[9], int flags, int place, int pair,
                                         OutQ<OUT_PEND, WITH_J> &q, int &npend, int lane, int *__restrict__ cell_count, int ncell, float4 *__restrict__ rec)
{
    const unsigned long long m = __ballot(want);
    if (m) {
        if (npend + __popcll(m) > OUT_PEND) {
            out_flush(G, q, npend, lane, cell_count, ncell, rec);
            npend = 0;
        }
        if (want) {
            const int at = npend + __popcll(m & ((1ull << lane) - 1ull));
            q.rec[at][0] = make_float4(x[0], x[1], x[2], __int_as_float(flags));
            q.pair[at] = pair;
            if constexpr (WITH_J) {
                q.rec[at][1] = make_float4(__int_as_float(-1), J[0], J[1], J[2]);
                q.rec[at][2] = make_float4(J[3], J[4], J[5], J[6]);
                q.rec[at][3] = make_float4(J[7], J[8], 0.0f, 0.0f);
                q.place[at] = place;
            }
        }
        npend += __popcll(m);
    }
    if (npend >= OUT_PEND - 16) {
        out_flush(G, q, npend, lane, cell_count, ncell, rec);
        npend = 0;
    }
}

// ---- corner records with zero weight need not be fetched ------------------------------------------------
// A coordinate outside the box is clamped, so its fraction is exactly 0 or 1 and the four corners on the far
// side of that axis get the weight 0: their records contribute 0 * T_c, i.e. nothing but possibly the sign of
// an exact zero.  A consumer of k_solve_ws may fetch only the other corners (bit c of the mask below); the
// registers of the skipped ones keep whatever finite record (or the initial zeros) they held before.  If a
// blended entry then comes out as an exact zero, the skipped records are fetched and the evaluation is
// repeated, so that even the sign of that zero is the one the full sum has (corners_needed).

// Issue order of the 24 loads of a cell.  The two z-neighbours of an (x, y) corner are 96 contiguous bytes, i.e. six
// 16-byte pieces in one or two cache lines; FS_LOAD_ORDER 1 issues the six pieces of a corner pair back to back
// (the compiler barrier keeps that order), 0 leaves the order to the compiler (four pieces of each pair, then the
// rest), 2 issues piece by piece across the four pairs (accesses of a lane to one line four instructions apart).
// Measured, Broyden kernel on the multi-pose / SMPL-scale batches: order 2: 2.20 / 0.42 ms, order 0: 1.69 / 0.35 ms:
// the vector cache rewards accesses to one line that follow each other closely.
#ifndef FS_LOAD_ORDER
#define FS_LOAD_ORDER 1
#endif
__device__ __forceinline__ void load_corners(const float *__restrict__ Tcell, const GridP &G, int mask, float (&q)[8][12])
{
#if FS_LOAD_ORDER == 0
#pragma unroll
    for (int c = 0; c < 8; ++c)
        if ((mask >> c) & 1) load12(Tcell + corner_off(G, c), q[c]);
#else
#pragma unroll
    for (int i = 0; i < 24; ++i) {
        const int j = FS_LOAD_ORDER == 1 ? i % 6 : i / 4, s4 = FS_LOAD_ORDER == 1 ? i / 6 : i % 4;
        const int c = s4 + 4 * (j / 3), e = 4 * (j % 3);
        if ((mask >> c) & 1) {
            const float4 v = *reinterpret_cast<const float4 *>(Tcell + corner_off(G, c) + e);
            q[c][e] = v.x; q[c][e + 1] = v.y; q[c][e + 2] = v.z; q[c][e + 3] = v.w;
        }
        if ((FS_LOAD_ORDER == 1 ? i % 6 == 5 : i % 4 == 3)) asm volatile("" ::: "memory");
    }
#endif
}

// all eight corner records of a cell
__device__ __forceinline__ void load_cell(const float *__restrict__ Tcell, const GridP &G, float (&q)[8][12])
{
    load_corners(Tcell, G, 0xFF, q);
}

// blend_apply that also tells whether one of the 12 blended entries is an exact zero
__device__ __forceinline__ bool blend_apply_z(const Cell &c, const float (&q)[8][12], const float x[3], float d[3])
{
    float om[8];
    corner_weights(c, om);
    float T[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) T[e] = om[0] * q[0][e];
#pragma unroll
    for (int k = 1; k < 8; ++k)
#pragma unroll
        for (int e = 0; e < 12; ++e) T[e] = FS_FMA(om[k], q[k][e], T[e]);
    apply12(T, x, d);
    float m = __builtin_fabsf(T[0]);
#pragma unroll
    for (int e = 1; e < 12; ++e) m = __builtin_fminf(m, __builtin_fabsf(T[e]));
    return m == 0.0f;
}

// One Broyden step of one pair per lane: the step, the field at the new x, the update of J~, the test.  q, held, held_mask: the corner records the
// lane holds, their cell's base inside the pose's grid (-1: none) and with SKIP which of them.  True: the pair has ended.
template <bool SKIP>
__device__ __forceinline__ bool lane_step(const GridP &G, const SolveP &S, const float *__restrict__ Tp, bool may_skip,
                                          const float (&xp)[3], float (&x)[3], float (&g)[3], float (&J)[9], int &it,
                                          float (&q)[8][12], int &held, int &held_mask, bool &conv)
{
    float dx[3], d[3], gn[3];
    advance(J, g, x, dx);
    // steps shrink as a lane converges, so it often stays in the cell it was in: the records are fetched again only when
    // the cell changed
    const Cell cell = locate(G, x);
    if (SKIP) {
        const int need = may_skip ? corners_needed(cell) : 0xFF;
        if (cell.base != held) {
            held = cell.base;
            held_mask = 0;
        }
        if (need & ~held_mask) {
            load_corners(Tp + cell.base, G, need & ~held_mask, q);
            held_mask |= need;
        }
        if (blend_apply_z(cell, q, x, d) && held_mask != 0xFF) {
            load_corners(Tp + cell.base, G, 0xFF & ~held_mask, q);
            held_mask = 0xFF;
            blend_apply(cell, q, x, d);
        }
    } else {
        if (cell.base != held) {
            load_cell(Tp + cell.base, G, q);
            held = cell.base;
        }
        blend_apply(cell, q, x, d);
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) gn[r] = d[r] - xp[r];
    return finish_step(S, dx, gn, g, J, it, conv);
}

// Pair number i of a batch that is handed out in tiles of TILE_PTS points, in a tile state after state: eight consecutive SIMD lanes
// are the same state of eight points, a batch of 64 eight states of them.  Neighbours in one state read and write consecutive addresses;
// states of one point often reach the same root and share its records and its atomic.  (Kernel us with all states of a point side by side / tiles of
// 8 / 16 / 64 points: 200 k points 711 / 684 / 687 / 685, 20 k points on 45x39x11 nodes 142 / 135 / 135 / 140, 65 k points with positions
// 313 / 313 / 317 / 339.)
// Quotients by div_by: the reciprocals that a division in plain C makes of S.K, S.N and the tile's size stay in vector registers
// through the producer's loop, and with one state per bone three of them were spilled.
constexpr unsigned TILE_PTS = 8;
__device__ __forceinline__ void tile_pair(const SolveP &S, unsigned i, int &n, int &k)
{
    const unsigned N = (unsigned)S.N, K = (unsigned)S.K;
    const unsigned t = div_by(i, K, S.mag_K) / TILE_PTS, r = i - t * (TILE_PTS * K), pts = min(TILE_PTS, N - t * TILE_PTS);     // the last tile may be short
    const unsigned kk = pts == TILE_PTS ? r / TILE_PTS : r / pts;
    k = (int)kk;
    n = (int)(t * TILE_PTS + r - kk * pts);
}

template <bool FUSED, bool WITH_J, int NCONS, bool SKIP>
__global__ __launch_bounds__(64 * (NCONS + 1), SKIP ? 3 : 2) void k_solve_ws(GridP G, SolveP S, InitP I, const float *__restrict__ T,
                                               const float *__restrict__ xq, const int32_t *__restrict__ pose,
                                               const float *__restrict__ x0, const float *__restrict__ J0,
                                               const uint8_t *__restrict__ valid0, float4 *__restrict__ rec,
                                               unsigned *__restrict__ cursor, const int2 *__restrict__ list,
                                               const int *__restrict__ list_len, int *__restrict__ cell_count,
                                               int ncell, int *__restrict__ give_up,
                                               const int *__restrict__ state)
{
    __shared__ float s_ring[ST_FIELDS][WS_RING];
    __shared__ int s_tail, s_claim, s_freed[WS_SEGMENTS];
    // One state per bone: 64 and 128 take the same time (fs_solve with positions, us, 64 / 128: 20 k points 111 / 112, 65 k 257 / 254, 200 k 706 / 700; 24 MB 137 / 137, 324 / 321, 895 / 884), in 34
    // instead of 52 KiB of LDS
    constexpr int OUT_PEND = SKIP ? 64 : 128;
    __shared__ OutQ<OUT_PEND, WITH_J> s_out[NCONS + 1];      // records on their way out, per wave
    if (threadIdx.x < WS_SEGMENTS) s_freed[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        s_claim = WS_RING;
        s_tail = 2 * WS_RING;
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) cursor[CUR_TOTAL] = 0u;          // for place_cells, later in this call
    const long long total = list ? (long long)*list_len : S.total;
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long N = S.N;
    int npend = 0;                   // wave-uniform: entries of the wave's s_out in use
    OutQ<OUT_PEND, WITH_J> &outq = s_out[wib];
    const int stride = (int)G.V * 12;          // of the poses' grids; P of them are below 2^31

    const bool producer = wib == NCONS;
    static_assert(NCONS == WS_SEGMENTS, "a consumer's own pairs fill a segment of the queue");
    int tail = producer ? WS_RING : 64 * wib;        // entries written
    int nown = 0;                   // of a consumer: pairs it has put into its segment itself
    // SKIP needs a grid of entries below SKIP_MAX (k_precompute says if this one is not)
    const bool may_skip = SKIP && may_skip_corners(state);
    {
        // ------------------------------------------- preparing pairs -------------------------------------------
        // every consumer of the grid takes `own` consecutive pairs from the front; the producers' chunks are those behind
        const bool ranges = S.xcd_ranges != 0;
        const unsigned consumers = gridDim.x * NCONS;
        const unsigned own = ranges ? 0u : ((unsigned)total >= 64u * consumers ? 64u : ((unsigned)total + consumers - 1u) / consumers);
        const long long heads = min(total, (long long)own * consumers), rest = total - heads;
        // the first chunk of block b is chunk b; the shared cursor counts what lies behind those.  (One cursor for the whole chip
        // on purpose: all XCDs then work through the same stretch of the points at the same time, and what one of them
        // brought into the memory-side cache serves the others.  With a cursor per XCD over its own eighth of the
        // points -- one pose per XCD on the multi-pose batch -- the kernel was 13 % slower: eight transform grids
        // instead of one compete for that cache.)
        //
        // On request the list, ordered by place, is cut into 8 ranges, one per XCD (blocks go to the XCDs in turn, so
        // block b runs on XCD b mod 8); a block whose range is used up takes chunks from the next ranges in turn.  The
        // XCD's own L2 then serves 0.72 instead of 0.47 of the requests and a third of the bytes come from beyond it,
        // but the kernel is no faster (1.29 against 1.26 ms with the ordered list behind one cursor): the vector cache
        // in front of the L2 is the limit.
        const int home = (int)(blockIdx.x & (N_XCD - 1));
        const long long per = ((total + (long long)N_XCD * S.chunk - 1) / ((long long)N_XCD * S.chunk)) * S.chunk;
        long long next, c1;             // of a producer: counted from the end of the consumers' own
        Chunks chunks = first_chunk(S, rest, (int)blockIdx.x, (int)gridDim.x, next, c1);
        if (!producer) {
            next = min(heads, (long long)(blockIdx.x * NCONS + wib) * own);
            c1 = min(heads, next + own);
        } else if (ranges) {
            const long long r1 = min(total, (home + 1) * per);
            next = home * per + (long long)(blockIdx.x >> 3) * S.chunk;
            c1 = min(r1, next + S.chunk);
        }
        int alive = 0;                    // ranges home, home + 1, ... home + alive - 1 are known to be used up
        bool lost = false;
        while (!lost) {
            if (next >= c1) {
                if (!producer) break;
                if (ranges) {
                    bool got = false;
                    while (alive < N_XCD) {
                        const int j = (home + alive) & (N_XCD - 1);
                        unsigned b = 0;
                        if (lane == 0) b = atomicAdd(cursor + CUR_XCD + j, (unsigned)S.chunk);
                        // the blocks of this range own its first chunks
                        b = (unsigned)__builtin_amdgcn_readfirstlane((int)b) + ((gridDim.x + (N_XCD - 1) - (unsigned)j) / N_XCD) * (unsigned)S.chunk;
                        const long long r1 = min(total, (j + 1) * per), at = j * per + (long long)b;
                        if ((long long)b < per && at < r1) {
                            next = at;
                            c1 = min(r1, at + S.chunk);
                            got = true;
                            break;
                        }
                        ++alive;
                    }
                    if (!got) break;
                } else {
                    if (!next_chunk(chunks, S, rest, cursor, lane, next, c1)) break;
                }
            }
            const bool mine = next + lane < c1;
            const long long pq = (producer ? heads : 0ll) + next + lane;
            next += min(64ll, c1 - next);
            bool keep = false, want_out = false;
            int out_place = -1, out_flags = 0, pair = 0;
            int nn = 0, nk = 0, np = 0;
            float nxp[3] = {0, 0, 0}, nx[3] = {0, 0, 0}, ng[3] = {0, 0, 0};
            float nJ[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            if (mine) {
                const unsigned upq = (unsigned)pq;        // K * N < 2^31
                int gcell = -1;                           // pose * ncell + correspondence cell, when the list gives it
                if (list) {
                    const int2 e = list[pq];
                    nn = e.x;
                    nk = e.y & 7;
                    gcell = e.y >> 3;
                } else if (S.point_major == 1) {
                    tile_pair(S, upq, nn, nk);
                } else if (S.point_major) {   // consecutive SIMD lanes: the K initial states of one point
                    nn = (int)div_by(upq, (unsigned)S.K, S.mag_K);
                    nk = (int)(upq - (unsigned)nn * (unsigned)S.K);
                } else {                      // consecutive SIMD lanes: consecutive points, same initial state
                    nk = (int)div_by(upq, (unsigned)N, S.mag_N);
                    nn = (int)(upq - (unsigned)nk * (unsigned)N);
                }
                np = pose_of(pose, nn, G.P);
                pair = (int)((long long)nk * N + nn);
                const float *Tn = T + (long long)np * G.V * 12;
                bool ok, norec = false;     // norec: no record needed, k_solve_unpack knows the answer
                float d[3] = {0, 0, 0};
                int base0 = 0;              // of the initial state's cell
#pragma unroll
                for (int r = 0; r < 3; ++r) nxp[r] = xq[r * N + nn];
                if (FUSED && SKIP) {
                    // one state per bone, Eq. (8)
                    const float *bi = I.Binv + ((long long)np * G.nb + nk) * 12;
                    ok = I.Bok[np * G.nb + nk] != 0;
                    if (ok) {
                        const float y[3] = {nxp[0] - bi[9], nxp[1] - bi[10], nxp[2] - bi[11]};
#pragma unroll
                        for (int r = 0; r < 3; ++r)
                            nx[r] = FS_FMA(bi[r * 3 + 0], y[0], FS_FMA(bi[r * 3 + 1], y[1], bi[r * 3 + 2] * y[2]));
                        const Cell c0 = locate(G, nx);
                        base0 = c0.base;
                        float Jac[9];
                        field_dJ_clamped(Tn, G, c0, may_skip, nx, d, Jac);
                        ok = inv3(Jac, nJ);
                        if (!ok) {
#pragma unroll
                            for (int e = 0; e < 9; ++e) nJ[e] = 0.0f;
                        }
                    }
                } else if (FUSED) {
                    // voxel-based candidates: x0, d(x0) and J~0 of a candidate do not depend on the query point and
                    // were computed once per pose (k_corr_init); a lane only looks its candidate up
                    if (gcell < 0) gcell = np * I.C.ncell + cell_index(I.C, I.bbox + np * 6, nxp);
                    const float4 *ci = I.cinit + ((long long)gcell * I.C.ck + nk) * 4;
                    const float4 a = ci[0], b = ci[1], c = ci[2], e = ci[3];
                    const int fl = __float_as_int(a.w);
                    ok = (fl & 1) != 0;
                    norec = (fl & 3) == 0;
                    base0 = (fl >> 2) * 12;
                    nx[0] = a.x; nx[1] = a.y; nx[2] = a.z;
                    d[0] = b.x; d[1] = b.y; d[2] = b.z;
                    nJ[0] = b.w; nJ[1] = c.x; nJ[2] = c.y; nJ[3] = c.z; nJ[4] = c.w;
                    nJ[5] = e.x; nJ[6] = e.y; nJ[7] = e.z; nJ[8] = e.w;
                } else {
#pragma unroll
                    for (int r = 0; r < 3; ++r) nx[r] = x0[((long long)nk * 3 + r) * N + nn];
#pragma unroll
                    for (int e = 0; e < 9; ++e) nJ[e] = J0[((long long)nk * 9 + e) * N + nn];
                    ok = valid0[(long long)nk * N + nn] != 0;
                    if (ok) {
                        const Cell c0 = locate(G, nx);
                        base0 = c0.base;
                        float qn[8][12];
#pragma unroll
                        for (int c = 0; c < 8; ++c) load12(Tn + c0.base + corner_off(G, c), qn[c]);
                        blend_apply(c0, qn, nx, d);
                    }
                }
                if (ok) {
#pragma unroll
                    for (int r = 0; r < 3; ++r) ng[r] = d[r] - nxp[r];
                    const float r2 = FS_FMA(ng[2], ng[2], FS_FMA(ng[1], ng[1], ng[0] * ng[0]));
                    const bool conv = r2 < S.tol2;
                    if (conv || !(r2 < S.div2) || 0 >= S.max_iters) {
                        want_out = true;
                        out_flags = conv ? 1 : 0;
                        if (cell_count && conv) out_place = np * stride + base0;
                    } else {
                        keep = true;
                    }
                }
                if (!ok && !norec) want_out = true;         // out_flags = 0, no position
            }
            const unsigned long long km = __ballot(keep);
            const int nkeep = __popcll(km);
            if (nkeep > 0) {
                // wait for room, which a consumer's segment has
                const int seg = (tail + nkeep - 1) / 64, lap = producer ? seg / WS_SEGMENTS : 0;
                int spins = 0;
                while (__builtin_amdgcn_readfirstlane(lds_load_acquire(&s_freed[seg - lap * WS_SEGMENTS])) < 64 * lap) {
                    if (++spins > S.spin_limit) { lost = true; break; }
                    __builtin_amdgcn_s_sleep(8);
                }
                if (lost) break;
                // Where pairs end after few steps the others wait for the producer: its wave goes first on its SIMD while less than a batch is left to claim
                // (not in the first round, while the others still prepare pairs themselves).  All equal / so, whole calls, us: 0.8 M points of 5 states 472 / 414,
                // 0.2 M of 8 196 / 182, of 24 577 / 576; 1 M ray samples 87 / 87.  From the first batch on: 0.3 M points of scans with candidates 60 / 63.
                if (lap >= 2) {
                    if (tail - __builtin_amdgcn_readfirstlane(__hip_atomic_load(&s_claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < 64) __builtin_amdgcn_s_setprio(3);
                    else __builtin_amdgcn_s_setprio(0);
                }
                if (keep) {
                    const int at = (int)((unsigned)(tail + __popcll(km & ((1ull << lane) - 1ull))) % WS_RING);
#pragma unroll
                    for (int r = 0; r < 3; ++r) {
                        s_ring[ST_XP + r][at] = nxp[r];
                        s_ring[ST_X + r][at] = nx[r];
                        s_ring[ST_G + r][at] = ng[r];
                    }
#pragma unroll
                    for (int e = 0; e < 9; ++e) s_ring[ST_J + e][at] = nJ[e];
                    s_ring[ST_N][at] = __int_as_float(nn);
                    s_ring[ST_K][at] = __int_as_float(nk);
                    s_ring[ST_P][at] = __int_as_float(np);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_wave_barrier();
                tail += nkeep;
                if (producer && lane == 0) lds_store_release(&s_tail, 2 * tail);
            }
            out_park(G, want_out, nx, nJ, out_flags, out_place, pair, outq, npend, lane, cell_count, ncell, rec);
            if (!producer) {
                nown = nkeep;
                break;
            }
        }
        if (producer) {
            __builtin_amdgcn_s_setprio(0);
            if (lost && lane == 0) *give_up = 1;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if (lane == 0) lds_store_release(&s_tail, 2 * tail + 1);
        }
    }

    // ---------------------------------------------------- iterating ----------------------------------------------------
    // the consumers from the beginning, the producer when there is nothing left to prepare
    // what becomes of a pair that has ended in a quad (wave-wide call; `ends` in one lane of the quad)
    auto emit = [&](bool ends, bool conv, const float (&xe)[3], const float (&Je)[9], int ite, int ne, int ke, int pe) {
        const int flags = (conv ? 1 : 0) | (ite << 8), pair = (int)((long long)ke * N + ne);
        int place = -1;
        if (WITH_J && ends && cell_count && conv) place = pe * stride + locate(G, xe).base;
        out_park(G, ends, xe, Je, flags, place, pair, outq, npend, lane, cell_count, ncell, rec);
    };
    bool active = false;
    int n = 0, k = 0, it = 0, pz = 0;
    const float *Tp = T;
    float xp[3] = {0, 0, 0}, x[3] = {0, 0, 0}, g[3] = {0, 0, 0};
    float J[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    float q[8][12];                  // corner records of the lane's current cell, kept across iterations
    int held = -1;                   // base of the cell whose corners q holds (-1: none)
    int held_mask = 0;               // SKIP: which of them
    if (SKIP) {
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int e = 0; e < 12; ++e) q[c][e] = 0.0f;
    }
    bool fin = false;                // wave-uniform: the producer has left and the queue is empty
    int nidle = 64;
    bool head = !producer;           // the wave's own pairs come first
    // Given states are read, not computed: where they are candidates, some four in ten end at once and the others soon, and waves that share out every
    // part of a batch as it comes all run with few lanes.  On large batches a wave therefore claims all that it has lanes for, or nothing yet.
    // Parts / whole, whole calls, us: candidates of 1 M points of scans 382 / 350, 0.5 M in four poses 196 / 184, 2 M ray samples 560 / 554; 0.11 M, 640 pairs per
    // block, 59 / 61; 24 states of 65 k points 307 either way.  (A wave that waits leaves the rest to the others, and the queue is never short of it: the
    // producer waits for room only where more than 64 entries are unclaimed.)
    const bool whole = !FUSED && total >= 2048ll * gridDim.x;
    do {                             // (test at the end: see k_solve_once)
        if (nidle >= S.refill_min && !fin) {
            int at = 64 * wib, got = nown, tail = 0, done = 0;
            if (!head && lane == 0) {  // entries [at, at + got) are this wave's; every failed exchange is another wave's success
                at = __hip_atomic_load(&s_claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const int t = lds_load_acquire(&s_tail);
                tail = t >> 1;
                done = t & 1;
                do {
                    got = max(min(nidle, tail - at), 0);
                    if (whole && !done && got < nidle) got = 0;
                } while (got > 0 && !__hip_atomic_compare_exchange_strong(&s_claim, &at, at + got, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                done = done && at + got >= tail;
            }
            at = __builtin_amdgcn_readfirstlane(at);
            got = __builtin_amdgcn_readfirstlane(got);
            fin = __builtin_amdgcn_readfirstlane(done) != 0;
            if (got > 0 || head) {
                const unsigned long long idle = __ballot(!active);
                const int rank = __popcll(idle & ((1ull << lane) - 1ull));
                if (!active && rank < got) {
                    const int e = (int)((unsigned)(at + rank) % WS_RING);
#pragma unroll
                    for (int r = 0; r < 3; ++r) {
                        xp[r] = s_ring[ST_XP + r][e];
                        x[r] = s_ring[ST_X + r][e];
                        g[r] = s_ring[ST_G + r][e];
                    }
#pragma unroll
                    for (int c = 0; c < 9; ++c) J[c] = s_ring[ST_J + c][e];
                    n = __float_as_int(s_ring[ST_N][e]);
                    k = __float_as_int(s_ring[ST_K][e]);
                    pz = __float_as_int(s_ring[ST_P][e]);
                    Tp = T + (long long)pz * stride;
                    it = 0;
                    held = -1;
                    active = true;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");      // the reads above are done
                __builtin_amdgcn_wave_barrier();
                if (lane == 0) {
                    const int first = head ? 64 : min(got, 64 - at % 64), seg = at / 64 % WS_SEGMENTS;
                    (void)__hip_atomic_fetch_add(&s_freed[seg], first, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (got > first)
                        (void)__hip_atomic_fetch_add(&s_freed[seg + 1 == WS_SEGMENTS ? 0 : seg + 1], got - first, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                head = false;
            }
        }
        // a consumer waits for nothing but its own block's producer, whose waits are all bounded and which raises
        // marks the tail as final on every way out: this loop ends when the producer has
        if (!__any(active) && !fin) __builtin_amdgcn_s_sleep(8);
        bool want_out = false;
        int out_place = -1, out_flags = 0;
        if (active) {
            bool conv;
            if (lane_step<SKIP>(G, S, Tp, may_skip, xp, x, g, J, it, q, held, held_mask, conv)) {
                want_out = true;
                out_flags = (conv ? 1 : 0) | (it << 8);
                if (cell_count && conv) out_place = pz * stride + held;
                active = false;
            } else if (!SKIP && S.prefetch) {
                // the corner records the next pass will need are asked for now: they travel while this pass parks
                // its results and the next one looks for work (q is free: its records went into d above).  On the
                // 8-pose grid, whose records come from beyond the L2: 1.34 -> 1.32 ms; on a grid the L2 holds the
                // second cell lookup costs more than the head start gains (0.172 -> 0.186 ms), hence the switch
                float xn[3] = {x[0], x[1], x[2]}, dn[3];
                advance(J, g, xn, dn);
                const Cell cn = locate(G, xn);
                if (cn.base != held) {
                    load_cell(Tp + cn.base, G, q);
                    held = cn.base;
                }
            }
        }
        out_park(G, want_out, x, J, out_flags, out_place, (int)((long long)k * N + n), outq, npend, lane, cell_count, ncell, rec);
        nidle = 64 - lanes_on(active);
    } while (!(fin && 64 - nidle <= QUADS));
    // the wave's last pairs, four lanes each
    quad_tail(G, S, T, active, lane, xp, x, g, J, it, n, k, pz, emit);
    if (npend > 0) out_flush(G, outq, npend, lane, cell_count, ncell, rec);
}

// Which pairs a wave of the kernels for small batches takes: `per` pairs (64, or 16 quads), as a tile of ki initial states
// times per / ki consecutive points.  Consecutive points share cache lines in the caller's arrays.  Initial states of one
// point often reach the same root and then share one atomic when positions are handed out (d_slot), but a point
// without a root keeps all its lanes busy to the last step, and a wave that holds 24 of those cannot go on in quads.
// ki = 1 without positions, 8 with them (16x16x4 grid, 98 k pairs with positions: ki 1 71, 4 50, 8 45, 24 52 us; 64x64x16:
// 72, 66, 66, 79 us).
__device__ __forceinline__ bool pair_of(unsigned w, unsigned i, unsigned per, unsigned N, int K, int ki, int &n, int &k)
{
    const unsigned pts = per / (unsigned)ki, tiles = (N + pts - 1u) / pts;
    const unsigned kb = w / tiles;
    k = (int)(kb * (unsigned)ki + i / pts);
    n = (int)((w - kb * tiles) * pts + i % pts);
    const bool live = i < per && k < K && n < (int)N;
    if (!live) n = k = 0;
    return live;
}

// ------------------------------------------------------------------------------------------------
// Broyden solve of a small batch: one quad of SIMD lanes per pair (see quad_step), no queue, no list, no records to
// unpack.  A wave takes 16 pairs of consecutive points (with positions and at least 8 states two points times eight states,
// see pair_of); the outputs go straight to the caller's arrays.  A batch this small is bound by its longest trajectories, i.e. by
// max_iters times the latency of a step.
// INIT: 0 one state per bone (Eq. (8)), 1 candidates of the correspondence grid, 2 the caller's initial states.
// LDS: the transform grids of all poses are copied into LDS first.
// rec (may be null): result records for the backward, with the positions in the cells' lists (cell_count not null).
// ------------------------------------------------------------------------------------------------
template <int INIT, bool LDS>
__global__ __launch_bounds__(LDS ? 1024 : 256) void k_solve_quad(GridP G, SolveP S, InitP I, const float *__restrict__ Tglobal,
                                               const float *__restrict__ xq, const int32_t *__restrict__ pose,
                                               const float *__restrict__ x0, const float *__restrict__ J0,
                                               const uint8_t *__restrict__ valid0, float *__restrict__ o_x,
                                               uint8_t *__restrict__ o_conv, float *__restrict__ o_J,
                                               uint8_t *__restrict__ o_it, int32_t *__restrict__ o_slot,
                                               float4 *__restrict__ rec, int *__restrict__ cell_count, int ncell, unsigned *__restrict__ total)
{
    extern __shared__ float4 s_grid[];
    if (cell_count && blockIdx.x == 0 && threadIdx.x == 0) *total = 0u;          // for place_cells, later in this call
    if (LDS) {
        const int n4 = (int)((long long)G.P * G.V * 3);      // float4 per record: 3
        const float4 *src = reinterpret_cast<const float4 *>(Tglobal);
        for (int i = threadIdx.x; i < n4; i += blockDim.x) s_grid[i] = src[i];
        __syncthreads();
    }
    const float *T = LDS ? reinterpret_cast<const float *>(s_grid) : Tglobal;
    const int lane = (int)(threadIdx.x & 63);
    const QuadAxis A = quad_axis(G, min(lane & 3, 2));
    const int row = A.row, lane3 = (int)(threadIdx.x & 3);
    const long long N = S.N;
    int n, k;
    const bool live = pair_of((blockIdx.x * blockDim.x + threadIdx.x) >> 6, (unsigned)lane >> 2, (unsigned)S.per, (unsigned)S.N, S.K, S.ki, n, k);
    const unsigned pair = (unsigned)k * (unsigned)N + (unsigned)n;
    const int p = pose_of(pose, n, G.P);
    const float *Tp = T + (long long)p * G.V * 12;
    float xp[3], x[3] = {0, 0, 0}, g[3] = {0, 0, 0}, J[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < 3; ++r) xp[r] = xq[r * N + n];
    const float xpr = pick3(row, xp[0], xp[1], xp[2]);
    bool ok;
    float dr = 0.0f;                 // d(x0) along the lane's axis
    if (INIT == 0) {
        const float *bi = I.Binv + ((long long)p * G.nb + k) * 12;
        ok = live && I.Bok[p * G.nb + k] != 0;
        if (ok) {
            const float y[3] = {xp[0] - bi[9], xp[1] - bi[10], xp[2] - bi[11]};
#pragma unroll
            for (int r = 0; r < 3; ++r)
                x[r] = FS_FMA(bi[r * 3 + 0], y[0], FS_FMA(bi[r * 3 + 1], y[1], bi[r * 3 + 2] * y[2]));
            const Cell c = locate(G, x);
            float q[8][4], om[8], Tr[4];
            quad_load(Tp + c.base, G, row, q);
            corner_weights(c, om);
            quad_blend(om, q, Tr);
            dr = quad_apply(Tr, x);
            // row r of jacobian_from_corners
            const float wx[2] = {1.0f - c.f[0], c.f[0]};
            const float wy[2] = {1.0f - c.f[1], c.f[1]};
            const float wz[2] = {1.0f - c.f[2], c.f[2]};
            float Jr[3] = {Tr[0], Tr[1], Tr[2]}, Jac[9];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int a = e & 1, b = (e >> 1) & 1, cz = (e >> 2) & 1;
                const float dc = quad_apply(q[e], x);
                float dw[3];
                dw[0] = c.cl[0] ? 0.0f : (a ? G.inv_h[0] : -G.inv_h[0]) * (wy[b] * wz[cz]);
                dw[1] = c.cl[1] ? 0.0f : (b ? G.inv_h[1] : -G.inv_h[1]) * (wx[a] * wz[cz]);
                dw[2] = c.cl[2] ? 0.0f : (cz ? G.inv_h[2] : -G.inv_h[2]) * (wx[a] * wy[b]);
#pragma unroll
                for (int j = 0; j < 3; ++j) Jr[j] = FS_FMA(dw[j], dc, Jr[j]);
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                Jac[j] = quad_get<0>(Jr[j]);
                Jac[3 + j] = quad_get<1>(Jr[j]);
                Jac[6 + j] = quad_get<2>(Jr[j]);
            }
            ok = inv3(Jac, J);
            if (!ok) {
#pragma unroll
                for (int e = 0; e < 9; ++e) J[e] = 0.0f;
            }
        }
    } else if (INIT == 1) {
        const int gcell = p * I.C.ncell + cell_index(I.C, I.bbox + p * 6, xp);
        const float4 *ci = I.cinit + ((long long)gcell * I.C.ck + k) * 4;
        const float4 a = ci[0], b = ci[1], c = ci[2], e = ci[3];
        ok = live && (__float_as_int(a.w) & 1) != 0;
        x[0] = a.x; x[1] = a.y; x[2] = a.z;
        dr = pick3(row, b.x, b.y, b.z);
        J[0] = b.w; J[1] = c.x; J[2] = c.y; J[3] = c.z; J[4] = c.w;
        J[5] = e.x; J[6] = e.y; J[7] = e.z; J[8] = e.w;
    } else {
#pragma unroll
        for (int r = 0; r < 3; ++r) x[r] = x0[((long long)k * 3 + r) * N + n];
#pragma unroll
        for (int e = 0; e < 9; ++e) J[e] = J0[((long long)k * 9 + e) * N + n];
        ok = live && valid0[pair] != 0;
        if (ok) {
            float q[8][4], om[8], Tr[4], f;
            quad_load(Tp + quad_place(A, pick3(row, x[0], x[1], x[2]), f), G, row, q);
            quad_weights(A, f, om);
            quad_blend(om, q, Tr);
            dr = quad_apply(Tr, x);
        }
    }
    bool conv = false, active = false;
    int it = 0;
    if (ok) {
        const float gr = dr - xpr;
        g[0] = quad_get<0>(gr);
        g[1] = quad_get<1>(gr);
        g[2] = quad_get<2>(gr);
        const float r2 = FS_FMA(g[2], g[2], FS_FMA(g[1], g[1], g[0] * g[0]));
        conv = r2 < S.tol2;
        active = !(conv || !(r2 < S.div2) || 0 >= S.max_iters);
    }
    QuadState state = quad_state(row, x, g, J);
    quad_run(G, S, A, T, active, lane, xpr, state, it, p, conv);
    quad_unpack(state, x, J);
    int pos = -1;
    if (cell_count) {
        const bool want = conv && lane3 == 0;
        const int cell = want ? p * ncell + cell_linear(G, locate(G, x)) : -1;
        const CellGroup cg = group_request(want, cell, threadIdx.x & 63, cell_count);
        const int at = group_position(cg);
        if (want) pos = at;
    }
    if (!live) return;
    if (lane3 < 3) {
        o_x[((long long)k * 3 + row) * N + n] = pick3(row, x[0], x[1], x[2]);
        if (o_J) {
#pragma unroll
            for (int j = 0; j < 3; ++j) o_J[((long long)k * 9 + row * 3 + j) * N + n] = pick3(row, J[j], J[3 + j], J[6 + j]);
        }
    } else {
        o_conv[pair] = conv ? 1 : 0;
        if (o_it) o_it[pair] = (uint8_t)it;
    }
    if (lane3 == 0 && o_slot) o_slot[pair] = pos;
    if (rec) {
        // lane i of the quad writes the i-th quarter of the record
        pos = quad_get<0>(pos);
        float4 v;
        if (lane3 == 0) v = make_float4(x[0], x[1], x[2], __int_as_float((conv ? 1 : 0) | (it << 8)));
        else if (lane3 == 1) v = make_float4(__int_as_float(pos), J[0], J[1], J[2]);
        else if (lane3 == 2) v = make_float4(J[3], J[4], J[5], J[6]);
        else v = make_float4(J[7], J[8], 0.0f, 0.0f);
        rec[(long long)pair * 4 + lane3] = v;
    }
}

// Broyden solve of a batch of medium size: one pair per SIMD lane for the steps that most pairs need, four lanes per pair
// for the rest (quad_tail).  Every wave owns 64 pairs and is done when they are: no queue, no cursor, no list, no
// records to unpack.  Pairs and outputs as in k_solve_quad.
template <int INIT, bool LDS>
__global__ __launch_bounds__(LDS ? 768 : 256, LDS ? 1 : 3) void k_solve_once(GridP G, SolveP S, InitP I, const float *__restrict__ Tglobal,
                                               const float *__restrict__ xq, const int32_t *__restrict__ pose,
                                               const float *__restrict__ x0, const float *__restrict__ J0,
                                               const uint8_t *__restrict__ valid0, float *__restrict__ o_x,
                                               uint8_t *__restrict__ o_conv, float *__restrict__ o_J,
                                               uint8_t *__restrict__ o_it, int32_t *__restrict__ o_slot,
                                               float4 *__restrict__ rec, int *__restrict__ cell_count, int ncell,
                                               const int *__restrict__ state, unsigned *__restrict__ total)
{
    extern __shared__ float4 s_grid[];
    if (cell_count && blockIdx.x == 0 && threadIdx.x == 0) *total = 0u;          // for place_cells, later in this call
    if (LDS) {
        const int n4 = (int)((long long)G.P * G.V * 3);      // float4 per record: 3
        const float4 *src = reinterpret_cast<const float4 *>(Tglobal);
        for (int i = threadIdx.x; i < n4; i += blockDim.x) s_grid[i] = src[i];
        __syncthreads();
    }
    constexpr bool SKIP = INIT != 1 && !LDS;      // as in k_solve_ws
    const float *T = LDS ? reinterpret_cast<const float *>(s_grid) : Tglobal;
    const int lane = threadIdx.x & 63;
    const long long N = S.N;
    int n, k;
    const bool live = pair_of((blockIdx.x * blockDim.x + threadIdx.x) >> 6, (unsigned)lane, WAVE, (unsigned)S.N, S.K, S.ki, n, k);
    const unsigned pair = (unsigned)k * (unsigned)N + (unsigned)n;
    const int p = pose_of(pose, n, G.P);
    const float *Tp = T + (long long)p * G.V * 12;
    float xp[3], x[3] = {0, 0, 0}, g[3] = {0, 0, 0}, d[3] = {0, 0, 0}, J[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    float q[8][12];
    int held = -1, held_mask = 0, it = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int e = 0; e < 12; ++e) q[c][e] = 0.0f;
#pragma unroll
    for (int r = 0; r < 3; ++r) xp[r] = xq[r * N + n];
    bool ok = false;
    if (live) {
        if (INIT == 0) {
            const float *bi = I.Binv + ((long long)p * G.nb + k) * 12;
            ok = I.Bok[p * G.nb + k] != 0;
            if (ok) {
                const float y[3] = {xp[0] - bi[9], xp[1] - bi[10], xp[2] - bi[11]};
#pragma unroll
                for (int r = 0; r < 3; ++r)
                    x[r] = FS_FMA(bi[r * 3 + 0], y[0], FS_FMA(bi[r * 3 + 1], y[1], bi[r * 3 + 2] * y[2]));
                const Cell c = locate(G, x);
                load_cell(Tp + c.base, G, q);
                held = c.base;
                held_mask = 0xFF;
                float Jac[9];
                jacobian_from_corners(G, c, q, x, d, Jac);
                ok = inv3(Jac, J);
                if (!ok) {
#pragma unroll
                    for (int e = 0; e < 9; ++e) J[e] = 0.0f;
                }
            }
        } else if (INIT == 1) {
            const int gcell = p * I.C.ncell + cell_index(I.C, I.bbox + p * 6, xp);
            const float4 *ci = I.cinit + ((long long)gcell * I.C.ck + k) * 4;
            const float4 a = ci[0], b = ci[1], c = ci[2], e = ci[3];
            ok = (__float_as_int(a.w) & 1) != 0;
            x[0] = a.x; x[1] = a.y; x[2] = a.z;
            d[0] = b.x; d[1] = b.y; d[2] = b.z;
            J[0] = b.w; J[1] = c.x; J[2] = c.y; J[3] = c.z; J[4] = c.w;
            J[5] = e.x; J[6] = e.y; J[7] = e.z; J[8] = e.w;
        } else {
#pragma unroll
            for (int r = 0; r < 3; ++r) x[r] = x0[((long long)k * 3 + r) * N + n];
#pragma unroll
            for (int e = 0; e < 9; ++e) J[e] = J0[((long long)k * 9 + e) * N + n];
            ok = valid0[pair] != 0;
            if (ok) {
                const Cell c = locate(G, x);
                load_cell(Tp + c.base, G, q);
                held = c.base;
                held_mask = 0xFF;
                blend_apply(c, q, x, d);
            }
        }
    }
    bool active = false;
    int flags = 0;                   // conv
    if (ok) {
#pragma unroll
        for (int r = 0; r < 3; ++r) g[r] = d[r] - xp[r];
        const float r2 = FS_FMA(g[2], g[2], FS_FMA(g[1], g[1], g[0] * g[0]));
        const bool conv = r2 < S.tol2;
        flags = conv ? 1 : 0;
        active = !(conv || !(r2 < S.div2) || 0 >= S.max_iters);
    }
    const bool may_skip = SKIP && may_skip_corners(state);
    // the test stands at the loop's end: at its head the compiler moves the whole state to other registers and back in every pass
    if (lanes_on(active) > QUADS) {
        do {
            if (active) {
                bool conv;
                if (lane_step<SKIP>(G, S, Tp, may_skip, xp, x, g, J, it, q, held, held_mask, conv)) {
                    active = false;
                    flags = conv ? 1 : 0;
                }
            }
        } while (lanes_on(active) > QUADS);
    }
    auto output = [&](bool ends, unsigned pr, bool conv, const float (&xe)[3], const float (&Je)[9], int ite, int ne, int ke, int pe) {
        int pos = -1;
        if (cell_count) {
            const bool want = ends && conv;
            if (__any(want)) {
                const int cell = want ? pe * ncell + cell_linear(G, locate(G, xe)) : -1;
                const CellGroup cg = group_request(want, cell, lane, cell_count);
                const int at = group_position(cg);
                if (want) pos = at;
            }
        }
        if (!ends) return;
#pragma unroll
        for (int r = 0; r < 3; ++r) o_x[((long long)ke * 3 + r) * N + ne] = xe[r];
        o_conv[pr] = conv ? 1 : 0;
        if (o_it) o_it[pr] = (uint8_t)ite;
        if (o_J) {
#pragma unroll
            for (int e = 0; e < 9; ++e) o_J[((long long)ke * 9 + e) * N + ne] = Je[e];
        }
        if (o_slot) o_slot[pr] = pos;
        if (rec) {
            float4 *o = rec + (long long)pr * 4;
            o[0] = make_float4(xe[0], xe[1], xe[2], __int_as_float((conv ? 1 : 0) | (ite << 8)));
            o[1] = make_float4(__int_as_float(pos), Je[0], Je[1], Je[2]);
            o[2] = make_float4(Je[3], Je[4], Je[5], Je[6]);
            o[3] = make_float4(Je[7], Je[8], 0.0f, 0.0f);
        }
    };
    // what has ended so far leaves together: consecutive lanes, consecutive points
    output(live && !active, pair, flags != 0, x, J, it, n, k, p);
    quad_tail(G, S, T, active, lane, xp, x, g, J, it, n, k, p,
              [&](bool ends, bool conv, const float (&xe)[3], const float (&Je)[9], int ite, int ne, int ke, int pe) {
                  output(ends, (unsigned)ke * (unsigned)N + (unsigned)ne, conv, xe, Je, ite, ne, ke, pe);
              });
}

// ------------------------------------------------------------------------------------------------
// Backward (Eq. (11)/(12), (15)).
// ------------------------------------------------------------------------------------------------
// The gradient w.r.t. the transform grid, G_T[p][v] = sum over converged lanes of
// omega_corner * lambda (x) [x*; 1], is accumulated without floating-point atomics (device-scope
// atomics leave the L2 on this chip and are slow): converged lanes are counting-sorted by the grid
// cell of x* (pass 1 below, or the positions k_solve hands out), crowded cells are summed once per
// corner (k_grad_pieces), and every grid node then adds what its 8 adjacent cells hold (k_grad_nodes_p).

// a[0..n) = 0
__global__ void k_fill_zero_i32(long long n, int *__restrict__ a)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) a[i] = 0;
}

// pass 1 (only when the solve did not hand out positions): one thread per lane; position of the lane
// inside its cell's list.  Bound: atomics on the cells' counters, which serialise on crowded cells; lanes of a wave in one
// cell share one.  A wave takes ki initial states of 64 / ki consecutive points (pair_of): states of one point often
// reach the same root.  (720 k lanes of 17 bones on 32x32x8 nodes: one atomic per lane 32 us, now 14.)
__global__ __launch_bounds__(256) void k_grad_count(GridP G, const float *__restrict__ xc,
                                                    const uint8_t *__restrict__ conv, const int32_t *__restrict__ pose,
                                                    long long N, int K, int ki, int ncell, int *__restrict__ count,
                                                    int *__restrict__ pos, unsigned *__restrict__ total)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *total = 0u;          // for place_cells, the next launch
    int n, k;
    const bool live = pair_of((blockIdx.x * 256u + threadIdx.x) >> 6, threadIdx.x & 63u, WAVE, (unsigned)N, K, ki, n, k);
    const long long q = (long long)k * N + n;
    const bool want = live && conv[q];
    int cell = 0;
    if (want) {
        const float x[3] = {xc[((long long)k * 3 + 0) * N + n], xc[((long long)k * 3 + 1) * N + n],
                            xc[((long long)k * 3 + 2) * N + n]};
        const Cell c = locate(G, x);
        cell = pose_of(pose, n, G.P) * ncell + cell_linear(G, c);
    }
    const CellGroup g = group_request(want, cell, threadIdx.x & 63, count);
    const int at = group_position(g);
    if (want) pos[q] = at;
}

// pass 2: a few threads per point share its lanes: lambda = -M^T g_x; the 32-byte record {x*[3], lambda[3],
// cell, 0} goes to the lane's slot of the cell-sorted list (one aligned sector per record);
// dL/dx' = sum_k M^T g_x without atomics.
constexpr int GREC = 8;           // floats per record
// FROM_REC: roots, masks, J~ and positions are taken from the result records the last solve left in the
// context (one contiguous 64-byte record per pair) instead of the caller's arrays; when that solve drew its
// pairs from the candidate list, only the first cand_cnt[n] lanes of point n have a record.
// JAC: lambda from J~, or (mode != 0) from the inverse of the exact Jacobian at x*, in one of three forms with the same bits; kernels of
// their own so that the J~ path does not carry the registers of a field evaluation.  The forms: all corners at once (112 and 120 registers, four
// waves per SIMD), in two halves of z-pairs (152 and 164, three), in halves and without corners of weight zero (171 and 182, two).
// REC_DEPTH (with FROM_REC and the J~ gradient only): lanes of a point in flight together, see below; 1 = one by one.
// Measured: depth 3 takes k_grad_records from 425 to 376 us on the 8-pose batch (one thread per point) and from 41 to
// 52 us on the SMPL-scale batch (8 threads per point, 5 instead of 8 waves per SIMD), hence a choice per launch.
enum { JAC_BROYDEN, JAC_CELL, JAC_HALVES, JAC_CLAMPED };
template <bool FROM_REC, int JAC, int REC_DEPTH = 1>
__global__ __launch_bounds__(256, JAC == JAC_CELL ? 4 : 1) void k_grad_records(GridP G, const float *__restrict__ T,
                                                      const float *__restrict__ xc, const float *__restrict__ Jinv,
                                                      const uint8_t *__restrict__ conv, const float *__restrict__ gxc,
                                                      const int32_t *__restrict__ pose, long long N, int K, int ncell,
                                                      const int *__restrict__ offset, const int *__restrict__ pos,
                                                      float4 *__restrict__ rec, float *__restrict__ gxq, int groups,
                                                      const float4 *__restrict__ srec, const uint8_t *__restrict__ cand_cnt,
                                                      const int *__restrict__ state)
{
    // `groups` (a power of two <= 8) threads share a point and take its lanes k = g, g + groups, ...;
    // consecutive threads of a group are consecutive points, so every load is coalesced
    __shared__ float s_gq[256 * 3];
    const int ppb = 256 / groups;                 // points per block
    constexpr bool EXACT = JAC != JAC_BROYDEN;
    const bool may_skip = JAC == JAC_CLAMPED && may_skip_corners(state);
    const int g = threadIdx.x / ppb, i = threadIdx.x - g * ppb;
    const long long n = (long long)blockIdx.x * ppb + i;
    float gq[3] = {0.0f, 0.0f, 0.0f};
    if (n < N) {
        const int p = pose_of(pose, n, G.P);
        const int nk = (FROM_REC && cand_cnt) ? min(K, (int)cand_cnt[n]) : K;
        if constexpr (FROM_REC && !EXACT && REC_DEPTH > 1) {
            // REC_DEPTH lanes of the point at a time, stage by stage, so that the dependent loads of a stage (record head,
            // rest of the record and g_x, cell offsets) travel together
            for (int k0 = g; k0 < nk; k0 += REC_DEPTH * groups) {
                float4 ra[REC_DEPTH], rb[REC_DEPTH], rc[REC_DEPTH], rd[REC_DEPTH];
                float gx[REC_DEPTH][3];
                bool on[REC_DEPTH];
                long long q[REC_DEPTH];
#pragma unroll
                for (int u = 0; u < REC_DEPTH; ++u) {
                    const int k = k0 + u * groups;
                    on[u] = k < nk;
                    q[u] = (long long)(on[u] ? k : 0) * N + n;
                    ra[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if (on[u]) ra[u] = srec[q[u] * 4];
                }
#pragma unroll
                for (int u = 0; u < REC_DEPTH; ++u) {
                    on[u] = on[u] && (__float_as_int(ra[u].w) & 1);
                    rb[u] = rc[u] = rd[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    gx[u][0] = gx[u][1] = gx[u][2] = 0.0f;
                    if (on[u]) {
                        rb[u] = srec[q[u] * 4 + 1];
                        rc[u] = srec[q[u] * 4 + 2];
                        rd[u] = srec[q[u] * 4 + 3];
                        const int k = k0 + u * groups;
#pragma unroll
                        for (int r = 0; r < 3; ++r) gx[u][r] = gxc[((long long)k * 3 + r) * N + n];
                    }
                }
                float lam[REC_DEPTH][3];
                int cl[REC_DEPTH], o0[REC_DEPTH], o1[REC_DEPTH];
#pragma unroll
                for (int u = 0; u < REC_DEPTH; ++u) {
                    const float M[9] = {rb[u].y, rb[u].z, rb[u].w, rc[u].x, rc[u].y, rc[u].z, rc[u].w, rd[u].x, rd[u].y};
                    const float x[3] = {ra[u].x, ra[u].y, ra[u].z};
                    cl[u] = 0;
                    o0[u] = o1[u] = 0;
#pragma unroll
                    for (int r = 0; r < 3; ++r) {
                        lam[u][r] = -FS_FMA(M[6 + r], gx[u][2], FS_FMA(M[3 + r], gx[u][1], M[r] * gx[u][0]));
                        if (on[u]) gq[r] -= lam[u][r];
                    }
                    if (on[u]) {
                        const Cell c = locate(G, x);
                        cl[u] = p * ncell + cell_linear(G, c);
                        const int *o = offset + place(cl[u]);
                        o0[u] = o[0];
                        o1[u] = o[1];
                    }
                }
#pragma unroll
                for (int u = 0; u < REC_DEPTH; ++u) {
                    const int pq = __float_as_int(rb[u].x);      // the position the solve kernel left in the record
                    const long long slot = (long long)o0[u] + pq;
                    if (!on[u] || pq < 0 || slot >= o1[u]) continue;
                    rec[slot * 2] = make_float4(ra[u].x, ra[u].y, ra[u].z, lam[u][0]);
                    rec[slot * 2 + 1] = make_float4(lam[u][1], lam[u][2], __int_as_float(cl[u]), 0.0f);
                }
            }
        } else
        for (int k = g; k < nk; k += groups) {
            const long long q = (long long)k * N + n;
            float x[3], gx[3], M[9];
            int pq;
            if (FROM_REC) {
                const float4 a = srec[q * 4];
                if (!(__float_as_int(a.w) & 1)) continue;
                x[0] = a.x; x[1] = a.y; x[2] = a.z;
                pq = __float_as_int(srec[q * 4 + 1].x);      // the position the solve kernel left in the record
                if (!EXACT) read_record_J(srec + q * 4, M);
            } else {
                if (!conv[q]) continue;
#pragma unroll
                for (int r = 0; r < 3; ++r) x[r] = xc[((long long)k * 3 + r) * N + n];
                pq = pos[q];
                if (!EXACT) {
#pragma unroll
                    for (int e = 0; e < 9; ++e) M[e] = Jinv[((long long)k * 9 + e) * N + n];
                }
            }
#pragma unroll
            for (int r = 0; r < 3; ++r) gx[r] = gxc[((long long)k * 3 + r) * N + n];
            bool ok = true;
            if (EXACT) {
                float d[3], J[9];
                const float *Tp = T + (long long)p * G.V * 12;
                if constexpr (JAC == JAC_CELL) {
                    field_dJ(Tp, G, x, d, J);
                } else {
                    const Cell c = locate(G, x);
                    if constexpr (JAC == JAC_HALVES) (void)prepare_jacobian(Tp + c.base, G, c, 0xFF, x, d, J);
                    else field_dJ_clamped(Tp, G, c, may_skip, x, d, J);
                }
                ok = inv3(J, M);
            }
            float lam[3] = {0.0f, 0.0f, 0.0f};
            if (ok) {
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    lam[r] = -FS_FMA(M[6 + r], gx[2], FS_FMA(M[3 + r], gx[1], M[r] * gx[0]));
                    gq[r] -= lam[r];
                }
            }
            const Cell c = locate(G, x);
            const int cl = p * ncell + cell_linear(G, c);
            const int *o = offset + place(cl);
            const long long slot = (long long)o[0] + pq;
            // positions that do not belong to these roots (a caller mixing arrays of different solves)
            // must not send the store outside the cell's part of the list
            if (pq < 0 || slot >= o[1]) continue;
            rec[slot * 2] = make_float4(x[0], x[1], x[2], lam[0]);
            rec[slot * 2 + 1] = make_float4(lam[1], lam[2], __int_as_float(cl), 0.0f);
        }
    }
    if (!gxq) return;
#pragma unroll
    for (int r = 0; r < 3; ++r) s_gq[threadIdx.x * 3 + r] = gq[r];
    __syncthreads();
    if (g == 0 && n < N) {
        for (int h = 1; h < groups; ++h)
#pragma unroll
            for (int r = 0; r < 3; ++r) gq[r] += s_gq[(h * ppb + i) * 3 + r];
#pragma unroll
        for (int r = 0; r < 3; ++r) gxq[r * N + n] = gq[r];
    }
}

// fraction of x along one axis inside the cell that starts at node i0: what locate() returns for a point of
// that cell (same clamping, same subtraction), without looking the cell up again
__device__ __forceinline__ float frac_in_cell(float x, float lo, float inv_h, float m, int i0)
{
    return __builtin_amdgcn_fmed3f((x - lo) * inv_h, 0.0f, m) - (float)i0;
}

// contribution of a sorted record {x*, lambda}, which lies in the cell with origin (cx, cy, cz), to the node that is that
// cell's corner (da, db, dc)
__device__ __forceinline__ void grad_accumulate(const GridP &G, const float4 r0, const float4 r1, int cx, int cy, int cz,
                                                int da, int db, int dc, float (&acc)[12])
{
    const float x[3] = {r0.x, r0.y, r0.z};
    const float lam[3] = {r0.w, r1.x, r1.y};
    const float fx = frac_in_cell(x[0], G.lo[0], G.inv_h[0], G.m[0], cx);
    const float fy = frac_in_cell(x[1], G.lo[1], G.inv_h[1], G.m[1], cy);
    const float fz = frac_in_cell(x[2], G.lo[2], G.inv_h[2], G.m[2], cz);
    const float wx = da ? fx : 1.0f - fx;
    const float wy = db ? fy : 1.0f - fy;
    const float wz = dc ? fz : 1.0f - fz;
    const float om = (wx * wy) * wz;
#pragma unroll
    for (int rr = 0; rr < 3; ++rr) {
        const float wl = om * lam[rr];
        acc[rr * 4 + 0] = FS_FMA(wl, x[0], acc[rr * 4 + 0]);
        acc[rr * 4 + 1] = FS_FMA(wl, x[1], acc[rr * 4 + 1]);
        acc[rr * 4 + 2] = FS_FMA(wl, x[2], acc[rr * 4 + 2]);
        acc[rr * 4 + 3] += wl;
    }
}

// the 12 sums of a piece for one corner
__device__ __forceinline__ void add_sums(const float4 (&v)[3], float (&acc)[12])
{
#pragma unroll
    for (int h = 0; h < 3; ++h) {
        acc[4 * h] += v[h].x;
        acc[4 * h + 1] += v[h].y;
        acc[4 * h + 2] += v[h].z;
        acc[4 * h + 3] += v[h].w;
    }
}

__device__ __forceinline__ int adjacent_cell(const GridP &G, int ncell, int p, int ix, int iy, int iz, int cn)
{
    const int cx = ix - (cn & 1), cy = iy - ((cn >> 1) & 1), cz = iz - ((cn >> 2) & 1);
    if (cx < 0 || cy < 0 || cz < 0 || cx > G.nx - 2 || cy > G.ny - 2 || cz > G.nz - 2) return -1;
    return p * ncell + (cx * (G.ny - 1) + cy) * (G.nz - 1) + cz;
}

// pass 3.  The cell-sorted record list is cut at every multiple of PIECE_R; a piece is what one cell owns
// of one such range.  A piece of at least PIECE_MIN records is replaced, in place, by its sums for the
// 8 corners of the cell (8 x 12 floats = the storage of 12 records), so that a node later reads 12
// floats per piece instead of every record of a crowded cell; shorter pieces stay as records.
constexpr int PIECE_R = 256;
constexpr int PIECE_MIN = 96 / GREC;
constexpr int PIECE_WAVES = PIECE_R / 64; // waves per range, a record per SIMD lane (2 waves, two records each: the same but on sparse lists, 62.6 instead of 54.6 us on 7.7 M records)

// Bound: instruction issue (vector units 0.6 and matrix cores 0.25 of the busy cycles with 25 records per cell), so a pass has a comparison and a
// select per group only where the piece may end in it, nothing is masked that nobody stores, and where pieces lie is found with scalar bit
// operations on one ballot per wave (1.3 M records in 60 k cells, pieces of some 25: 30.1 -> 23.1 us; 0.48 M 13.3 -> 10.6).  Persistent blocks that ask
// for the next range's records early: 37 instead of 30 us; loading records before the total is known: nothing on full lists, 20 -> 53 us on others.
// One block of PIECE_WAVES waves per range: a thread loads and expands a record, the waves
// take the long pieces in turn.  Every record of the range is expanded once (SIMD lane = record) into its 8 corner
// weights omega_c and its 12 products lambda_r [x*; 1]_j, staged in LDS; the sums of a piece are then the
// matrix product  S[c][rj] = sum_t omega_c(t) * (lambda_r [x;1]_j)(t),  an 8 x len by len x 12 contraction,
// taken four records at a time by the 16x16x4 fp32 MFMA (rows 8..15 and columns 12..15 are zero padding).
// Operand layout of that instruction: lane 16k+i supplies A[i][k] and B[k][i]; lane 16g+j receives
// D[4g+q][j] in accumulator register q.
constexpr int PIECE_ROW = 20;     // floats per staged record: 8 weights + 12 products
typedef float v4f __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(64 * PIECE_WAVES) void k_grad_pieces(GridP G, const unsigned *__restrict__ records, float *rec)
{
    __shared__ float4 sm4[(PIECE_R + 16) * PIECE_ROW / 4 + 1];          // ... 16 rows of zeros, and the four columns read behind the last
    __shared__ unsigned long long s_start[PIECE_WAVES];
    float *sm = reinterpret_cast<float *>(sm4);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long s = (long long)blockIdx.x * PIECE_R;
    const long long total = *records;
    if (s >= total) return;
    const int e = (int)min((long long)PIECE_R, total - s);
    // thread t loads and expands record t of the range.  A piece starts where the cell differs from the one before (lane 0 reads the record of the
    // wave before for that); the first of the range always starts one, and so does the end of the list, for what lies before it.
    const int t = threadIdx.x;
    float4 r0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), r1 = r0;
    int before = -1;
    if (t < e) {
        const float4 *r = reinterpret_cast<const float4 *>(rec + (s + t) * GREC);
        r0 = r[0];
        r1 = r[1];
        if (lane == 0 && t > 0) before = __float_as_int(r[-1].z);
    }
    {
        const int cell = __float_as_int(r1.z), left = __shfl_up(cell, 1);
        if (lane > 0) before = left;
        const unsigned long long b = __ballot(t == e || (t < e && (t == 0 || cell != before)));
        if (lane == 0) s_start[w] = b;
    }
    __syncthreads();
    // Every wave finds the long pieces of the whole range, with scalar instructions: a start is one if none of the next PIECE_MIN - 1 places is a
    // start.
    unsigned long long start[PIECE_WAVES], many[PIECE_WAVES], any_long = 0ull;
#pragma unroll
    for (int b = 0; b < PIECE_WAVES; ++b) {
        const unsigned long long v = s_start[b];
        start[b] = (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32)) << 32 |
                   (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
    }
#pragma unroll
    for (int b = 0; b < PIECE_WAVES; ++b) {
        const unsigned long long after = b + 1 < PIECE_WAVES ? start[b + 1] : 1ull;         // the range ends behind its last record
        static_assert(PIECE_MIN == 12, "the next 11 places");
        unsigned long long lo = start[b] >> 1 | after << 63, hi = after >> 1;               // bit l: place l + 1
        lo |= lo >> 1 | hi << 63, hi |= hi >> 1;
        lo |= lo >> 2 | hi << 62, hi |= hi >> 2;
        lo |= lo >> 4 | hi << 60, hi |= hi >> 4;                                            // places l + 1 .. l + 8
        lo |= lo >> 3 | hi << 61;
        many[b] = start[b] & ~lo;
        if (e < 64 * (b + 1)) many[b] &= e > 64 * b ? (1ull << (e - 64 * b)) - 1ull : 0ull; // the end of the list is no piece
        any_long |= many[b];
    }
    if (!any_long) return;              // nothing to summarise here (sparse lists end here); same in every wave
    // expand the records
    if (threadIdx.x <= 16 * PIECE_ROW / 4) sm4[PIECE_R * PIECE_ROW / 4 + threadIdx.x] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    {
        float4 o[5];
#pragma unroll
        for (int h = 0; h < 5; ++h) o[h] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (t < e) {
            const float x[3] = {r0.x, r0.y, r0.z};
            const float lam[3] = {r0.w, r1.x, r1.y};
            const Cell cl = locate(G, x);
            float om[8];
            corner_weights(cl, om);
            o[0] = make_float4(om[0], om[1], om[2], om[3]);
            o[1] = make_float4(om[4], om[5], om[6], om[7]);
#pragma unroll
            for (int rr = 0; rr < 3; ++rr) o[2 + rr] = make_float4(lam[rr] * x[0], lam[rr] * x[1], lam[rr] * x[2], lam[rr]);
        }
#pragma unroll
        for (int h = 0; h < 5; ++h) sm4[t * (PIECE_ROW / 4) + h] = o[h];
    }
    __syncthreads();
    const int col = lane & 15, kq = lane >> 4, zero = (PIECE_R + kq) * PIECE_ROW + col;
    int turn = 0;                        // the waves take the long pieces in turn
#pragma unroll
    for (int i = 0; i < PIECE_WAVES; ++i) {
        unsigned long long m = many[i];
        while (m) {
            const int src = __ffsll((long long)m) - 1;
            m &= m - 1ull;
            const bool mine = turn == w;
            turn = turn + 1 == PIECE_WAVES ? 0 : turn + 1;
            if (!mine) continue;
            // it ends where the next one starts
            const int ps = 64 * i + src;
            const unsigned long long rest = start[i] >> src >> 1;
            int pe = PIECE_R;
#pragma unroll
            for (int b = PIECE_WAVES - 1; b > i; --b)
                if (start[b]) pe = 64 * b + __ffsll((long long)start[b]) - 1;
            if (rest) pe = ps + __ffsll((long long)rest);
            // Four groups per pass into four accumulators: their LDS reads are in flight together and no MFMA waits for the one before it.
            // Records behind the piece enter as rows of zeros; rows 8..15 and columns 12..15 are sums of whatever lies there, which nobody
            // stores.  `at`: this lane's entry of the pass's first group; a group is 4 rows further.
            v4f acc4[4];
            int at = (ps + kq) * PIECE_ROW + col, n = pe - ps;
            {
                float av[4], bv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float *q = sm + (4 * u + kq < n ? at : zero) + 4 * u * PIECE_ROW;
                    av[u] = q[0];
                    bv[u] = q[8];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) acc4[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], bv[u], (v4f){0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
            }
            for (n -= 16, at += 16 * PIECE_ROW; n >= 16; n -= 16, at += 16 * PIECE_ROW) {
                float av[4], bv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    av[u] = sm[at + 4 * u * PIECE_ROW];
                    bv[u] = sm[at + 4 * u * PIECE_ROW + 8];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) acc4[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], bv[u], acc4[u], 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (4 * u < n) {
                    const float *q = sm + (4 * u + kq < n ? at : zero) + 4 * u * PIECE_ROW;
                    acc4[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[0], q[8], acc4[u], 0, 0, 0);
                }
            const v4f acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
            if (kq < 2 && col < 12) {
                float *o = rec + (s + ps) * GREC + (4 * kq) * 12 + col;
                o[0] = acc[0];
                o[12] = acc[1];
                o[24] = acc[2];
                o[36] = acc[3];
            }
        }
    }
}

// v of the lane that the DPP control names, all lanes taking part
template <int CTRL>
__device__ __forceinline__ float lane_from(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// G_T of every node from the pieces of its 8 adjacent cells, for crowded cells (k_grad_nodes_z takes the sparse ones): 8 threads
// share a node, one per adjacent cell, and add what they have in a butterfly.
// Bound: vector instructions (0.75 of the busy cycles), then the chain of the most crowded cell (at the box's corners, 12 k records of 1.3 M), whose whole ranges
// are therefore added four at a time (65 k points 15.7 -> 14.0 us, with the butterfly on DPP and one clamp per fraction; four sums or several records
// asked for at a time wherever there is more than one: 18 to 19).
// Measured on the multi-pose batch (7.7 M records over 4.2 M nodes, one thread per node: 450 us) and not adopted: a block per brick
// of 4 x 4 x 16 nodes that first copies the records of the cells around it into LDS and gathers from there, same loops:
// 450 .. 518 us (fewer resident threads, three barriers per block); the same with one loop over all records of a node's
// 8 cells instead of a loop per cell: 751 us (the bookkeeping costs more than the shorter loop saves); a block per brick
// that adds every record's 8 x 12 contributions into LDS sums with LDS float atomics: 4.5 ms (about 0.5 SIMD lanes per
// clock and CU).
__global__ __launch_bounds__(256) void k_grad_nodes_p(GridP G, int ncell, const int *__restrict__ offset,
                                                      const float *__restrict__ rec, float *__restrict__ GT)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long i = t >> 3;
    const int cn = (int)(t & 7);
    if (i >= (long long)G.P * G.V) return;
    const int p = (int)div_by((unsigned)i, (unsigned)G.V, G.mag_V);          // P * V < 2^31
    const unsigned v = (unsigned)(i - (long long)p * G.V), tz = div_by(v, (unsigned)G.nz, G.mag_nz);
    const int iz = (int)(v - tz * (unsigned)G.nz), ix = (int)div_by(tz, (unsigned)G.ny, G.mag_ny);
    const int iy = (int)(tz - (unsigned)ix * (unsigned)G.ny);
    float acc[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) acc[e] = 0.0f;
    const int c = adjacent_cell(G, ncell, p, ix, iy, iz, cn);
    const int a = c < 0 ? 0 : offset[place(c)], b = c < 0 ? 0 : offset[place(c) + 1];
    for (int ps = a, pe; ps < b; ps = pe) {
        const float4 *q = reinterpret_cast<const float4 *>(rec + (long long)ps * GREC + cn * 12);
        if (ps % PIECE_R == 0 && b - ps >= 4 * PIECE_R) {          // four whole ranges: their sums on the way together
            float4 v[4][3];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < 3; ++h) v[u][h] = q[u * (PIECE_R * GREC / 4) + h];
#pragma unroll
            for (int u = 0; u < 4; ++u) add_sums(v[u], acc);
            pe = ps + 4 * PIECE_R;
            continue;
        }
        pe = min(b, (ps / PIECE_R + 1) * PIECE_R);
        if (pe - ps >= PIECE_MIN) {
            const float4 v[3] = {q[0], q[1], q[2]};
            add_sums(v, acc);
        } else {
            for (int s = ps; s < pe; ++s) {
                const float4 *r = reinterpret_cast<const float4 *>(rec + (long long)s * GREC);
                grad_accumulate(G, r[0], r[1], ix - (cn & 1), iy - ((cn >> 1) & 1), iz - ((cn >> 2) & 1), cn & 1, (cn >> 1) & 1,
                                (cn >> 2) & 1, acc);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 12; ++e) {
        acc[e] += lane_from<0xB1>(acc[e]);           // the neighbour of a pair, then of a quad
        acc[e] += lane_from<0x4E>(acc[e]);
        acc[e] += lane_from<0x141>(acc[e]);          // the other quad of eight lanes
    }
    if (cn == 0) {
        float4 *o = reinterpret_cast<float4 *>(GT + i * 12);
        o[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        o[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
        o[2] = make_float4(acc[8], acc[9], acc[10], acc[11]);
    }
}

// One record {x*, lambda} of the cell with origin (cx, cy, cz): its share for the cell's (x, y) corner (bx, by) at the lower
// z (into lo) and at the upper z (into hi)
template <bool LO, bool HI>
__device__ __forceinline__ void grad_record_pair(const GridP &G, const float4 r0, const float4 r1, bool bx, bool by, int cx, int cy,
                                                 int cz, float (&lo)[12], float (&hi)[12])
{
    const float x[3] = {r0.x, r0.y, r0.z};
    const float lam[3] = {r0.w, r1.x, r1.y};
    const float fx = frac_in_cell(x[0], G.lo[0], G.inv_h[0], G.m[0], cx);
    const float fy = frac_in_cell(x[1], G.lo[1], G.inv_h[1], G.m[1], cy);
    const float fz = frac_in_cell(x[2], G.lo[2], G.inv_h[2], G.m[2], cz);
    const float wxy = (bx ? fx : 1.0f - fx) * (by ? fy : 1.0f - fy);
    const float w0 = wxy * (1.0f - fz), w1 = wxy * fz;
#pragma unroll
    for (int rr = 0; rr < 3; ++rr) {
        if (LO) {
            const float wl = w0 * lam[rr];
            lo[rr * 4 + 0] = FS_FMA(wl, x[0], lo[rr * 4 + 0]);
            lo[rr * 4 + 1] = FS_FMA(wl, x[1], lo[rr * 4 + 1]);
            lo[rr * 4 + 2] = FS_FMA(wl, x[2], lo[rr * 4 + 2]);
            lo[rr * 4 + 3] += wl;
        }
        if (HI) {
            const float wl = w1 * lam[rr];
            hi[rr * 4 + 0] = FS_FMA(wl, x[0], hi[rr * 4 + 0]);
            hi[rr * 4 + 1] = FS_FMA(wl, x[1], hi[rr * 4 + 1]);
            hi[rr * 4 + 2] = FS_FMA(wl, x[2], hi[rr * 4 + 2]);
            hi[rr * 4 + 3] += wl;
        }
    }
}

// What the records of cell (cx, cy, cz), list entries [a, b), add to the two nodes at its (x, y) corner `ab`
// (= a + 2b): `lo` is the node at cz, `hi` the one at cz + 1.  Pieces that k_grad_pieces replaced by their corner
// sums enter as those sums.  Either output may be switched off.
template <bool LO, bool HI>
__device__ __forceinline__ void grad_cell_pair(const GridP &G, const float *__restrict__ rec, int a, int b, int ab, int cx,
                                               int cy, int cz, float (&lo)[12], float (&hi)[12])
{
    for (int j = a / PIECE_R; j <= (b - 1) / PIECE_R; ++j) {
        const int ps = max(a, j * PIECE_R), pe = min(b, (j + 1) * PIECE_R);
        if (pe - ps >= PIECE_MIN) {
            const float4 *q0 = reinterpret_cast<const float4 *>(rec + (long long)ps * GREC + ab * 12);
            const float4 *q1 = q0 + 12;                   // corner ab + 4
#pragma unroll
            for (int h = 0; h < 3; ++h) {
                if (LO) {
                    const float4 u = q0[h];
                    lo[4 * h] += u.x; lo[4 * h + 1] += u.y; lo[4 * h + 2] += u.z; lo[4 * h + 3] += u.w;
                }
                if (HI) {
                    const float4 u = q1[h];
                    hi[4 * h] += u.x; hi[4 * h + 1] += u.y; hi[4 * h + 2] += u.z; hi[4 * h + 3] += u.w;
                }
            }
        } else {
            for (int s = ps; s < pe; ++s) {
                const float4 *r = reinterpret_cast<const float4 *>(rec + (long long)s * GREC);
                grad_record_pair<LO, HI>(G, r[0], r[1], ab & 1, ab & 2, cx, cy, cz, lo, hi);
            }
        }
    }
}

// G_T of every node for sparse lists (a few records per cell): one thread per node, consecutive SIMD lanes consecutive
// nodes along z.  A node-by-node gather over its 8 adjacent cells reads every record 8 times, and a wave runs as long
// as the sum over the 8 cells of the longest list among its lanes.  Here a lane walks only the 4 cells at its own height
// (cz = iz), adds each record's share for the lower z-corner to its own node and collects the share for the upper
// z-corner, which belongs to the node above it: the next SIMD lane, which receives it with one shuffle per entry.  Every
// record is read 4 times and the loops are half as long.  A lane whose lower neighbour sits in another wave (lane 0 of
// a wave that starts inside a column) walks that neighbour's 4 cells itself.
__global__ __launch_bounds__(256) void k_grad_nodes_z(GridP G, int ncell, const int *__restrict__ offset,
                                                      const float *__restrict__ rec, float *__restrict__ GT)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool valid = i < (long long)G.P * G.V;
    int p = 0, ix = 0, iy = 0, iz = 0;
    if (valid) {
        p = (int)div_by((unsigned)i, (unsigned)G.V, G.mag_V);          // P * V < 2^31
        const unsigned v = (unsigned)(i - (long long)p * G.V), t = div_by(v, (unsigned)G.nz, G.mag_nz);
        iz = (int)(v - t * (unsigned)G.nz);
        ix = (int)div_by(t, (unsigned)G.ny, G.mag_ny);
        iy = (int)(t - (unsigned)ix * (unsigned)G.ny);
    }
    float acc[12], up[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) acc[e] = up[e] = 0.0f;
    if (valid && iz <= G.nz - 2) {
        // Cells with fewer than PIECE_MIN records hold records only (no sums): those of the 4 cells are walked as one list,
        // four records per round whose loads travel together, so that a wave runs as long as the longest sum of four lists
        // among its lanes.  Bound: vector ALU (2700 instructions per wave with the 4 lists side by side, a record of
        // each per round, as long as the longest list of any lane: 282 us on 8 poses of 128x128x32 nodes with 7.7 M
        // records, now 226).  The other cells follow one by one.
        int a[4], from[4], upto[4];       // upto[ab]: records of the cells up to and with ab; record t of the walk is from[ab] + t
        bool small[4];
        int walk = 0;
#pragma unroll
        for (int ab = 0; ab < 4; ++ab) {
            const int cx = ix - (ab & 1), cy = iy - (ab >> 1);
            int b = a[ab] = 0;
            if (!(cx < 0 || cy < 0 || cx > G.nx - 2 || cy > G.ny - 2)) {
                const int c = p * ncell + (cx * (G.ny - 1) + cy) * (G.nz - 1) + iz;
                a[ab] = offset[place(c)];
                b = offset[place(c) + 1];
            }
            small[ab] = b - a[ab] < PIECE_MIN;
            from[ab] = a[ab] - walk;
            if (small[ab]) walk += b - a[ab];
            upto[ab] = walk;
        }
        for (int j = 0; j < walk; j += 4) {
            float4 r0[4], r1[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = j + u;
                int f = from[0];
                f = t >= upto[0] ? from[1] : f;
                f = t >= upto[1] ? from[2] : f;
                f = t >= upto[2] ? from[3] : f;
                if (t < walk) {
                    const float4 *r = reinterpret_cast<const float4 *>(rec + (long long)(f + t) * GREC);
                    r0[u] = r[0];
                    r1[u] = r[1];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = j + u;
                const bool by = t >= upto[1], bx = t >= upto[2] || (t >= upto[0] && !by);
                if (t < walk) grad_record_pair<true, true>(G, r0[u], r1[u], bx, by, bx ? ix - 1 : ix, by ? iy - 1 : iy, iz, acc, up);
            }
        }
#pragma unroll
        for (int ab = 0; ab < 4; ++ab)
            if (!small[ab]) grad_cell_pair<true, true>(G, rec, a[ab], offset[place(p * ncell + ((ix - (ab & 1)) * (G.ny - 1) + iy - (ab >> 1)) * (G.nz - 1) + iz) + 1], ab, ix - (ab & 1), iy - (ab >> 1), iz, acc, up);
    }
    // what the node below collected for this one (lane - 1 is node i - 1: the same column when iz > 0)
    const bool from_lane = lane > 0 && valid && iz > 0;
#pragma unroll
    for (int e = 0; e < 12; ++e) {
        const float below = __shfl_up(up[e], 1);
        if (from_lane) acc[e] += below;
    }
    if (valid && iz > 0 && !from_lane) {
        for (int ab = 0; ab < 4; ++ab) {
            const int cx = ix - (ab & 1), cy = iy - (ab >> 1);
            if (cx < 0 || cy < 0 || cx > G.nx - 2 || cy > G.ny - 2) continue;
            const int c = p * ncell + (cx * (G.ny - 1) + cy) * (G.nz - 1) + iz - 1;
            const int a = offset[place(c)], b = offset[place(c) + 1];
            if (a != b) grad_cell_pair<false, true>(G, rec, a, b, ab, cx, cy, iz - 1, up, acc);
        }
    }
    // the wave's 64 records are contiguous: they leave as whole cache lines
    __shared__ __attribute__((aligned(16))) float s_tiles[4][64 * 12];
    const long long i0 = i - lane;
    wave_store_rows<12>(GT + i0 * 12, acc, (int)min(64ll, (long long)G.P * G.V - i0), s_tiles[threadIdx.x >> 6]);
}

// The two gradients that are read off G_T, in one pass over it:
//   gW[v][b]    = sum_p sum_e G_T[p][v][e] B[p][b][e]     per node a 12 P x n_b product
//   gB[p][b][e] = sum_v W[v][b] G_T[p][v][e]              n_b x V by V x 12 P, a long inner dimension
// Bound: memory, 48 P + 8 n_b bytes per node, with many poses the matrix cores beside it.  A wave takes 16 nodes at a time;
// the 12 entries of up to eight poses are one row of 12 P, of which a lane holds 16-byte quarters: quarter 4s + k of
// node i in slot s of lane 16k + i.  Both products run on the 16x16x4 fp32 MFMA with no padding between poses.  The quarters
// are the A operand of gW as they lie, entry u of each in step u (the order in the inner sum is free).  gB contracts over
// the nodes and reads the same tile back from LDS the other way round, 16 columns per slot.  gB stays in registers over all
// tiles of a wave; a block leaves one partial result [n_b][12] per pose, which k_grad_bones_final adds.  Weights come
// and gW goes through LDS as whole lines.  The next tile's loads are under way while one is multiplied.
// MT = number of 16-bone tiles, S = slots: 1 for one pose, 3 for four, 6 for eight (with up to 32 bones: beyond, the
// registers of two waves per SIMD are used up); more poses take further passes, which add to gW.
// Two kernels, gW with vector FMAs on bones in LDS and gB on the MFMA, both over all of G_T: 85 + 82 us on 8 poses of 128x128x32
// nodes, 5.5 + 8.8 on one of 64x64x16; this one 82 (3.7 TB/s) and 6.6.  With 16 padded columns per pose it took 128, without
// the way through LDS for weights and gW 146.
template <int MT, int S>
__global__ __launch_bounds__(256, 2) void k_grad_outputs(GridP G, const float *__restrict__ W, const float *__restrict__ GT,
                                                         const float *__restrict__ B, float *gW, float *__restrict__ part)
{
    constexpr int PC = S * 4 / 3, ROW = S * 16 + 8;          // poses per pass; floats per row of the tile in LDS (padded: no bank twice)
    __shared__ float4 s_bone[S * 4][MT * 16];    // quarter x bone, zero where there is no such pose or bone
    __shared__ float4 s_tile[4][16 * ROW / 4];
    __shared__ float4 s_w[4][MT * 64];          // the weights of a wave's tile, then its part of gW
    __shared__ v4f s_acc[3][MT][64];
    const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6, col = lane & 15, kq = lane >> 4;
    const int wave = blockIdx.x * 4 + wib, nwaves = gridDim.x * 4;
    const int tiles = (int)((G.V + 15) / 16), nout = G.nb * 12, V = (int)G.V;      // 12 P V < 2^31
    float *const tw = reinterpret_cast<float *>(s_w[wib]);
    const float *const tile = reinterpret_cast<const float *>(s_tile[wib]);
    for (int p0 = 0; p0 < G.P; p0 += PC) {
        const int np = min(PC, G.P - p0);
        for (int i = threadIdx.x; i < S * 4 * MT * 16; i += 256) {
            const int q = i / (MT * 16), b = i - q * (MT * 16), pose = q / 3;
            float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (pose < np && b < G.nb) o = *reinterpret_cast<const float4 *>(B + ((p0 + pose) * G.nb + b) * 12 + (q - 3 * pose) * 4);
            s_bone[q][b] = o;
        }
        v4f acc[S][MT];
        int src[S];                             // this lane's quarter of node 0 (12 P V < 2^31)
        bool have[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int q = 4 * s + kq, pose = q / 3, part4 = q - 3 * pose;
            have[s] = pose < np;
            src[s] = (p0 + (have[s] ? pose : 0)) * V * 12 + 4 * part4;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[s][mt] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
        }
        float4 g[S], w[MT];
        auto fetch = [&](int t) {
            const int v0 = t * 16;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                g[s] = *reinterpret_cast<const float4 *>(GT + src[s] + min(v0 + col, V - 1) * 12);
                if (!(have[s] && v0 + col < V)) g[s] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
            // the rows of a tile are contiguous and start at a multiple of 64 bytes
            const float *wsrc = W + (long long)v0 * G.nb;
            if (v0 + 16 <= V) {
#pragma unroll
                for (int m = 0; m < MT; ++m) w[m] = *reinterpret_cast<const float4 *>(wsrc + min((m * 64 + lane) * 4, 16 * G.nb - 4));
            } else {
                const int n = (V - v0) * G.nb;
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const int i = (m * 64 + lane) * 4;
                    w[m].x = i < n ? wsrc[i] : 0.0f;
                    w[m].y = i + 1 < n ? wsrc[i + 1] : 0.0f;
                    w[m].z = i + 2 < n ? wsrc[i + 2] : 0.0f;
                    w[m].w = i + 3 < n ? wsrc[i + 3] : 0.0f;
                }
            }
        };
        if (wave < tiles) fetch(wave);
        __syncthreads();                       // s_bone
        for (int t = wave; t < tiles; t += nwaves) {
            float wc[4][MT];
            // the wave's own part of LDS: its accesses stay in order, the fences only keep the compiler from moving them
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int s = 0; s < S; ++s) s_tile[wib][col * (ROW / 4) + 4 * s + kq] = g[s];
#pragma unroll
            for (int m = 0; m < MT; ++m) s_w[wib][m * 64 + lane] = w[m];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (t + nwaves < tiles) fetch(t + nwaves);
            const int v0 = t * 16;
            v4f gw[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                gw[mt] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int u = 0; u < 4; ++u) wc[u][mt] = tw[(4 * u + kq) * G.nb + mt * 16 + col];      // beyond n_b: sums that nobody stores
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                // one slot's reads of LDS at a time: all of them at once need more registers than there are
                if (S > 1) __builtin_amdgcn_sched_barrier(0);
                int at = 0;
                if (S > 1) asm volatile("" : "+v"(at));            // ... and the bones are read again for every tile
                const float4 g4 = s_tile[wib][col * (ROW / 4) + 4 * s + kq];
                const float gs[4] = {g4.x, g4.y, g4.z, g4.w};
                float e[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) e[u] = tile[(4 * u + kq) * ROW + 16 * s + col];
                float bs[MT][4];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const float4 b4 = s_bone[4 * s + kq + at][mt * 16 + col];
                    bs[mt][0] = b4.x; bs[mt][1] = b4.y; bs[mt][2] = b4.z; bs[mt][3] = b4.w;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        gw[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(gs[u], bs[mt][u], gw[mt], 0, 0, 0);
                        acc[s][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wc[u][mt], e[u], acc[s][mt], 0, 0, 0);
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                if (mt * 16 + col < G.nb) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) tw[(4 * kq + r) * G.nb + mt * 16 + col] = gw[mt][r];
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            float *dst = gW + (long long)v0 * G.nb;
            const int n = min(16, V - v0) * G.nb;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const int i = (m * 64 + lane) * 4;
                if (i + 4 <= n) {
                    float4 o = s_w[wib][m * 64 + lane];
                    if (p0 > 0) {                           // on top of what this lane stored in the pass before
                        const float4 before = *reinterpret_cast<const float4 *>(dst + i);
                        o.x += before.x; o.y += before.y; o.z += before.z; o.w += before.w;
                    }
                    *reinterpret_cast<float4 *>(dst + i) = o;
                } else
                    for (int j = i; j < n; ++j) dst[j] = p0 > 0 ? dst[j] + tw[j] : tw[j];
            }
        }
        // the block's 4 waves add their results in LDS, 16 columns at a time; wave 0 writes the block's partial
        int first = 4 * kq;
        asm volatile("" : "+v"(first));            // addresses are made here, not before the loop, where they would fill the registers
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (4 * s < 3 * np) {                           // the same for the whole block
                if (wib > 0) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) s_acc[wib - 1][mt][lane] = acc[s][mt];
                }
                __syncthreads();
                const int c = 16 * s + col, pose = c / 12, e = c - 12 * pose;
                if (wib == 0 && pose < np) {
                    float *o = part + ((long long)(p0 + pose) * gridDim.x + blockIdx.x) * nout;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const v4f t = acc[s][mt] + s_acc[0][mt][lane] + s_acc[1][mt][lane] + s_acc[2][mt][lane];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int b = mt * 16 + first + r;
                            if (b < G.nb) o[b * 12 + e] = t[r];
                        }
                    }
                }
                __syncthreads();
            }
        }
    }
}

// sum of the per-block partial results of k_grad_outputs: a block takes 16 outputs (64 contiguous bytes of every partial;
// a wave reads four of them), 64 threads share the partials of one (one wave per output, 4 bytes of a line per
// load: 14.7 us on 8 poses, now 4.7).
__global__ __launch_bounds__(1024) void k_grad_bones_final(int nblk, int nout, const float *__restrict__ part, float *__restrict__ gB)
{
    __shared__ float s_sum[16][16];
    const int j = threadIdx.x & 15, h = threadIdx.x >> 4, p = blockIdx.y, o = blockIdx.x * 16 + j;
    float a = 0.0f;
    if (o < nout)
        for (int b0 = h; b0 < nblk; b0 += 512) {          // eight loads on their way together
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = b0 + 64 * i < nblk ? part[((long long)p * nblk + b0 + 64 * i) * nout + o] : 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) a += v[i];
        }
    a += __shfl_xor(a, 16);
    a += __shfl_xor(a, 32);
    if ((threadIdx.x & 63) < 16) s_sum[threadIdx.x >> 6][j] = a;
    __syncthreads();
    if (threadIdx.x < 16 && o < nout) {
        a = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) a += s_sum[i][j];
        gB[p * nout + o] = a;
    }
}

// ------------------------------------------------------------------------------------------------
// Duplicate removal (Sec. 3.1 "Remove Duplicate Correspondences") and packing of the surviving roots.
// Lanes in increasing k; a converged lane is kept iff no lane kept before it is closer than min_dist.  In other words: the
// first lane not yet settled is kept and settles every later one that is closer than min_dist to it, and again, as many
// rounds as the point has distinct roots (1 to 4) instead of one per lane.
// Two launches.  The points are cut into at most DD_TILES tiles.  k_dedupe leaves what it kept of a point in offsets[n]
// (the mask itself for K <= 32, else the number) and the sum of every tile; k_dedupe_pack adds up the sums before its
// tile, scans its points and packs.
// ------------------------------------------------------------------------------------------------
constexpr int DD_TILES = 2048;

__device__ __forceinline__ bool closer(const float (&a)[3], const float (&b)[3], float md2)
{
    const float e0 = a[0] - b[0], e1 = a[1] - b[1], e2 = a[2] - b[2];
    return FS_FMA(e2, e2, FS_FMA(e1, e1, e0 * e0)) < md2;
}

// a block's sum of `mine` into sums[block]; up to four waves
__device__ __forceinline__ void tile_sum(int mine, int *__restrict__ sums)
{
    __shared__ int s_sum[4];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += s_sum[w];
        sums[blockIdx.x] = t;
    }
}

constexpr int DD_FEW = 4;
// what is kept of point n (K <= DD_FEW), by one thread with everything in registers
__device__ __forceinline__ unsigned dedupe_point(long long N, int K, long long n, float md2, const float *__restrict__ xc,
                                                 const uint8_t *__restrict__ conv, uint8_t *__restrict__ keep)
{
            bool on[DD_FEW];
            float x[DD_FEW][3];
#pragma unroll
            for (int k = 0; k < DD_FEW; ++k) on[k] = k < K && conv[(long long)min(k, K - 1) * N + n] != 0;
#pragma unroll
            for (int k = 0; k < DD_FEW; ++k)
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    x[k][r] = 0.0f;
                    if (on[k]) x[k][r] = xc[((long long)k * 3 + r) * N + n];
                }
            unsigned kept = 0u;
#pragma unroll
            for (int k = 0; k < DD_FEW; ++k) {
#pragma unroll
                for (int j = 0; j < k; ++j)
                    if (((kept >> j) & 1u) && closer(x[k], x[j], md2)) on[k] = false;
                kept |= (on[k] ? 1u : 0u) << k;
            }
#pragma unroll
    for (int k = 0; k < DD_FEW; ++k)
        if (k < K) keep[(long long)k * N + n] = (uint8_t)((kept >> k) & 1u);
    return kept;
}
// the same for the four points from n on, whose bytes and floats are read and written as words and quadruples at whatever address they lie
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32_any __attribute__((aligned(1)));
__device__ __forceinline__ int4 dedupe_four(long long N, int K, long long n, float md2, const float *__restrict__ xc,
                                            const uint8_t *__restrict__ conv, uint8_t *__restrict__ keep)
{
    unsigned on[DD_FEW];
    v4f_any x[DD_FEW][3];
#pragma unroll
    for (int k = 0; k < DD_FEW; ++k) on[k] = k < K ? *reinterpret_cast<const u32_any *>(conv + (long long)k * N + n) : 0u;
#pragma unroll
    for (int k = 0; k < DD_FEW; ++k)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            x[k][r] = (v4f_any){0.0f, 0.0f, 0.0f, 0.0f};
            if (on[k]) x[k][r] = *reinterpret_cast<const v4f_any *>(xc + ((long long)k * 3 + r) * N + n);
        }
    unsigned word[DD_FEW] = {0u, 0u, 0u, 0u};
    int kept[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned m = 0u;
#pragma unroll
        for (int k = 0; k < DD_FEW; ++k) {
            bool o = ((on[k] >> (8 * i)) & 0xffu) != 0u;
            const float a[3] = {x[k][0][i], x[k][1][i], x[k][2][i]};
#pragma unroll
            for (int j = 0; j < k; ++j) {
                const float b[3] = {x[j][0][i], x[j][1][i], x[j][2][i]};
                if (((m >> j) & 1u) && closer(a, b, md2)) o = false;
            }
            m |= (o ? 1u : 0u) << k;
            word[k] |= (o ? 1u : 0u) << (8 * i);
        }
        kept[i] = (int)m;
    }
#pragma unroll
    for (int k = 0; k < DD_FEW; ++k)
        if (k < K) *reinterpret_cast<u32_any *>(keep + (long long)k * N + n) = word[k];
    return make_int4(kept[0], kept[1], kept[2], kept[3]);
}
// PTS: points per thread and pass; 4 for large batches.  Bound: number of memory instructions, a byte per lane
// and row with one point (1 M ray samples of 3 candidates 10.2 us, with four 6.8; k_dedupe_pack with four, whose roots are then apart, 8.7 instead of 8.0).
template <int PTS>
__global__ __launch_bounds__(256) void k_dedupe_few(long long N, int K, float md2, const float *__restrict__ xc,
                                                    const uint8_t *__restrict__ conv, uint8_t *__restrict__ keep,
                                                    int *__restrict__ offsets, int tile, int *__restrict__ sums)
{
    const long long n0 = (long long)blockIdx.x * tile, n1 = min(N, n0 + tile);
    int mine = 0;
    for (long long n = n0 + threadIdx.x * PTS; n < n1; n += blockDim.x * PTS) {
        if (PTS == 4 && n + 4 <= n1) {
            const int4 kept = dedupe_four(N, K, n, md2, xc, conv, keep);
            *reinterpret_cast<int4 *>(offsets + n) = kept;
            mine += __popc(kept.x) + __popc(kept.y) + __popc(kept.z) + __popc(kept.w);
        } else {
            for (long long i = n; i < min(n1, n + PTS); ++i) {
                const unsigned kept = dedupe_point(N, K, i, md2, xc, conv, keep);
                offsets[i] = (int)kept;
                mine += __popc(kept);
            }
        }
    }
    tile_sum(mine, sums);
}

// Eight threads per point: SIMD lane 8 g + i holds lanes k = g, 8 + g, ... (at most 8 T) of the i-th of the wave's 8 points,
// so that all loads of a point travel together.  Returns what is kept of the point, bit k for lane k (wave-wide call).
// Bound: memory (13 bytes per lane) on large batches, two round trips and the launch on small ones.  (One thread per point
// and lane after lane, kept roots read again for every comparison: 48 us on 200,000 points x 24 lanes, 19 us on 37; now
// 21 and 4.5.)
template <int T>
__device__ __forceinline__ u64 dedupe_points(long long N, int K, long long n, bool live, float md2, const float *__restrict__ xc,
                                             const uint8_t *__restrict__ conv, uint8_t *__restrict__ keep)
{
    const int lane = threadIdx.x & 63, i = lane & 7, g = lane >> 3;
    const u64 point = 0x0101010101010101ull << i;        // the SIMD lanes of this lane's point
    unsigned open = 0u, kept = 0u;          // bit t: lane 8 t + g of the point
#pragma unroll
    for (int t = 0; t < T; ++t)
        if (8 * t + g < K && live) open |= (conv[(long long)(8 * t + g) * N + n] != 0 ? 1u : 0u) << t;
    float x[T][3];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            x[t][r] = 0.0f;
            if ((open >> t) & 1u) x[t][r] = xc[((long long)(8 * t + g) * 3 + r) * N + n];
        }
    while (__any(open != 0u)) {
        // the point's first open lane: slot ft of SIMD lane src
        int ft = 0, src = lane;
        bool found = false;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const unsigned long long m = __ballot((open >> t) & 1u) & point;
            if (!found && m) {
                found = true;
                ft = t;
                src = __ffsll((long long)m) - 1;
            }
        }
        float y[3] = {x[0][0], x[0][1], x[0][2]}, c[3];
#pragma unroll
        for (int t = 1; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 3; ++r) y[r] = ft == t ? x[t][r] : y[r];      // ft is the same in all lanes of the point
#pragma unroll
        for (int r = 0; r < 3; ++r) c[r] = __shfl(y[r], src);
        if (found) {
            if (lane == src) {
                kept |= 1u << ft;
                open &= ~(1u << ft);
            }
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (closer(x[t], c, md2)) open &= ~(1u << t);
        }
    }
    u64 mask = 0ull;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const unsigned long long m = __ballot((kept >> t) & 1u) & point;
        // the bits of the point's 8 lanes, 8 places apart, side by side
        mask |= (((m >> i) * 0x0102040810204080ull) >> 56) << (8 * t);
        if (8 * t + g < K && live) keep[(long long)(8 * t + g) * N + n] = (uint8_t)((kept >> t) & 1u);
    }
    return mask;
}
template <int T>
__global__ __launch_bounds__(256) void k_dedupe(long long N, int K, float md2, const float *__restrict__ xc,
                                                const uint8_t *__restrict__ conv, uint8_t *__restrict__ keep,
                                                int *__restrict__ offsets, int tile, int *__restrict__ sums)
{
    const int lane = threadIdx.x & 63, i = lane & 7, g = lane >> 3;
    const long long n0 = (long long)blockIdx.x * tile, n1 = min(N, n0 + tile);
    int mine = 0;
    for (long long b = n0 + (threadIdx.x >> 6) * 8; b < n1; b += 32) {  // wave-uniform
        const long long n = min(b + i, n1 - 1);
        const u64 kept = dedupe_points<T>(N, K, n, b + i < n1, md2, xc, conv, keep);
        if (g == 0 && b + i < n1) {
            offsets[n] = K <= 32 ? (int)(unsigned)kept : __popcll(kept);
            mine += __popcll(kept);
        }
    }
    tile_sum(mine, sums);
}

// The kept roots of point n, bits of m, from place o of the packed list on (entries from cap on are left out)
__device__ __forceinline__ void pack_point(long long N, long long cap, long long n, u64 m, long long o, const float *__restrict__ xc,
                                           float *__restrict__ roots, int32_t *__restrict__ lane)
{
    for (; m && o < cap; m &= m - 1ull, ++o) {
        const int k = __builtin_ctzll(m);
        if (roots) {
            roots[o * 3 + 0] = xc[((long long)k * 3 + 0) * N + n];
            roots[o * 3 + 1] = xc[((long long)k * 3 + 1) * N + n];
            roots[o * 3 + 2] = xc[((long long)k * 3 + 2) * N + n];
        }
        if (lane) lane[o] = k;
    }
}

// Removal and packing in one launch: a block takes 1024 points (T = 0, K <= DD_FEW) or 128 (K <= 8 T), keeps what it found of them in registers or
// LDS, and learns by tickets and look-back (k_scan) how much the blocks before it kept.  A single block asks nobody.
// look: the words of this kernel alone, its own last block clears them (look_finish).
// Bound: latency of launch, loads and look-back; where it is launched, and its times, see launch_dedupe_one.
template <int T>
__global__ __launch_bounds__(1024) void k_dedupe_one(long long N, int K, long long cap, float md2, const float *__restrict__ xc,
                                                     const uint8_t *__restrict__ conv, uint8_t *__restrict__ keep,
                                                     int *__restrict__ offsets, float *__restrict__ roots, int32_t *__restrict__ lane_out,
                                                     u64 *__restrict__ look)
{
    constexpr int PTS = T == 0 ? 1024 : 128;
    __shared__ u64 s_mask[T == 0 ? 1 : PTS];
    __shared__ int s_tot[16], s_before;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, ticket = gridDim.x > 1 ? look_ticket(look) : 0;
    const long long n0 = (long long)ticket * PTS, n = n0 + threadIdx.x;
    const bool mine = threadIdx.x < PTS && n < N;             // the point that this thread packs
    u64 kept = 0ull;
    if constexpr (T == 0) {
        if (mine) kept = dedupe_point(N, K, n, md2, xc, conv, keep);
    } else {
        const int i = wid * 8 + (lane & 7);
        const u64 m = dedupe_points<T>(N, K, min(n0 + i, N - 1), n0 + i < N, md2, xc, conv, keep);
        if (lane < 8) s_mask[i] = m;
        __syncthreads();
        if (mine) kept = s_mask[threadIdx.x];
    }
    const int c = __popcll(kept);
    int inc = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
    }
    if (lane == 63) s_tot[wid] = inc;
    __syncthreads();
    if (wid == 0) {
        const int sum = scan_totals(s_tot, 16, lane), before = gridDim.x > 1 ? look_back(look, ticket, sum, lane) : 0;
        if (lane == 0) {
            s_before = before;
            if (ticket == (int)gridDim.x - 1) offsets[N] = before + sum;
        }
    }
    __syncthreads();
    if (mine) {
        const int o = s_before + s_tot[wid] + inc - c;
        offsets[n] = o;
        if (roots || lane_out) pack_point(N, cap, n, kept, o, xc, roots, lane_out);
    }
    if (gridDim.x > 1 && wid == 0) look_finish(look, (int)gridDim.x, lane);
}

// offsets and the packed list: roots [total][3] and lane index k, point n owns entries offsets[n] .. offsets[n+1]
__global__ __launch_bounds__(256) void k_dedupe_pack(long long N, int K, long long cap, const float *__restrict__ xc,
                                                     const uint8_t *__restrict__ keep, int *__restrict__ offsets, int tile,
                                                     const int *__restrict__ sums, float *__restrict__ roots,
                                                     int32_t *__restrict__ lane)
{
    __shared__ int s_sum[4];
    const int wid = threadIdx.x >> 6, l = threadIdx.x & 63;
    int before = 0;
    for (int j = threadIdx.x; j < (int)blockIdx.x; j += 256) before += sums[j];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) before += __shfl_xor(before, d);
    if (l == 0) s_sum[wid] = before;
    __syncthreads();
    int run = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
    const long long n0 = (long long)blockIdx.x * tile, n1 = min(N, n0 + tile);
    for (long long b = n0; b < n1; b += 256) {
        const long long n = b + threadIdx.x;
        const int info = n < n1 ? offsets[n] : 0;
        const int c = K <= 32 ? __popc((unsigned)info) : info;
        int inc = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(inc, d);
            if (l >= d) inc += o;
        }
        __syncthreads();                     // s_sum is still read for the step before
        if (l == 63) s_sum[wid] = inc;
        __syncthreads();
        const int t0 = s_sum[0], t1 = s_sum[1], t2 = s_sum[2], t3 = s_sum[3];
        const int at = run + inc - c + (wid > 0 ? t0 : 0) + (wid > 1 ? t1 : 0) + (wid > 2 ? t2 : 0);
        run += t0 + t1 + t2 + t3;
        if (n >= n1) continue;
        offsets[n] = at;
        if (!roots && !lane) continue;
        const long long o = at;
        unsigned long long m = (unsigned)info;
        if (K > 32) {
            m = 0ull;
            if (c > 0)
                for (int k = 0; k < K; ++k) m |= (unsigned long long)(keep[(long long)k * N + n] != 0) << k;
        }
        pack_point(N, cap, n, m, o, xc, roots, lane);
    }
    if (threadIdx.x == 0 && n1 == N) offsets[N] = run;
}

}  // namespace fs
