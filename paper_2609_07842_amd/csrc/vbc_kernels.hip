// vbc_kernels.hip -- gfx950 kernels of the VBC hot path.
//
// Passes (Section 2, paragraph on the cost of the correction: a count sweep and a force
// sweep of the neighbour list; the force itself follows from differentiating eq. (Vhat)):
//   count  : n_i = sum_j omega(r_ij, r_l, r_h)                       eq. (counter)
//            s_i = omega(n_i, f - delta, f - delta + 1)              eq. (Psi), (Psidelta)
//   embed  : A_i = dU/dn_i = s'_i sum_j s_j V_a(r_ij), only for particles whose count lies
//            inside the switching window (elsewhere s'_i = 0); a workgroup whose brick holds
//            no such particle exits at once
//   force  : phi_ij = V_r'(r) + s_i s_j V_a'(r) + (A_i + A_j) c'(r),  F_i = -sum_j phi_ij r_hat_ij
//            plus the integrator update of the particle, fused in the same pass.
// The energy gradient needs A of every counted neighbour, which is only final once all
// counts are, hence the separate sparse embed pass between the two list sweeps.
//
// List build (when some particle has moved more than half the buffer): every workgroup
// gathers the particles now inside its brick from the one-cell halo of the previous
// layout, orders them by (cell, tag) in LDS and writes the next layout; a second kernel
// copies each brick to the live arrays and builds its list.  Starting from unsorted input
// (after vbc_set_state), particles are first binned into per-brick buckets with atomics.
//
// Data flow of one workgroup in a pass: it owns one brick; it stages its own particles and
// the halo into LDS in a brick-local frame, then sweeps each own particle's list (16-bit
// indices into the staging order, eight per 16-byte chunk) reading neighbours from LDS.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <tuple>

#include "vbc_internal.h"

namespace vbc {

#define VBC_WAVE 64
#define VBC_GROUP 8  // lanes that copy one cell during staging

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

template <class T> struct V4;
template <> struct V4<float> { using t = float4; };
template <> struct V4<double> { using t = double4; };
template <class T> struct V2;
template <> struct V2<float> { using t = float2; };
template <> struct V2<double> { using t = double2; };

// Pair arithmetic: the hardware square root and reciprocal square root in FP32 (<= 1 ulp),
// the exactly rounded ones in FP64.
__device__ __forceinline__ float rsqrt_r(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsqrt_r(double x) { return 1.0 / sqrt(x); }
__device__ __forceinline__ float sqrt_r(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double sqrt_r(double x) { return sqrt(x); }
__device__ __forceinline__ float clamp01(float u) { return __builtin_amdgcn_fmed3f(u, 0.0f, 1.0f); }
__device__ __forceinline__ double clamp01(double u) { return fmin(fmax(u, 0.0), 1.0); }

// Map workgroups to bricks so that consecutive bricks (which share halo cells) land on
// the same XCD: workgroups are dealt round-robin over the 8 XCDs, so workgroup g runs on
// XCD g % 8; give that XCD a contiguous run of the T bricks to visit.  The grid is padded
// to a multiple of 8, at least T.  The bricks are either the contiguous range
// [b_lo, b_lo + nb_launch) (P.list < 0: all bricks, or one replica's) or the entries of
// work list P.list, which the step computes on the GPU.  Returns false for a workgroup
// with nothing to do (padding, or a free brick).
__device__ __forceinline__ bool brick_of_block(const Launch &P, const Buffers &B, int &b)
{
    const int g = blockIdx.x, j = g >> 3;
    const int T = P.list < 0 ? P.nb_launch : B.wl_n[P.list];
    const int chunk = (T + 7) >> 3;
    const int k = (g & 7) * chunk + j;
    if (j >= chunk || k >= T) return false;
    b = P.list < 0 ? P.b_lo + k : B.wl[P.list][k];
    return true;
}

__device__ __forceinline__ bool resolve_brick(const Launch &P, const Buffers &B, int &b, int &r)
{
    if (!brick_of_block(P, B, b)) return false;
    r = B.brick_rep[b];
    return r >= 0;
}

// The second of two launches of a pass (see parts): a workgroup looks at up to 64 bricks, far
// apart, and does those with more than t_lo staged particles one after the other.  The grid is
// as many workgroups as the chip holds at once (dense_grid): one per brick, with the full
// capacity's LDS, would need as many rounds of the chip to find nothing to do as the pass takes
// in all.  The mask is a scalar, the same in every wave.
constexpr int DENSE_BLOCK = 512;  // at most so many threads: their registers are not what limits them
template <class F>
__device__ __forceinline__ void each_dense(const Launch &P, const Buffers &B, F &&body)
{
    const int T = P.list < 0 ? P.nb_launch : B.wl_n[P.list];
    const int lane = threadIdx.x % VBC_WAVE, kl = blockIdx.x + lane * gridDim.x;
    bool dense = false;
    if (kl < T) dense = B.stotal[P.list < 0 ? P.b_lo + kl : B.wl[P.list][kl]] > P.t_lo;
    uint64_t mask = __ballot(dense);
    while (mask) {
        const int k = blockIdx.x + __builtin_ctzll(mask) * gridDim.x;
        mask &= mask - 1;
        body(P.list < 0 ? P.b_lo + k : B.wl[P.list][k]);
        __syncthreads();
    }
}

// Smooth step of eq. (omega) and its derivative, in FP64 (used for the switching factor).
__device__ __forceinline__ double omega_d64(double x, double x1, double x2)
{
    if (x <= x1) return 1.0;
    if (x >= x2) return 0.0;
    double u = (x - x1) / (x2 - x1);
    double q = 1.0 - u * u;
    return q * q;
}

__device__ __forceinline__ double omega_dd64(double x, double x1, double x2)
{
    if (x <= x1 || x >= x2) return 0.0;
    double w = x2 - x1;
    double u = (x - x1) / w;
    return -4.0 * u * (1.0 - u * u) / w;
}

// Smooth step of eq. (omega) over the unit-width switching window [x1, x1 + 1] of
// eq. (Psidelta), in the pair-arithmetic precision.
template <class Real>
__device__ __forceinline__ Real omega_win(Real x, Real x1)
{
    const Real u = clamp01(x - x1), q = fma(-u, u, Real(1));
    return q * q;
}

// Philox4x32 with 10 rounds (Salmon, Moraes, Dror & Shaw, SC'11): two 32x32->64-bit
// multiplies by fixed odd constants per round, high halves xor-ed with the other two
// counter words and the round key; the key is bumped by two Weyl constants per round.
__device__ __forceinline__ void philox4x32_10(uint32_t &c0, uint32_t &c1, uint32_t &c2,
                                              uint32_t &c3, uint32_t k0, uint32_t k1)
{
    const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
    const uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += W0;
            k1 += W1;
        }
        // one 32x32->64-bit product each (a single multiply instruction for both halves)
        const uint64_t p0 = (uint64_t)M0 * c0, p1 = (uint64_t)M1 * c2;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        uint32_t n0 = hi1 ^ c1 ^ k0;
        uint32_t n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
}

// Zero-mean unit-variance uniform variates sqrt(3)(2u - 1) from the first three words,
// u = (word + 1/2) 2^-32; key = the halves of seed, counter = the halves of step, then of
// tag: only exactly rounded operations.
__device__ __forceinline__ void langevin_noise(uint64_t seed, uint64_t tag, uint64_t step,
                                               double xi[3])
{
#pragma clang fp contract(off)
    uint32_t c0 = (uint32_t)step, c1 = (uint32_t)(step >> 32), c2 = (uint32_t)tag,
             c3 = (uint32_t)(tag >> 32);
    philox4x32_10(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
    const double SQRT3 = 1.7320508075688772;
    xi[0] = (2.0 * (((double)c0 + 0.5) * 0x1.0p-32) - 1.0) * SQRT3;
    xi[1] = (2.0 * (((double)c1 + 0.5) * 0x1.0p-32) - 1.0) * SQRT3;
    xi[2] = (2.0 * (((double)c2 + 0.5) * 0x1.0p-32) - 1.0) * SQRT3;
}

template <class T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int o = VBC_WAVE / 2; o > 0; o >>= 1) v += __shfl_down(v, o, VBC_WAVE);
    return v;
}

// Eight sums over the wave at once.  At each of the first three halvings a lane keeps half
// of its values and trades the other half with the lane 32, 16 or 8 away, so that from
// then on every lane carries one value, which three more exchanges finish: ten shuffles
// instead of the 48 of eight separate sums.  Returns, in lane L, the total of value
// 4 b5 + 2 b4 + b3 (the bits of L): value k's total is in lane 8k.  The order of the
// additions is fixed.
__device__ __forceinline__ double wave_sum8(const double (&a)[8])
{
    const int lane = threadIdx.x % VBC_WAVE;
    double s[4], t[2];
    bool hi = lane & 32;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double keep = hi ? a[k + 4] : a[k], give = hi ? a[k] : a[k + 4];
        s[k] = keep + __shfl_xor(give, 32, VBC_WAVE);
    }
    hi = lane & 16;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double keep = hi ? s[k + 2] : s[k], give = hi ? s[k] : s[k + 2];
        t[k] = keep + __shfl_xor(give, 16, VBC_WAVE);
    }
    hi = lane & 8;
    double u = (hi ? t[1] : t[0]) + __shfl_xor(hi ? t[0] : t[1], 8, VBC_WAVE);
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) u += __shfl_xor(u, o, VBC_WAVE);
    return u;
}

// Sum of v over this and the lower lanes of the wave: shifts within rows of sixteen, then the
// last lane of each row and of the lower half handed up, all in the vector unit (the same by
// lane shuffles through LDS took 1.2 us for 216 cells).
__device__ __forceinline__ int wave_inclusive_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Exclusive scan of a[0..n) in place by one whole wave; the total.
__device__ __forceinline__ int wave_exclusive_scan(int *a, int n)
{
    const int lane = threadIdx.x % VBC_WAVE;
    int carry = 0;
    for (int base = 0; base < n; base += VBC_WAVE) {
        const int q = base + lane;
        const int v = q < n ? a[q] : 0;
        const int incl = wave_inclusive_sum(v);
        if (q < n) a[q] = carry + incl - v;
        carry += __builtin_amdgcn_readlane(incl, VBC_WAVE - 1);
    }
    return carry;
}

// The same by the first wave, which gets the total.  Call from all threads of the block between
// barriers.
__device__ __forceinline__ int wave0_exclusive_scan(int *a, int n)
{
    return threadIdx.x < VBC_WAVE ? wave_exclusive_scan(a, n) : 0;
}

// Wrap one coordinate into [0, L).
__device__ __forceinline__ double wrap1(double t, double L)
{
    if (t < 0.0 || t >= L) {
        t = t - L * floor(t / L);
        if (t >= L) t -= L;
        if (t < 0.0) t = 0.0;
    }
    return t;
}

__device__ __forceinline__ int cell_of(double t, double h, int nc)
{
    int c = (int)floor(t / h);
    return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

// ---------------------------------------------------------------------------
// brick geometry and staging
// ---------------------------------------------------------------------------

struct StageHdr {
    int64_t base;   // first slot of the brick
    int n_own;
    int total;
    int rank0;
    int nh, ncb;
    int c0[3], e[3], H[3];
    double O[3];
    int overflow;
};

struct StageTabs {
    int *q_off;    // staged offset of each halo-grid cell (own and halo)
    int *q_cnt;    // particles in the cell
    int *q_src;    // first slot of the cell
    int *q_hpre;   // exclusive prefix of halo-cell counts (own cells contribute 0)
    int *q_w;      // packed image shift (wx+1) | (wy+1) << 2 | (wz+1) << 4
};

__device__ __forceinline__ int unpack_w(int w, int a) { return ((w >> (2 * a)) & 3) - 1; }

__device__ __forceinline__ size_t align32(size_t b) { return (b + 31) & ~(size_t)31; }

__device__ __forceinline__ StageTabs carve_tabs(unsigned char *smem, int nh_cap)
{
    StageTabs T;
    int *p = (int *)smem;
    T.q_off = p;
    T.q_cnt = p + nh_cap;
    T.q_src = p + 2 * nh_cap;
    T.q_hpre = p + 3 * nh_cap;
    T.q_w = p + 4 * nh_cap;
    return T;
}

__device__ __forceinline__ unsigned char *after_tabs(unsigned char *smem, int nh_cap)
{
    return smem + align32((size_t)5 * nh_cap * sizeof(int));
}

// Geometry of brick lb of replica R (one thread).
__device__ __forceinline__ void brick_geometry(const RepDev &R, int lb, StageHdr &S)
{
    int Bc[3] = {lb % R.nb[0], (lb / R.nb[0]) % R.nb[1], lb / (R.nb[0] * R.nb[1])};
    S.ncb = 1;
    for (int a = 0; a < 3; ++a) {
        S.c0[a] = Bc[a] * R.bd[a];
        S.e[a] = min(R.bd[a], R.nc[a] - S.c0[a]);
        S.H[a] = S.e[a] + 2;
        S.ncb *= S.e[a];
        S.O[a] = ((double)S.c0[a] + 0.5 * (double)S.e[a]) * R.h[a];
    }
    S.nh = S.H[0] * S.H[1] * S.H[2];
    S.base = R.p_off + (int64_t)lb * R.bcap;
}

// The cells of a brick's halo grid: first slot, count, image shift, staged offset of the own
// ones (-1: halo) and the halo counts; all: every cell's count, if asked.
__device__ __forceinline__ void stage_cells(const RepDev &R, const StageHdr &S, const int32_t *cell_rank,
                                            const int32_t *cstart, const int32_t *ccnt, StageTabs T,
                                            int *all)
{
    for (int q = threadIdx.x; q < S.nh; q += blockDim.x) {
        int h[3] = {q % S.H[0], (q / S.H[0]) % S.H[1], q / (S.H[0] * S.H[1])};
        int g[3], w = 0;
        bool own = true;
        for (int a = 0; a < 3; ++a) {
            int ga = S.c0[a] - 1 + h[a];
            int wa = ga < 0 ? -1 : (ga >= R.nc[a] ? 1 : 0);
            g[a] = ga - wa * R.nc[a];
            w |= (wa + 1) << (2 * a);
            own = own && (h[a] >= 1 && h[a] <= S.e[a]);
        }
        int rank = cell_rank[R.c_off + g[0] + R.nc[0] * (g[1] + R.nc[1] * g[2])];
        int st = cstart[R.c_off + rank];
        int cnt = ccnt[R.c_off + rank];
        T.q_src[q] = st;
        T.q_cnt[q] = cnt;
        T.q_w[q] = w;
        T.q_off[q] = own ? (int)(st - S.base) : -1;
        T.q_hpre[q] = own ? 0 : cnt;
        if (all) all[q] = cnt;
    }
}

// Lay out the staging of brick b (local index lb) of replica R from a set of cell tables:
// own particles first (the brick's slot range), then every halo cell of the (e+2)^3 grid
// in x-fastest order.  All threads of the block call this.
__device__ void stage_tables(const RepDev &R, int b, int lb, const int32_t *brick_rank0,
                             const int32_t *cell_rank, const int32_t *cstart,
                             const int32_t *ccnt, const int32_t *bcnt, StageHdr &S,
                             StageTabs T, int stage_cap)
{
    if (threadIdx.x == 0) {
        brick_geometry(R, lb, S);
        S.rank0 = brick_rank0[b];
        S.n_own = bcnt[b];
    }
    __syncthreads();
    stage_cells(R, S, cell_rank, cstart, ccnt, T, nullptr);
    __syncthreads();
    int tot = wave0_exclusive_scan(T.q_hpre, S.nh);
    if (threadIdx.x == 0) {
        S.total = S.n_own + tot;
        S.overflow = S.total > stage_cap;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < S.nh; q += blockDim.x)
        if (T.q_off[q] < 0) T.q_off[q] = S.n_own + T.q_hpre[q];
    __syncthreads();
}

// Call fn(staged_slot, source_slot, packed_shift) for every staged particle.  Groups of
// eight lanes take one cell at a time, so no search is needed and the loads of all cells
// are in flight together.
template <class F>
__device__ __forceinline__ void stage_copy(const StageHdr &S, const StageTabs &T, F &&fn)
{
    int gid = threadIdx.x / VBC_GROUP, gl = threadIdx.x % VBC_GROUP;
    int ng = blockDim.x / VBC_GROUP;
    for (int q = gid; q < S.nh; q += ng) {
        int off = T.q_off[q], src = T.q_src[q], cnt = T.q_cnt[q], w = T.q_w[q];
        for (int k = gl; k < cnt; k += VBC_GROUP) fn(off + k, src + k, w);
    }
}

// Header of brick b for a pass over the current layout: geometry, own range and the
// staged count recorded by the last list build (one thread).
__device__ __forceinline__ void pass_header(const RepDev &R, const Buffers &B, int b, int lb,
                                            int stage_cap, StageHdr &S)
{
    brick_geometry(R, lb, S);
    S.n_own = B.bcnt[0][b];
    S.total = B.stotal[b];
    S.overflow = S.total > stage_cap;
}

// Every particle staged by brick b, from the staging map the list build recorded (one
// coalesced read, no cell-table walk), four per thread at a time: the map reads of all four go
// out first, then fn(staged_slot, source_slot, packed_shift, valid) for each; fn must do
// its own loads unconditionally (the indices are clamped into the staging) and guard only
// its stores with valid, so that the gathers of the four overlap.
//
// The map entries of the first four (threadIdx.x + j blockDim.x) are read by map_prefetch
// as soon as the brick is known, before its header: their latency then overlaps the
// header's, and the gathers can go out as soon as the header is known.  Entries past the
// staged count are stale but valid slot indices (the map is cleared at creation and only
// ever holds slots), and their stores are not made.
struct MapFirst {
    int src[4], w[4];
};

__device__ __forceinline__ MapFirst map_prefetch(const Buffers &B, int b, int stage_cap)
{
    const int32_t *sm = B.smap + (size_t)b * stage_cap;
    const uint8_t *wm = B.wmap + (size_t)b * stage_cap;
    MapFirst m;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = min((int)(threadIdx.x + j * blockDim.x), stage_cap - 1);
        m.src[j] = sm[t];
        m.w[j] = (int)wm[t];
    }
    return m;
}

template <class F>
__device__ __forceinline__ void stage_map4(const Buffers &B, int b, int stage_cap, const StageHdr &S,
                                           const MapFirst &first, F &&fn)
{
    const int32_t *sm = B.smap + (size_t)b * stage_cap;
    const uint8_t *wm = B.wmap + (size_t)b * stage_cap;
    const int nt = blockDim.x, last = S.total - 1;
    for (int t0 = threadIdx.x; t0 < S.total; t0 += 4 * nt) {
        int src[4], w[4];
        if (t0 == (int)threadIdx.x) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                src[j] = first.src[j];
                w[j] = first.w[j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = min(t0 + j * nt, last);
                src[j] = sm[t];
                w[j] = (int)wm[t];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) fn(t0 + j * nt, src[j], w[j], t0 + j * nt < S.total);
    }
}

// ---------------------------------------------------------------------------
// state in / out, flags
// ---------------------------------------------------------------------------

// Caller-order input of replica r (element tag at in_off + tag of each stride-in_stride
// component array) into the live arrays at slot p_off + tag: the unsorted layout that the
// next full build starts from.
__device__ __forceinline__ void put_state(const Buffers &B, const RepDev &R, int64_t S_, int cur, int r,
                                          int64_t tg, int64_t in_off, int64_t in_stride,
                                          const double *__restrict__ x, const double *__restrict__ v,
                                          const int32_t *__restrict__ type, uint64_t step0)
{
    int64_t i = in_off + tg;
    int64_t d = R.p_off + tg;
    for (int a = 0; a < 3; ++a) {
        B.x[cur][3 * d + a] = x[a * in_stride + i];
        B.v[a * S_ + d] = v ? v[a * in_stride + i] : 0.0;
    }
    B.tag[d] = (int32_t)tg;
    int ty = type ? type[i] : 0;
    B.type[d] = (ty >= 0 && ty < R.ntypes) ? ty : 0;
    if (tg == 0) {
        B.step[r] = step0;
        B.flags[r] = VBC_FLAG_REBUILD | FLAG_FULL;
    }
}

__global__ void k_set_state(Buffers B, int64_t S_, int cur, int r, int64_t in_off,
                            int64_t in_stride, const double *__restrict__ x,
                            const double *__restrict__ v, const int32_t *__restrict__ type,
                            uint64_t step0)
{
    const RepDev &R = B.reps[r];
    int64_t tg = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tg >= R.n) return;
    put_state(B, R, S_, cur, r, tg, in_off, in_stride, x, v, type, step0);
}

// Every live replica at once: the workgroup of brick b takes the tags whose unsorted slots
// fall in the brick's slot range (a replica has at least as many slots as particles).  One
// launch for all replicas: one for each cost 2.6 us apiece, 2.6 ms for a handle of 1024.
__global__ void k_set_state_all(Buffers B, int64_t S_, int cur, int64_t in_stride,
                                const double *__restrict__ x, const double *__restrict__ v,
                                const int32_t *__restrict__ type, uint64_t step0)
{
    const int b = blockIdx.x, r = B.brick_rep[b];
    if (r < 0) return;
    const RepDev &R = B.reps[r];
    const int64_t t0 = (int64_t)(b - R.b_off) * R.bcap, t1 = min(t0 + R.bcap, R.n);
    for (int64_t tg = t0 + threadIdx.x; tg < t1; tg += blockDim.x)
        put_state(B, R, S_, cur, r, tg, R.o_off, in_stride, x, v, type, step0);
}

// Live state of the particle at slot out in caller order (element out_off + tag).
__device__ __forceinline__ void take_state(const Buffers &B, const RepDev &R, int64_t S_, int cur, int64_t slot,
                                           int64_t out_off, int64_t out_stride, double *__restrict__ x,
                                           double *__restrict__ v)
{
    int64_t dst = out_off + B.tag[slot];
    for (int a = 0; a < 3; ++a) {
        if (x) x[a * out_stride + dst] = wrap1(B.x[cur][3 * slot + a], R.L[a]);
        if (v) v[a * out_stride + dst] = B.v[a * S_ + slot];
    }
}

// Replica r.
__global__ void k_get_state(Buffers B, int64_t S_, int cur, int r, int64_t out_off,
                            int64_t out_stride, double *__restrict__ x, double *__restrict__ v)
{
    const RepDev &R = B.reps[r];
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)R.nbrick * R.bcap) return;
    int lb = (int)(k / R.bcap);
    // before a full build and after resident steps the particles stand in caller order
    if (B.flags[r] & FLAG_FULL) {
        if (k >= R.n) return;
    } else if (k - (int64_t)lb * R.bcap >= B.bcnt[0][R.b_off + lb]) {
        return;
    }
    take_state(B, R, S_, cur, R.p_off + k, out_off, out_stride, x, v);
}

// The state of one large replica by way of records in caller order.  A particle's six
// coordinates go to six places far apart in the caller's arrays, a line of memory each; with
// hundreds of thousands of particles that bounds the read (a million: 83 us for 100 MB).
// Written as two records of 24 bytes into space that a brick replica leaves free between list
// builds (xref, and vs, the next layout's velocities), a third as many lines are touched, and a second pass spreads the records into the arrays in order.
__global__ void k_get_records(Buffers B, int64_t S_, int cur, int r)
{
    const RepDev &R = B.reps[r];
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)R.nbrick * R.bcap) return;
    const int lb = (int)(k / R.bcap);
    if (k - (int64_t)lb * R.bcap >= B.bcnt[0][R.b_off + lb]) return;
    const int64_t i = R.p_off + k;
    const int64_t c = 3 * (R.p_off + B.tag[i]);
    double x[3], v[3];
    for (int a = 0; a < 3; ++a) {
        x[a] = wrap1(B.x[cur][3 * i + a], R.L[a]);
        v[a] = B.v[a * S_ + i];
    }
    for (int a = 0; a < 3; ++a) {
        B.xref[c + a] = x[a];
        B.vs[c + a] = v[a];
    }
}

__global__ void k_put_records(Buffers B, int r, int64_t out_off, int64_t out_stride, double *__restrict__ x,
                              double *__restrict__ v)
{
    const RepDev &R = B.reps[r];
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= R.n) return;
    const double *xr = B.xref + 3 * (R.p_off + t), *vr = B.vs + 3 * (R.p_off + t);
    for (int a = 0; a < 3; ++a) {
        if (x) x[a * out_stride + out_off + t] = xr[a];
        if (v) v[a * out_stride + out_off + t] = vr[a];
    }
}

// Every live replica at once, a workgroup per brick (a launch per replica: 4.6 us each, a
// twelfth of a ten-step call of 32 replicas).
__global__ void k_get_state_all(Buffers B, int64_t S_, int cur, int64_t out_stride, double *__restrict__ x,
                                double *__restrict__ v)
{
    const int b = blockIdx.x, r = B.brick_rep[b];
    int n = B.bcnt[0][b];
    if (r < 0) return;
    const RepDev &R = B.reps[r];
    const int64_t k0 = (int64_t)(b - R.b_off) * R.bcap, base = R.p_off + k0;
    if (B.flags[r] & FLAG_FULL) n = (int)min((int64_t)R.bcap, R.n - k0);  // caller order
    for (int t = threadIdx.x; t < n; t += blockDim.x)
        take_state(B, R, S_, cur, base + t, R.o_off, out_stride, x, v);
}

__global__ void k_flags(Buffers B, int r_lo, int r_n, uint32_t bits, int set)
{
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= r_n) return;
    r += r_lo;
    if (set) B.flags[r] |= bits; else B.flags[r] &= ~bits;
}

// The replicas that a full build has just built are no longer due.
__global__ void k_full_done(Buffers B, int r_lo, int r_n)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x, r = r_lo + k;
    if (k < r_n && (B.flags[r] & FLAG_FULL)) B.flags[r] &= ~(uint32_t)(VBC_FLAG_REBUILD | FLAG_FULL | FLAG_RES);
}

// Rank of a cell in the brick-major order (bricks x-fastest, cells x-fastest inside a
// brick; edge bricks are cut by the box): every brick before brick (bx, by, bz) covers,
// whole, the z-slabs below its first cell, the rows below it in its own slab and the
// columns before it in its own row.
__device__ __forceinline__ int32_t brick_major_rank(const RepDev &R, const int g[3])
{
    int c0[3], e[3], l[3];
    for (int a = 0; a < 3; ++a) {
        c0[a] = g[a] / R.bd[a] * R.bd[a];
        e[a] = min(R.bd[a], R.nc[a] - c0[a]);
        l[a] = g[a] - c0[a];
    }
    int64_t rank0 = (int64_t)c0[2] * R.nc[0] * R.nc[1] + (int64_t)c0[1] * R.nc[0] * e[2] +
                    (int64_t)c0[0] * e[1] * e[2];
    return (int32_t)(rank0 + l[0] + e[0] * (l[1] + e[1] * l[2]));
}

// A replica enters the workspace: its static tables (brick owner, brick-major cell ranks)
// and cleared per-brick, per-cell and per-replica state.
__global__ void k_admit(Buffers B, int r)
{
    const RepDev &R = B.reps[r];
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < R.nbrick) {
        int lb = (int)t, b = R.b_off + lb;
        int g[3] = {lb % R.nb[0] * R.bd[0], lb / R.nb[0] % R.nb[1] * R.bd[1],
                    lb / (R.nb[0] * R.nb[1]) * R.bd[2]};
        B.brick_rep[b] = r;
        B.brick_rank0[b] = brick_major_rank(R, g);
        B.bcnt[0][b] = 0;
        B.bcnt[1][b] = 0;
        B.bfill[b] = 0;
        B.stotal[b] = 0;
        B.wcnt[b] = 0;
        for (int k = 0; k < 8; ++k) B.part[(size_t)b * 8 + k] = 0.0;
        B.bevals[b] = 0ull;
        B.bentries[b] = 0u;
    }
    if (t < R.ncell) {
        int c = (int)t;
        int g[3] = {c % R.nc[0], c / R.nc[0] % R.nc[1], c / (R.nc[0] * R.nc[1])};
        int64_t k = R.c_off + c;
        B.cell_rank[k] = brick_major_rank(R, g);
        B.cstart[0][k] = 0;
        B.cstart[1][k] = 0;
        B.ccnt[0][k] = 0;
        B.ccnt[1][k] = 0;
    }
    if (t == 0) {
        B.flags[r] = 0u;
        B.step[r] = 0ull;
        for (int k = 0; k < 4; ++k) B.stats[4 * r + k] = 0ull;
    }
}

// A replica leaves: its bricks become free (brick kernels skip them) and its descriptor
// empty (reductions over it give zeros).
__global__ void k_retire(Buffers B, int r, int b_off, int nbrick)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < nbrick) B.brick_rep[b_off + t] = -1;
    if (t == 0) {
        B.reps[r].n = 0;
        B.reps[r].nbrick = 0;
        B.reps[r].ncell = 0;
    }
}

// Device time stamp at the end of a step (stream order: after every kernel of the step).
__global__ void k_stamp(Buffers B, uint32_t mask)
{
    unsigned long long k = B.stamp_n[0];
    B.stamps[k & mask] = wall_clock64();
    B.stamp_n[0] = k + 1ull;
}

// Work lists of the capacity-wide launches, made on the GPU at the start of every step
// from the replica table: list 0 = every brick of every live replica (pools; a fixed set's
// bricks are all live, in order, and need no list), list 1 = the bricks of the replicas whose
// list is due for an incremental rebuild.  Replica slots in order, bricks in order inside a
// replica, so consecutive entries are neighbouring bricks.  Every workgroup scans the table
// itself and writes its share of the entries: one workgroup for all took 32 us for 27,648
// bricks of 1024 replicas and 7.3 us for 6,912 of 32.
constexpr int WL_PER_GROUP = 2048;  // entries per workgroup

__global__ void __launch_bounds__(1024) k_worklist(Buffers B, int nrep, int first)
{
    __shared__ int pre[2][MAX_REPLICAS + 1];
    __shared__ int boff[MAX_REPLICAS];
    __shared__ int tot[2];
    for (int r = threadIdx.x; r < nrep; r += blockDim.x) {
        const RepDev &R = B.reps[r];
        const int nb = R.nbrick;  // 0 for a free slot
        const uint32_t fl = B.flags[r];
        pre[0][r] = nb;
        pre[1][r] = ((fl & VBC_FLAG_REBUILD) && !(fl & FLAG_FULL)) ? nb : 0;
        boff[r] = R.b_off;
    }
    __syncthreads();
    for (int l = first; l < 2; ++l) {
        const int t = wave0_exclusive_scan(pre[l], nrep);
        if (threadIdx.x == 0) {
            tot[l] = t;
            if (blockIdx.x == 0) B.wl_n[l] = t;
        }
    }
    __syncthreads();
    for (int l = first; l < 2; ++l) {
        const int T = tot[l];
        for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < T; k += gridDim.x * blockDim.x) {
            // the last replica whose first entry is <= k (empty entries share their
            // successor's start, so the one found has bricks)
            int lo = 0, hi = nrep - 1;
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if (pre[l][mid] <= k) lo = mid; else hi = mid - 1;
            }
            B.wl[l][k] = boff[lo] + (k - pre[l][lo]);
        }
    }
}

// ---------------------------------------------------------------------------
// list build, step 1: the next sorted layout
// ---------------------------------------------------------------------------

struct SortTabs {
    int *m_src;    // [bcap] source slot of each member
    int *m_tag;    // [bcap]
    int *m_lc;     // [bcap] cell inside the brick
    int *bucket;   // [bcap] members grouped by cell
    int *hist;     // [ncb_max]
    int *cpre;     // [ncb_max]
    int *fill;     // [ncb_max]
};

__device__ __forceinline__ SortTabs carve_sort(unsigned char *p, int bcap, int ncb_max)
{
    SortTabs T;
    int *q = (int *)p;
    T.m_src = q;
    T.m_tag = q + bcap;
    T.m_lc = q + 2 * bcap;
    T.bucket = q + 3 * bcap;
    T.hist = q + 4 * bcap;
    T.cpre = T.hist + ncb_max;
    T.fill = T.cpre + ncb_max;
    return T;
}

// Order the nmem members gathered in LDS by (cell, tag), then write them in that order
// into the next layout of brick b, with the brick's cell tables.  Positions are wrapped
// into the box as they are copied.  On entry hist holds the members per cell, cpre a
// copy of it and fill zeros.
__device__ void place_members(const Buffers &B, const RepDev &R, int r, int b,
                              const StageHdr &S, SortTabs T, int nmem, int cur, int64_t S_)
{
    wave0_exclusive_scan(T.cpre, S.ncb);
    __syncthreads();
    for (int m = threadIdx.x; m < nmem; m += blockDim.x) {
        int lc = T.m_lc[m];
        int p = T.cpre[lc] + atomicAdd(&T.fill[lc], 1);
        T.bucket[p] = m;
    }
    __syncthreads();
    for (int p = threadIdx.x; p < nmem; p += blockDim.x) {
        int m = T.bucket[p];
        int lc = T.m_lc[m];
        int lo = T.cpre[lc], hi = lo + T.hist[lc];
        int key = T.m_tag[m];
        int rank = 0;
        for (int k = lo; k < hi; ++k) rank += (T.m_tag[T.bucket[k]] < key) ? 1 : 0;
        int64_t ns = S.base + lo + rank;
        int64_t o = T.m_src[m];
        for (int a = 0; a < 3; ++a) {
            B.xs[3 * ns + a] = wrap1(B.x[cur][3 * o + a], R.L[a]);
            B.vs[a * S_ + ns] = B.v[a * S_ + o];
        }
        B.tags[ns] = key;
        B.types[ns] = B.type[o];
        B.lcells[ns] = (uint8_t)lc;
        // caller index -> slot: read only for the bond partners of chains (a scattered
        // write per particle, left out without bonds)
        if (R.chain_len > 1) B.inv[R.o_off + key] = (int32_t)ns;
    }
    for (int lc = threadIdx.x; lc < S.ncb; lc += blockDim.x) {
        B.cstart[1][R.c_off + S.rank0 + lc] = (int32_t)(S.base + T.cpre[lc]);
        B.ccnt[1][R.c_off + S.rank0 + lc] = T.hist[lc];
    }
    if (threadIdx.x == 0) B.bcnt[1][b] = nmem;
}

// Local cell of position x inside brick S, or -1 if the particle is not in the brick.
__device__ __forceinline__ int local_cell(const RepDev &R, const StageHdr &S, const double *xw)
{
    int l[3];
    for (int a = 0; a < 3; ++a) {
        int c = cell_of(xw[a], R.h[a], R.nc[a]) - S.c0[a];
        if (c < 0 || c >= S.e[a]) return -1;
        l[a] = c;
    }
    return l[0] + S.e[0] * (l[1] + S.e[1] * l[2]);
}

// Full build, part 1: bin the unsorted particle tg of replica r into its brick's bucket.
__device__ __forceinline__ void bin_particle(const Buffers &B, const RepDev &R, int cur, int r, int64_t tg)
{
    int64_t d = R.p_off + tg;
    int c[3];
    bool bad = false;
    for (int a = 0; a < 3; ++a) {
        double t = B.x[cur][3 * d + a];
        if (!isfinite(t)) {
            bad = true;
            t = 0.0;
        }
        t = wrap1(t, R.L[a]);
        B.x[cur][3 * d + a] = t;
        c[a] = cell_of(t, R.h[a], R.nc[a]) / R.bd[a];
    }
    if (bad) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_NONFINITE);
    int lb = c[0] + R.nb[0] * (c[1] + R.nb[1] * c[2]);
    int idx = atomicAdd(&B.bfill[R.b_off + lb], 1);
    if (idx < R.bcap)
        B.src[R.p_off + (int64_t)lb * R.bcap + idx] = (int32_t)d;
    else
        atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_STAGE_OVERFLOW);
}

__global__ void k_gbin(Buffers B, int64_t S_, int cur, int r)
{
    const RepDev &R = B.reps[r];
    int64_t tg = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tg >= R.n) return;
    if (!(B.flags[r] & FLAG_FULL)) return;
    bin_particle(B, R, cur, r, tg);
}

// Every replica with unsorted input at once (workgroups as in k_set_state_all).
__global__ void k_gbin_all(Buffers B, int cur)
{
    const int b = blockIdx.x, r = B.brick_rep[b];
    if (r < 0 || !(B.flags[r] & FLAG_FULL)) return;
    const RepDev &R = B.reps[r];
    const int64_t t0 = (int64_t)(b - R.b_off) * R.bcap, t1 = min(t0 + R.bcap, R.n);
    for (int64_t tg = t0 + threadIdx.x; tg < t1; tg += blockDim.x) bin_particle(B, R, cur, r, tg);
}

// Full build, part 2: order each bucket and write the next layout.
__global__ void k_gsort(Buffers B, Launch P, int cur)
{
    extern __shared__ __align__(32) unsigned char smem[];
    __shared__ StageHdr S;
    int b, r;
    if (!resolve_brick(P, B, b, r)) return;
    const RepDev &R = B.reps[r];
    if (!(B.flags[r] & FLAG_FULL)) return;
    int lb = b - R.b_off;
    SortTabs T = carve_sort(smem, P.bcap_max, P.ncb_max);
    if (threadIdx.x == 0) {
        brick_geometry(R, lb, S);
        S.rank0 = B.brick_rank0[b];
    }
    __syncthreads();
    for (int lc = threadIdx.x; lc < S.ncb; lc += blockDim.x) {
        T.hist[lc] = 0;
        T.fill[lc] = 0;
    }
    __syncthreads();
    int nmem = min(B.bfill[b], R.bcap);
    const int64_t S_ = P.nslots;
    for (int m = threadIdx.x; m < nmem; m += blockDim.x) {
        int d = B.src[S.base + m];
        double xw[3] = {B.x[cur][3 * d], B.x[cur][3 * d + 1], B.x[cur][3 * d + 2]};
        int lc = local_cell(R, S, xw);
        if (lc < 0) lc = 0;  // not reached: binned from the same wrapped coordinates
        T.m_src[m] = d;
        T.m_tag[m] = B.tag[d];
        T.m_lc[m] = lc;
        atomicAdd(&T.hist[lc], 1);
    }
    __syncthreads();
    for (int lc = threadIdx.x; lc < S.ncb; lc += blockDim.x) T.cpre[lc] = T.hist[lc];
    __syncthreads();
    place_members(B, R, r, b, S, T, nmem, cur, S_);
    __syncthreads();
    if (threadIdx.x == 0) B.bfill[b] = 0;
}

// Incremental build: gather the particles now inside the brick from the one-cell halo of
// the current layout (a particle moves less than one cell between builds), order them and
// write the next layout.
__global__ void k_resort(Buffers B, Launch P, int cur)
{
    extern __shared__ __align__(32) unsigned char smem[];
    __shared__ StageHdr Ssh;
    __shared__ int nmem_s;
    int b;
    if (!brick_of_block(P, B, b)) return;
    // replica 0's flags read beside the owner: with one replica (the usual case) the test
    // that ends most launches needs no dependent read
    const uint32_t fl0 = B.flags[0];
    const int r = B.brick_rep[b];
    const int tot = B.stotal[b];
    if (r < 0) return;
    const uint32_t fl = r == 0 ? fl0 : B.flags[r];
    if (!(fl & VBC_FLAG_REBUILD) || (fl & FLAG_FULL)) return;
    // the staging map's first entries are read only once a build is due: a launch on a
    // step without a build (most steps) then reads nothing but the flags
    const MapFirst mf = map_prefetch(B, b, P.stage_cap);
    const RepDev &R = B.reps[r];
    int lb = b - R.b_off;
    int nh_cap = (P.nh_max + 3) & ~3;
    StageTabs Q = carve_tabs(smem, nh_cap);
    SortTabs T = carve_sort(after_tabs(smem, nh_cap), P.bcap_max, P.ncb_max);
    // the candidates (the brick and its one-cell halo in the live layout) are exactly the
    // particles the last list build staged: read them through its staging map (header in
    // every thread, no cell-table walk); after an overflowed build, walk the cell tables
    const bool use_map = tot <= P.stage_cap;
    StageHdr S;
    if (use_map) {
        pass_header(R, B, b, lb, P.stage_cap, S);
        S.rank0 = B.brick_rank0[b];
    } else {
        stage_tables(R, b, lb, B.brick_rank0, B.cell_rank, B.cstart[0], B.ccnt[0], B.bcnt[0], Ssh, Q,
                     1 << 30);
        S = Ssh;
    }
    for (int lc = threadIdx.x; lc < S.ncb; lc += blockDim.x) {
        T.hist[lc] = 0;
        T.fill[lc] = 0;
    }
    if (threadIdx.x == 0) nmem_s = 0;
    __syncthreads();
    const int64_t S_ = P.nslots;
    const int bcap = R.bcap;
    auto member = [&](int src, bool ok) {
        double xw[3];
        for (int a = 0; a < 3; ++a) xw[a] = wrap1(B.x[cur][3 * src + a], R.L[a]);
        const int tg = B.tag[src];
        int lc = local_cell(R, S, xw);
        if (ok && lc >= 0) {
            int m = atomicAdd(&nmem_s, 1);
            if (m < bcap) {
                T.m_src[m] = src;
                T.m_tag[m] = tg;
                T.m_lc[m] = lc;
                atomicAdd(&T.hist[lc], 1);
            }
        }
    };
    if (use_map) stage_map4(B, b, P.stage_cap, S, mf, [&](int t, int src, int w, bool ok) { member(src, ok); });
    else stage_copy(S, Q, [&](int t, int src, int w) { member(src, true); });
    __syncthreads();
    int nmem = nmem_s;
    if (nmem > bcap) {
        if (threadIdx.x == 0) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_STAGE_OVERFLOW);
        nmem = bcap;
    }
    for (int lc = threadIdx.x; lc < S.ncb; lc += blockDim.x) T.cpre[lc] = T.hist[lc];
    __syncthreads();
    place_members(B, R, r, b, S, T, nmem, cur, S_);
}

// ---------------------------------------------------------------------------
// list build, step 2: copy to live, build the list
// ---------------------------------------------------------------------------

// Copy brick b of the next layout into the live arrays and list, for each own particle,
// every staged j != i with minimum-image r^2 < r_list^2.  The decision is exact: the
// staged FP32 brick-local positions decide every pair whose r^2 is further than 1e-4 from
// r_list^2 (their error is below 2e-5), and the remaining pairs are tested with the same
// FP64 expression as the plain definition -- t = x_i - x_j, d = t - L k with k the image
// of the halo cell, r^2 = (dx dx + dy dy) + dz dz, no contraction.  Entries are written
// eight at a time as 16-byte chunks.
//
// The candidate scan reads a second copy of the staged positions in LDS, laid out in the
// x-fastest order of the whole (e+2)^3 cell grid, own and halo cells together: the three
// cells of a stencil row along x are then one contiguous range, and a particle has 9 ranges
// instead of 27 cells (a wave pays the longest range among its lanes, about 20 % fewer
// iterations).  Entries are the staging-order indices, so the lists are the same.
//
// Three lanes scan for one particle, a plane of the stencil (three rows) each: first the masks
// of its rows' neighbours, then, with the lanes' counts added up, the entries, gathered in LDS
// and written out as chunks.  What bounds a build is the chain of one wave: LDS reads, the
// loop over a row's candidates and the loop over its entries, at two waves per SIMD or fewer.
// With one lane per particle a workgroup took 25 to 27 us at density 0.3 (scan 16) and 20 at
// 0.05 (7.7 of them the staging, a memory round trip per few cells); now 13 and 9.  At density
// 0.5 and a million particles a build takes 10 % less, near the issue rate of the test of
// some 270 candidates per particle.  The registers must stay below 80 with none spilled: a
// kernel that uses scratch memory costs 0.5 us more in every step without a build.
#ifndef NLIST_ATTR
#define NLIST_ATTR __attribute__((amdgpu_waves_per_eu(6)))
#endif
#ifndef SCAN_UNROLL
#define SCAN_UNROLL 4  // candidate positions read ahead in the list build's scan
#endif
constexpr int NL_PPW = VBC_WAVE / 3;  // particles of one wave (its last lane idles)

template <bool LARGE>
__device__ __forceinline__ void nlist_brick(const Buffers &B, const Launch &P, int cur, int b)
{
    extern __shared__ __align__(32) unsigned char smem[];
    __shared__ unsigned long long lost_sum;
    __shared__ unsigned ent_sum;
    __shared__ int halo_s;          // staged particles of the halo cells
    const uint32_t fl0 = B.flags[0];  // as in k_resort
    const int r = B.brick_rep[b];
    if (r < 0) return;
    if (!((r == 0 ? fl0 : B.flags[r]) & P.due)) return;
    const RepDev &R = B.reps[r];
    const int lb = b - R.b_off;
    const int nh_cap = (P.nh_max + 3) & ~3;
    StageTabs T = carve_tabs(smem, nh_cap);
    float4 *hpos = (float4 *)after_tabs(smem, nh_cap);    // staged positions, grid order
    int *hq = (int *)(hpos + P.lds_cap + SCAN_UNROLL);  // first grid-order index of each cell
    uint16_t *wbuf = (uint16_t *)(hq + nh_cap + 4);       // entries on their way out, per particle
    const int bstride = P.list_win + CHUNK;
    uint16_t *conv = wbuf + (blockDim.x / VBC_WAVE) * (NL_PPW * bstride);  // grid order -> staging order
    const int64_t S_ = P.nslots;

    // every thread forms the header itself (uniform values)
    StageHdr S;
    brick_geometry(R, lb, S);
    S.rank0 = B.brick_rank0[b];
    S.n_own = B.bcnt[1][b];
    if (threadIdx.x == 0) {
        lost_sum = 0ull;
        ent_sum = 0u;
    }
    stage_cells(R, S, B.cell_rank, B.cstart[1], B.ccnt[1], T, hq);
    __syncthreads();
    // halo offsets by the first wave, grid-order offsets by the second
    {
        const int w2 = blockDim.x > VBC_WAVE ? 1 : 0;
        if (threadIdx.x < VBC_WAVE) {
            const int tot = wave_exclusive_scan(T.q_hpre, S.nh);
            if (threadIdx.x == 0) halo_s = tot;
        }
        if (threadIdx.x / VBC_WAVE == w2) {
            const int tot = wave_exclusive_scan(hq, S.nh);
            if (threadIdx.x % VBC_WAVE == 0) hq[S.nh] = tot;
        }
    }
    __syncthreads();
    S.total = S.n_own + halo_s;
    S.overflow = S.total > P.stage_cap;
    if (!LARGE && S.total > P.t_hi) {
        if (threadIdx.x == 0) B.stotal[b] = S.total;  // the second launch takes it
        return;
    }

    if (!S.overflow) {
        // the brick's staging map and, at each particle's grid-order index, a record of where
        // it comes from: no memory is read, so a cell's few particles cost no round trip
        int32_t *sm = B.smap + (size_t)b * P.stage_cap;
        uint8_t *wm = B.wmap + (size_t)b * P.stage_cap;
        const int gid = threadIdx.x / VBC_GROUP, gl = threadIdx.x % VBC_GROUP;
        const int ng = blockDim.x / VBC_GROUP;
        for (int q = gid; q < S.nh; q += ng) {
            const int own = T.q_off[q], src0 = T.q_src[q], cnt = T.q_cnt[q], w = T.q_w[q], h0 = hq[q];
            const int off = own >= 0 ? own : S.n_own + T.q_hpre[q];
            for (int k = gl; k < cnt; k += VBC_GROUP) {
                const int t = off + k, src = src0 + k;
                sm[t] = src;
                wm[t] = (uint8_t)w;
                *(int4 *)(hpos + h0 + k) = make_int4(src, w, t, 0);
            }
        }
        __syncthreads();
        // then every staged position, gathered all at once, with |p|^2 in the fourth component
        // (brick-centred FP32 coordinates); the own particles go into the live arrays on the way.
        // An empty brick needs the map only, for the re-sort.
        if (S.n_own > 0) {
            const int nt = blockDim.x, last = S.total - 1;
            const int64_t i0 = S.base + min((int)threadIdx.x, S.n_own - 1);
            const double v0[3] = {B.vs[i0], B.vs[S_ + i0], B.vs[2 * S_ + i0]};
            const int32_t tag0 = B.tags[i0];
            const auto type0 = B.types[i0];
            const auto lc0 = B.lcells[i0];
            for (int h0 = threadIdx.x; h0 < S.total; h0 += 2 * nt) {
                int4 rec[2];
                double x[2][3];
#pragma unroll
                for (int j = 0; j < 2; ++j) rec[j] = *(const int4 *)(hpos + min(h0 + j * nt, last));
                // a record past the end may be a position by now: not used as an index
                if (h0 + nt > last) rec[1] = rec[0];
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    for (int a = 0; a < 3; ++a) x[j][a] = B.xs[3 * rec[j].x + a];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int h = h0 + j * nt, w = rec[j].y;
                    float4 p;
                    p.x = (float)((x[j][0] + R.L[0] * (double)unpack_w(w, 0)) - S.O[0]);
                    p.y = (float)((x[j][1] + R.L[1] * (double)unpack_w(w, 1)) - S.O[1]);
                    p.z = (float)((x[j][2] + R.L[2] * (double)unpack_w(w, 2)) - S.O[2]);
                    p.w = fmaf(p.x, p.x, fmaf(p.y, p.y, p.z * p.z));
                    if (h <= last) {
                        hpos[h] = p;
                        conv[h] = (uint16_t)rec[j].z;
                        if (rec[j].z < S.n_own)
                            for (int a = 0; a < 3; ++a) B.x[cur][3 * rec[j].x + a] = x[j][a];
                    }
                }
            }
            if ((int)threadIdx.x < S.n_own) {
                for (int a = 0; a < 3; ++a) B.v[a * S_ + i0] = v0[a];
                B.tag[i0] = tag0;
                B.type[i0] = type0;
                B.lcell[i0] = lc0;
            }
            for (int t = threadIdx.x + nt; t < S.n_own; t += nt) {
                const int64_t i = S.base + t;
                for (int a = 0; a < 3; ++a) B.v[a * S_ + i] = B.vs[a * S_ + i];
                B.tag[i] = B.tags[i];
                B.type[i] = B.types[i];
                B.lcell[i] = B.lcells[i];
            }
        }
        // the scan reads up to SCAN_UNROLL - 1 records past a row's end: far-away padding
        if ((int)threadIdx.x < SCAN_UNROLL) hpos[S.total + threadIdx.x] = make_float4(1e18f, 1e18f, 1e18f, 3e36f);
        __syncthreads();

        // The pre-filter forms d = (|p_u|^2 - c_i) - 2 p_i.p_u with c_i = mid - |p_i|^2, mid the
        // middle of [lo2, hi2]: one subtraction and three fused steps per candidate.  With
        // u = 2^-24 and Q = (|p_i| + |p_u|)^2 + hi2, the rounded squares, the subtractions and the
        // fused steps (whose partial sums stay below 2 Q) err by less than 26 u Q in total, and
        // the direct form |p_i - p_u|^2 differs from the exact local distance by at most 5 u hi2.
        // A candidate within a hundredth of the list radius of it has |p_u| < |p_i| + 1.01 sqrt(rl2),
        // so that with hd = (hi2 - lo2) / 2 + 64 u ((2 |p_i| + 1.01 sqrt(rl2))^2 + hi2), over twice
        // the bound, d <= -hd puts the direct form below lo2 (in the list) and d >= hd above hi2
        // (not in it); one further off has |d| above 0.02 rl2, a hundred times the error
        // over a brick, and the right sign.  The few in between (one row in a thousand holds
        // one: the smallest |d| of the row tells) are decided by the direct form against lo2 and
        // hi2, and in FP64 between those.
        // (R.scan; read where they are used, which costs scalar loads instead of registers)
        const int kmax = P.k_max, W = P.list_win;
        // read once: the global descriptor cannot be kept in registers across the list stores
        const int xspan = R.excl_span, cl = R.chain_len;
        // division of a cell index (below 256) by the brick's edges: ceil(2^16 / e)
        const uint32_t d0 = (65535u + S.e[0]) / (uint32_t)S.e[0], d1 = (65535u + S.e[1]) / (uint32_t)S.e[1];
        const int lane = threadIdx.x % VBC_WAVE, nwv = blockDim.x / VBC_WAVE;
        const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / VBC_WAVE);
        const int g = lane / 3, sub = lane - 3 * g;  // particle of the wave, plane of the stencil
        uint16_t *buf = wbuf + (wv * NL_PPW + min(g, NL_PPW - 1)) * bstride;
        for (int t0 = wv * NL_PPW; t0 < S.n_own; t0 += nwv * NL_PPW) {
            const bool live = g < NL_PPW && t0 + g < S.n_own;
            const int t = live ? t0 + g : t0;
            const int64_t i = S.base + t;
            const uint32_t loc = B.lcells[i];
            const uint32_t lyz = (loc * d0) >> 16;  // ly + e1 lz
            const int lz = (int)((lyz * d1) >> 16), ly = (int)lyz - S.e[1] * lz,
                      lx = (int)loc - S.e[0] * (int)lyz;
            const int qs = (lx + 1) + S.H[0] * ((ly + 1) + S.H[1] * (lz + 1));
            const int hs = hq[qs] + (t - T.q_off[qs]);  // this particle in grid order
            const float4 pi = hpos[hs];
            const float mx = -2.0f * pi.x, my = -2.0f * pi.y, mz = -2.0f * pi.z, ci = R.scan.mid - pi.w;
            const float reach = 2.0f * sqrtf(pi.w) + R.scan.reach;
            const float hd = R.scan.half + 0x1p-18f * fmaf(reach, reach, R.scan.hi2);
            // the neighbours among the n <= 32 candidates u0, u0 + 1, ... of the row of cells
            // q0, q0 + 1, q0 + 2, candidate k at bit 31 - k
            auto segment = [&](int u0, int n, int q0) -> uint32_t {
                if (n <= 0) return 0u;
                uint32_t near = 0u;
                float closest = 3e38f;
                int k0 = 0;
                for (; k0 < n; k0 += SCAN_UNROLL) {
                    const float4 *pp = hpos + (u0 + k0);
                    float4 pu[SCAN_UNROLL];
                    float d[SCAN_UNROLL];
#pragma unroll
                    for (int j = 0; j < SCAN_UNROLL; ++j) pu[j] = pp[j];
#pragma unroll
                    for (int j = 0; j < SCAN_UNROLL; ++j) {
                        d[j] = fmaf(pu[j].z, mz, fmaf(pu[j].y, my, fmaf(pu[j].x, mx, pu[j].w - ci)));
                        near = __builtin_amdgcn_alignbit(near, __float_as_uint(d[j]), 31);
                    }
#pragma unroll
                    for (int j = 0; j < SCAN_UNROLL; j += 2)
                        closest = fminf(closest, fminf(fabsf(d[j]), fabsf(d[j + 1])));
                }
                near <<= 32 - k0;
                if (n < 32) near &= ~(0xffffffffu >> n);  // reads past the row
                if (closest < hd) {
                    uint32_t close = 0u;
                    for (k0 = 0; k0 < n; k0 += SCAN_UNROLL) {
#pragma unroll
                        for (int j = 0; j < SCAN_UNROLL; ++j) {
                            const float4 pu = hpos[u0 + k0 + j];
                            const float d = fmaf(pu.z, mz, fmaf(pu.y, my, fmaf(pu.x, mx, pu.w - ci)));
                            close = __builtin_amdgcn_alignbit(close, __float_as_uint(fabsf(d) - hd), 31);
                        }
                    }
                    close <<= 32 - k0;
                    if (n < 32) close &= ~(0xffffffffu >> n);
                    while (close) {
                        const int k = __builtin_clz(close);
                        const uint32_t bit = 0x80000000u >> k;
                        close &= ~bit;
                        const float4 pu = hpos[u0 + k];
                        const float ex = -0.5f * mx - pu.x, ey = -0.5f * my - pu.y, ez = -0.5f * mz - pu.z;
                        const float r2f = ex * ex + ey * ey + ez * ez;
                        bool in = r2f < R.scan.lo2;
                        if (!in && r2f < R.scan.hi2) {
                            // near the list radius: decide with the exact FP64 expression
                            const int u = u0 + k;
                            const int q = q0 + (u >= hq[q0 + 1] ? 1 : 0) + (u >= hq[q0 + 2] ? 1 : 0);
                            const int w = T.q_w[q];
                            const int64_t js = T.q_src[q] + (u - hq[q]);
                            // axis by axis: a rare path that must not cost the scan registers
                            double r2 = 0.0;
#pragma unroll 1
                            for (int a = 0; a < 3; ++a) {
#pragma clang fp contract(off)
                                double ta = B.xs[3 * i + a] - B.xs[3 * js + a];
                                double da = ta - R.L[a] * (double)unpack_w(w, a);
                                r2 = r2 + da * da;
                            }
                            in = r2 < R.rlist2;
                        }
                        near = in ? (near | bit) : (near & ~bit);
                    }
                }
                if (u0 <= hs && hs < u0 + n) near &= ~(0x80000000u >> (hs - u0));  // not itself
                return near;
            };
            // the masks of the first 64 candidates of each row are kept (the rows' pairs of
            // masks rotate through three); longer rows (dense clusters) are scanned again when
            // their entries are written
            uint32_t ma[2] = {0u, 0u}, mb[2] = {0u, 0u}, mc[2] = {0u, 0u};
            int cnt = 0;
            const int qz = lx + S.H[0] * (ly + S.H[1] * (lz + sub));
#pragma unroll 1
            for (int dy = 0; dy < 3; ++dy) {
                const int q0 = qz + S.H[0] * dy, ub = hq[q0], ue = live ? hq[q0 + 3] : ub;
                ma[0] = mb[0], ma[1] = mb[1];
                mb[0] = mc[0], mb[1] = mc[1];
                mc[0] = mc[1] = 0u;
#pragma unroll 1
                for (int u0 = ub; u0 < ue; u0 += 32) {
                    const uint32_t mk = segment(u0, min(32, ue - u0), q0);
                    if (u0 == ub) mc[0] = mk;
                    if (u0 == ub + 32) mc[1] = mk;
                    cnt += __popc(mk);
                }
            }
            const int n0 = __shfl(cnt, 3 * g), n1 = __shfl(cnt, 3 * g + 1), n2 = __shfl(cnt, 3 * g + 2);
            const int tot = live ? n0 + n1 + n2 : 0;
            const int off = sub == 0 ? 0 : (sub == 1 ? n0 : n0 + n1);
            // bit 15 of an entry: chain neighbours up to excl_span beads apart
            auto excluded = [&](int u, int q0) -> uint32_t {
                const int q = q0 + (u >= hq[q0 + 1] ? 1 : 0) + (u >= hq[q0 + 2] ? 1 : 0);
                const int ta = B.tags[i], tb = B.tags[T.q_src[q] + (u - hq[q])];
                const int db = ta - tb;
                return ta / cl == tb / cl && db <= xspan && -db <= xspan ? 0x8000u : 0u;
            };
            // entries in windows of W: one window unless a list is longer
            for (int w0 = 0; __any(tot > w0); w0 += W) {
                int pos = off - w0;
#pragma unroll 1
                for (int dy = 0; dy < 3; ++dy) {
                    const int q0 = qz + S.H[0] * dy, ub = hq[q0], ue = live ? hq[q0 + 3] : ub;
                    const uint32_t m0 = ma[0], m1 = ma[1];
                    ma[0] = mb[0], ma[1] = mb[1];
                    mb[0] = mc[0], mb[1] = mc[1];
                    mc[0] = m0, mc[1] = m1;
#pragma unroll 1
                    for (int u0 = ub; u0 < ue; u0 += 32) {
                        uint32_t todo = u0 == ub ? m0 : m1;
                        if (u0 > ub + 32) todo = segment(u0, min(32, ue - u0), q0);
                        // a segment with no entry inside the window is passed over
                        const int pc = __popc(todo);
                        if (pos + pc <= 0 || pos >= W) {
                            pos += pc;
                            todo = 0u;
                        }
                        // two entries at a time, so that their reads overlap
                        while (todo) {
                            const int k = __builtin_clz(todo);
                            const uint32_t rest = todo & ~(0x80000000u >> k);
                            const int k2 = rest ? __builtin_clz(rest) : k;
                            uint32_t hv = (uint32_t)conv[u0 + k], hv2 = (uint32_t)conv[u0 + k2];
                            if (xspan > 0) {
                                hv |= excluded(u0 + k, q0);
                                hv2 |= excluded(u0 + k2, q0);
                            }
                            // entries outside the window go to the spare places behind it; the
                            // first entry of a chunk stands in its last place
                            const unsigned p2 = rest ? (unsigned)(pos + 1) : (unsigned)W;
                            buf[min((unsigned)pos, (unsigned)W) ^ (CHUNK - 1)] = (uint16_t)hv;
                            buf[min(p2, (unsigned)W) ^ (CHUNK - 1)] = (uint16_t)hv2;
                            pos += rest ? 2 : 1;
                            todo = rest & ~(0x80000000u >> k2);
                        }
                    }
                }
                // pad the last chunk with the dummy staged slot (far away: contributes nothing)
                const int fill = min(tot - w0, W);
                for (int k = fill + sub; k < ((fill + CHUNK - 1) & ~(CHUNK - 1)); k += 3)
                    if (fill > 0) buf[k ^ (CHUNK - 1)] = (uint16_t)S.total;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                for (int c = sub; c * CHUNK < fill; c += 3) {
                    const int ch = w0 / CHUNK + c;
                    if (ch < P.nchunk) B.nl[(size_t)ch * S_ + i] = *(const uint4 *)(buf + c * CHUNK);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            if (live && sub == 0) {
                if (tot > kmax) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_NLIST_OVERFLOW);
                B.nn[i] = (uint16_t)min(tot, kmax);
                atomicAdd(&ent_sum, (unsigned)min(tot, kmax));
            }
        }
    } else {
        for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
            const int64_t i = S.base + t;
            for (int a = 0; a < 3; ++a) {
                B.x[cur][3 * i + a] = B.xs[3 * i + a];
                B.v[a * S_ + i] = B.vs[a * S_ + i];
            }
            B.tag[i] = B.tags[i];
            B.type[i] = B.types[i];
            B.lcell[i] = B.lcells[i];
            B.nn[i] = 0;
        }
        if (threadIdx.x == 0) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_STAGE_OVERFLOW);
    }

    // next layout's own cell tables -> live
    for (int lc = threadIdx.x; lc < S.ncb; lc += blockDim.x) {
        B.cstart[0][R.c_off + S.rank0 + lc] = B.cstart[1][R.c_off + S.rank0 + lc];
        B.ccnt[0][R.c_off + S.rank0 + lc] = B.ccnt[1][R.c_off + S.rank0 + lc];
    }
    if (lb == 0) {
        // every particle must have been placed in exactly one brick of the next layout
        unsigned long long placed = 0;
        for (int k = threadIdx.x; k < R.nbrick; k += blockDim.x) placed += B.bcnt[1][R.b_off + k];
        placed = wave_sum(placed);
        if ((threadIdx.x % VBC_WAVE) == 0 && placed) atomicAdd(&lost_sum, placed);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        B.bcnt[0][b] = S.n_own;
        B.stotal[b] = S.total;
        B.bentries[b] = ent_sum;
        if (lb == 0) {
            B.stats[4 * r + 0] += 1ull;
            if (lost_sum != (unsigned long long)R.n) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_LOST);
        }
    }
}

__global__ void __launch_bounds__(1024) NLIST_ATTR k_nlist(Buffers B, Launch P, int cur)
{
    int b;
    if (brick_of_block(P, B, b)) nlist_brick<false>(B, P, cur, b);
}

__global__ void __launch_bounds__(DENSE_BLOCK) k_nlist_dense(Buffers B, Launch P, int cur)
{
    each_dense(P, B, [&](int b) { nlist_brick<true>(B, P, cur, b); });
}

// ---------------------------------------------------------------------------
// list sweep helper
// ---------------------------------------------------------------------------

// The descriptor of replica r: the launch's own copy for a fixed single replica, else the
// workspace's.
template <bool ONE>
__device__ __forceinline__ const RepDev &rep_of(const OneRep<ONE> &R1, const Buffers &B, int r)
{
    if constexpr (ONE) return R1.R;
    else return B.reps[r];
}

// Length and first chunk of a particle's list (the chunk row 0 exists for every slot).  The
// count and force passes of a single replica read a thread's first one before the staging,
// whose latency then covers it (10 to 12 us of ten steps of 100,000 and of a million
// particles; in a set of mostly empty bricks the reads would cost as much as they save).
struct ListHead {
    int nn;
    uint4 q;
};
__device__ __forceinline__ ListHead list_head(const Buffers &B, int64_t i) { return ListHead{(int)B.nn[i], B.nl[i]}; }

// Visit the list of one own particle in whole chunks of eight entries (the last chunk is
// padded with the dummy staged slot, whose terms all vanish), with the next chunk's load
// issued before the current one is processed.  fn(staged index) is called for every entry
// of a chunk without a guard, so the eight LDS gathers of a chunk can be in flight together.
template <class F, class G>
__device__ __forceinline__ void for_each_neighbour(const uint4 *__restrict__ nl, int64_t S_,
                                                   int64_t i, const ListHead &head, F &&fn, G &&done)
{
    int nch = (head.nn + CHUNK - 1) / CHUNK;
    if (nch == 0) return;
    const uint4 *lp = nl + i;
    uint4 q = head.q;
    for (int c = 0; c < nch; ++c) {
        uint4 qn = (c + 1 < nch) ? lp[(size_t)(c + 1) * S_] : q;
        uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < CHUNK; ++e) fn((int)((w[e >> 1] >> (16 * (e & 1))) & 0xffffu));
        done();
        q = qn;
    }
}

template <class F>
__device__ __forceinline__ void for_each_neighbour(const uint4 *__restrict__ nl, int64_t S_,
                                                   int64_t i, int nn, F &&fn)
{
    if (nn > 0) for_each_neighbour(nl, S_, i, ListHead{nn, nl[i]}, fn, []() {});
}

// The value of lane j of each group of two (ls = 1) or four lanes, within the vector unit.
template <int LS, int J>
__device__ __forceinline__ double group_lane(double v)
{
    constexpr int ctrl = LS == 2 ? J * 0x55 : J * 0x55 + 0xa0;  // quad_perm: jjjj or j,j,2+j,2+j
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// sum + the group's values in the order of its lanes: the order in which one lane adds the
// chunks of a list.
__device__ __forceinline__ double add_group(double sum, double v, int ls)
{
    if (ls == 1) return (sum + group_lane<1, 0>(v)) + group_lane<1, 1>(v);
    return (((sum + group_lane<2, 0>(v)) + group_lane<2, 1>(v)) + group_lane<2, 2>(v)) + group_lane<2, 3>(v);
}

// The list of one particle by the 2^ls lanes that share it: lane `sub` takes every 2^ls-th
// chunk, and after each round of chunks every lane calls done() (a lane without a chunk left
// with nothing summed).
template <class F, class G>
__device__ __forceinline__ void for_each_neighbour_shared(const uint4 *__restrict__ nl, int64_t S_,
                                                          int64_t i, int nn, int sub, int ls, F &&fn, G &&done)
{
    const int nch = (nn + CHUNK - 1) / CHUNK, dc = 1 << ls;
    const uint4 *lp = nl + i;
    uint4 q = lp[(size_t)min(sub, max(nch - 1, 0)) * S_];
    for (int c0 = 0; c0 < nch; c0 += dc) {
        const int c = c0 + sub;
        const uint4 qn = (c + dc < nch) ? lp[(size_t)(c + dc) * S_] : q;
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        if (c < nch) {
#pragma unroll
            for (int e = 0; e < CHUNK; ++e) fn((int)((w[e >> 1] >> (16 * (e & 1))) & 0xffffu));
        }
        done();
        q = qn;
    }
}

// The dummy staged slot that pads list chunks: far from every particle of the brick.
template <class R4>
__device__ __forceinline__ R4 dummy_pos()
{
    R4 p;
    p.x = 1.0e6f;
    p.y = 1.0e6f;
    p.z = 1.0e6f;
    p.w = 0;
    return p;
}

// ---------------------------------------------------------------------------
// pass 1: counts
// ---------------------------------------------------------------------------

// Pair constants converted to the pair-arithmetic precision.
template <class Real>
struct PairR {
    Real E_r, c_r, inv_rr2, E_a, c_a, m, inv_w, inv_dw, c_c, rc2;
    Real k_r;      // -c_r / r_r^2: V_r'(r)/r = c_r + k_r r^2 inside the core
    Real nm_w;     // -m / w:  u_a = r / w + nm_w
    Real nrl_dw;   // -r_l / (r_h - r_l):  u_c = r / (r_h - r_l) + nrl_dw
};

template <class Real>
__device__ __forceinline__ PairR<Real> pair_r(const PairDev &p, double rc2)
{
    PairR<Real> q;
    q.E_r = (Real)p.E_r;
    q.c_r = (Real)p.c_r;
    q.inv_rr2 = (Real)p.inv_rr2;
    q.E_a = (Real)p.E_a;
    q.c_a = (Real)p.c_a;
    q.m = (Real)p.m;
    q.inv_w = (Real)p.inv_w;
    q.inv_dw = (Real)p.inv_dw;
    q.c_c = (Real)p.c_c;
    q.rc2 = (Real)rc2;
    q.k_r = (Real)(-p.c_r * p.inv_rr2);
    q.nm_w = (Real)(-p.m * p.inv_w);
    q.nrl_dw = (Real)(-p.r_l * p.inv_dw);
    return q;
}

// Brick-local position of a staged particle: (x + k L) - O, rounded once to Real.
template <class Real>
__device__ __forceinline__ typename V4<Real>::t local_pos(const RepDev &R, const StageHdr &S,
                                                          const double *__restrict__ X,
                                                          int64_t S_, int src, int w, int type)
{
    typename V4<Real>::t p;
    p.x = (Real)((X[3 * src] + R.L[0] * (double)unpack_w(w, 0)) - S.O[0]);
    p.y = (Real)((X[3 * src + 1] + R.L[1] * (double)unpack_w(w, 1)) - S.O[1]);
    p.z = (Real)((X[3 * src + 2] + R.L[2] * (double)unpack_w(w, 2)) - S.O[2]);
    p.w = (Real)type;
    return p;
}

// Type pair (i, j) of the general pair path as three records of four, so that a list entry
// takes three LDS reads of its pair instead of one per constant: the lanes of a wave read at
// most 16 different records, which lie in different banks.  Absent interactions are zero
// coefficients (no attraction: c_a = E_a = 0; j not counted by i: the mask bit in cnt.x), so
// that the pair terms need no branch.  The general force pass is bound by VALU issue: with one
// read per constant, a division per switching factor and branches that nearly every wave took
// both sides of, it ran at 118.7 us on a melt of 250,000 beads (density 0.85, two types); this
// form takes 61.7 us, and the dU/dn pass with its gathers in phases 12.4 us instead of 14.7.
template <class Real>
struct PairM {
    typename V4<Real>::t core;  // c_r, k_r, c_a, x1
    typename V4<Real>::t geo;   // 1/w, -m/w, 1/(r_h - r_l), -r_l/(r_h - r_l)
    typename V4<Real>::t cnt;   // c_c [i counts j], c_c [j counts i], E_r / c_r^2, E_a
};

template <class Real>
__device__ __forceinline__ PairM<Real> pair_m(const RepDev &R, int a, int c)
{
    const PairDev &p = R.pair[a * MAXT + c];
    PairM<Real> q;
    q.core.x = (Real)p.c_r;
    q.core.y = (Real)(-p.c_r * p.inv_rr2);
    q.core.z = p.attract ? (Real)p.c_a : Real(0);
    q.core.w = (Real)p.x1;
    q.geo.x = (Real)p.inv_w;
    q.geo.y = (Real)(-p.m * p.inv_w);
    q.geo.z = (Real)p.inv_dw;
    q.geo.w = (Real)(-p.r_l * p.inv_dw);
    q.cnt.x = ((R.mask[a] >> c) & 1u) ? (Real)p.c_c : Real(0);
    q.cnt.y = ((R.mask[c] >> a) & 1u) ? (Real)p.c_c : Real(0);
    q.cnt.z = p.E_r > 0.0 ? (Real)(p.E_r / (p.c_r * p.c_r)) : Real(0);
    q.cnt.w = p.attract ? (Real)p.E_a : Real(0);
    return q;
}

// Thread 0 writes the constants of the only type pair.
template <class Real>
__device__ __forceinline__ void load_pairs(const RepDev &R, PairR<Real> *pt)
{
    if (threadIdx.x == 0) pt[0] = pair_r<Real>(R.pair[0], R.rc2);
}

// One thread per type pair writes its record (the general path).
template <class Real>
__device__ __forceinline__ void load_pairs_m(const RepDev &R, PairM<Real> *pm, int tid)
{
    const int nt = R.ntypes;
    if (tid < nt * nt) {
        const int a = tid / nt, c = tid % nt;
        pm[a * MAXT + c] = pair_m<Real>(R, a, c);
    }
}

// One term of eq. (counter) in FP64: omega(r, r_l, r_h) = (1 - u^2)^2 with
// u = (r - r_l)/(r_h - r_l), exactly 1 inside r_l and 0 beyond r_h.
__device__ __forceinline__ double count_term64(double r2, const PairDev &p)
{
    if (r2 <= p.rl2) return 1.0;
    if (r2 >= p.rh2) return 0.0;
    const double u = (sqrt(r2) - p.r_l) * p.inv_dw;
    const double q = 1.0 - u * u;
    return q * q;
}

// With FP32 pair arithmetic a particle is listed for an FP64 recount when its FP32 count
// lies within this margin of a switching window (the FP32 count is within about 1e-5 of
// the exact one), so that every particle whose exact count lies inside a window is listed.
constexpr double COUNT_MARGIN = 1e-4;

// Counts in FP64 of the particles the FP32 count pass listed (brick b, its first nw
// entries of wlst): their switching factor s and dU/dn depend steeply on n (eq. (Psi),
// eq. (Psidelta)), so the count is summed again from the FP64 positions, gathered through
// the brick's staging map, instead of the FP32 staged ones (whose rounding would move each
// count term by up to about 3e-6).  A group of LANES lanes per particle: lane l takes list
// entry l % 8 of chunk l / 8 (+ LANES / 8 per further chunk it reads), CP chunks per lane
// in a phase of three dependent gathers (list chunk, staging map, position) that go out
// together; the partial sums are added in a fixed order.  Writes n (FP64), s (or n with
// several types) and, if asked, the caller-order count.
template <class Real, bool MULTI, int LANES, int CP>
__device__ __forceinline__ void recount_window(const Buffers &B, const Launch &P, const RepDev &R, int b,
                               int total, int64_t base, int nw, const double *__restrict__ X,
                               double *__restrict__ n_out)
{
    using R2 = typename V2<Real>::t;
    constexpr int CG = LANES / CHUNK;  // chunks read side by side by one group
    const int g = threadIdx.x / LANES, l = threadIdx.x % LANES, ng = blockDim.x / LANES;
    const int e = l % CHUNK, cl = l / CHUNK;
    const int64_t S_ = P.nslots;
    const int32_t *sm = B.smap + (size_t)b * P.stage_cap;
    const uint8_t *wm = B.wmap + (size_t)b * P.stage_cap;
    const bool xr = R.excl_span > 0;
    const double L0 = R.L[0], L1 = R.L[1], L2 = R.L[2];
    const PairDev p0 = R.pair[0];
    R2 *sA = (R2 *)B.sA;
    for (int k = g; k < nw; k += ng) {
        const int t = B.wlst[base + k];
        const int64_t i = base + t;
        const double xi0 = X[3 * i], xi1 = X[3 * i + 1], xi2 = X[3 * i + 2];
        const int ti = MULTI ? B.type[i] : 0;
        const int nch = (B.nn[i] + CHUNK - 1) / CHUNK;
        double acc = 0.0;
        // no branch between the loads of a phase; rows past the list (every slot has nchunk
        // rows) and the padding slot read valid memory and are masked
        for (int c0 = 0; c0 < nch; c0 += CG * CP) {
            uint4 q[CP];
#pragma unroll
            for (int j = 0; j < CP; ++j) q[j] = B.nl[(size_t)min(c0 + cl + j * CG, P.nchunk - 1) * S_ + i];
            int uj[CP], src[CP], w[CP];
            bool vj[CP];
#pragma unroll
            for (int j = 0; j < CP; ++j) {
                const uint32_t wd = (e < 2) ? q[j].x : (e < 4) ? q[j].y : (e < 6) ? q[j].z : q[j].w;
                int u = (int)((wd >> (16 * (e & 1))) & 0xffffu);
                bool ok = c0 + cl + j * CG < nch;
                if (MULTI && xr) {
                    ok = ok && !(u >> 15);  // excluded pair: not counted
                    u &= 0x7fff;
                }
                vj[j] = ok && u < total;  // else padding of the last chunk
                uj[j] = vj[j] ? u : 0;
            }
#pragma unroll
            for (int j = 0; j < CP; ++j) {
                src[j] = sm[uj[j]];
                w[j] = wm[uj[j]];
            }
            double xj[CP][3];
#pragma unroll
            for (int j = 0; j < CP; ++j)
                for (int a = 0; a < 3; ++a) xj[j][a] = X[3 * src[j] + a];
#pragma unroll
            for (int j = 0; j < CP; ++j) {
                const double dx = xi0 - (xj[j][0] + L0 * (double)unpack_w(w[j], 0));
                const double dy = xi1 - (xj[j][1] + L1 * (double)unpack_w(w[j], 1));
                const double dz = xi2 - (xj[j][2] + L2 * (double)unpack_w(w[j], 2));
                const double r2 = (dx * dx + dy * dy) + dz * dz;
                if (MULTI) {
                    const int tj = B.type[src[j]];
                    if (vj[j] && ((R.mask[ti] >> tj) & 1u)) acc += count_term64(r2, R.pair[ti * MAXT + tj]);
                } else {
                    if (vj[j]) acc += count_term64(r2, p0);
                }
            }
        }
#pragma unroll
        for (int o = LANES / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, LANES);
        if (l == 0) {
            B.nd[i] = acc;
            sA[i] = R2{MULTI ? (Real)acc : (Real)omega_d64(acc, p0.x1, p0.x2), Real(0)};
            if (n_out) n_out[R.o_off + B.tag[i]] = acc;
        }
    }
}

template <int UN>
__device__ __forceinline__ double replica_sum(const Buffers &B, const RepDev &R);
template <int UN>
__device__ __forceinline__ void thermo_add(const Buffers &B, const RepDev &R, int r);

// STATS: also count the ordered pairs inside the interaction cutoff (the pair-evaluation
// statistic); the step loop samples it on one step in eight.
template <class Real, bool MULTI, bool STATS, bool ONE, bool SPLIT, bool LARGE>
__device__ __forceinline__ void count_brick(const Buffers &B, const Launch &P, int cur, double *__restrict__ n_out,
                                            int advance, const OneRep<ONE> &R1, int b)
{
    using R4 = typename V4<Real>::t;
    using R2 = typename V2<Real>::t;
    extern __shared__ __align__(32) unsigned char smem[];
    __shared__ int nwin;  // own particles inside a switching window
    __shared__ unsigned long long ev_sum;
    __shared__ PairR<Real> pt[1];
    __shared__ PairM<Real> pm[MULTI ? MAXT * MAXT : 1];
    const MapFirst mf = map_prefetch(B, b, P.stage_cap);
    // one fixed replica: its descriptor comes with the launch, no owner lookup
    const int r = ONE ? 0 : B.brick_rep[b];
    if (r < 0) return;
    const RepDev &R = rep_of<ONE>(R1, B, r);
    int lb = b - R.b_off;
    // the replica's first brick adds the energy and virial sums the last time step's force
    // pass left (with the sums on), after its own work
    const int pend = lb == 0 ? B.tpend[r] : 0;
    R4 *spos = (R4 *)smem;
    constexpr bool SOA = !MULTI && sizeof(Real) == 4;
    float2 *sxy = (float2 *)smem;
    // a pass over one replica in one launch has the whole capacity
    constexpr bool WHOLE = ONE && !SPLIT;
    const int cap = WHOLE ? P.stage_cap : P.lds_cap;
    float *sza = (float *)(sxy + cap + 1);
    const int64_t S_ = P.nslots;
    load_pairs<Real>(R, pt);
    if (MULTI) load_pairs_m<Real>(R, pm, threadIdx.x);
    if (threadIdx.x == 0) {
        nwin = 0;
        ev_sum = 0ull;
    }
    // every thread reads the header itself (uniform values), so that the staging gathers
    // need not wait for a barrier; the staging barrier orders pt, nwin and ev_sum
    StageHdr S;
    pass_header(R, B, b, lb, P.stage_cap, S);
    if (!LARGE && !WHOLE && S.total > P.t_hi) return;
    if (lb == 0 && threadIdx.x == 0) atomicAnd(&B.flags[r], ~(uint32_t)VBC_FLAG_REBUILD);
    R2 *sA = (R2 *)B.sA;
    if (S.overflow) {
        for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
            int64_t i = S.base + t;
            B.nd[i] = 0.0;
            sA[i] = R2{Real(0), Real(0)};
        }
        if (threadIdx.x == 0) {
            atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_STAGE_OVERFLOW);
            B.wcnt[b] = 0;
        }
        if (pend) thermo_add<1>(B, R, r);
        return;
    }
    const double *X = B.x[cur];
    constexpr bool AHEAD = ONE && !SPLIT && !MULTI;
    ListHead head;
    if (AHEAD) head = list_head(B, S.base + min((int)threadIdx.x, R.bcap - 1));
    // an empty brick stages nothing (many small replicas; a single one has few)
    if (ONE || S.n_own > 0) stage_map4(B, b, P.stage_cap, S, mf, [&](int t, int src, int w, bool ok) {
        const R4 p = local_pos<Real>(R, S, X, S_, src, w, MULTI ? B.type[src] : 0);
        if (ok) {
            if (SOA) {
                sxy[t] = make_float2((float)p.x, (float)p.y);
                sza[t] = (float)p.z;
            } else {
                spos[t] = p;
            }
        }
    });
    if (threadIdx.x == 0) {
        if (SOA) {
            sxy[S.total] = make_float2(1.0e6f, 1.0e6f);
            sza[S.total] = 1.0e6f;
        } else {
            spos[S.total] = dummy_pos<R4>();
        }
    }
    __syncthreads();

    const PairR<Real> p0 = pt[0];
    const bool xr = R.excl_span > 0;  // list entries carry the exclusion bit 15
    // read once: the global descriptor cannot be kept in registers across the stores below
    const double wx1 = R.pair[0].x1, wx2 = R.pair[0].x2;
    const bool watt = R.pair[0].attract;
    const int64_t o_off = R.o_off;
    unsigned long long evals = 0;
    const int ls = SPLIT ? P.split : 0, sub = SPLIT ? threadIdx.x & ((1 << ls) - 1) : 0;
    for (int t = threadIdx.x >> ls; t < S.n_own; t += blockDim.x >> ls) {
        int64_t i = S.base + t;
        R4 pi;
        if (SOA) {
            const float2 q = sxy[t];
            pi.x = q.x;
            pi.y = q.y;
            pi.z = sza[t];
            pi.w = 0;
        } else {
            pi = spos[t];
        }
        int ti = MULTI ? (int)pi.w : 0;
        int inside = 0;
        double n = 0.0;
        Real chunk = Real(0);
        int e = 0;
        // omega(r, r_l, r_h) = (1 - u^2)^2 with u = clamp((r - r_l)/(r_h - r_l), 0, 1): exactly 1
        // inside r_l and 0 beyond r_h; partial sums of eight terms are added in FP64
        auto entry = [&](int u) {
            int ex = 0;  // pair excluded from counting and attraction (chain neighbours)
            if (MULTI && xr) {
                ex = u >> 15;
                u &= 0x7fff;
            }
            R4 pj;
            if (SOA) {
                const float2 q = sxy[u];
                pj.x = q.x;
                pj.y = q.y;
                pj.z = sza[u];
                pj.w = 0;
            } else {
                pj = spos[u];
            }
            Real dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
            Real r2 = dx * dx + dy * dy + dz * dz;
            if (STATS) inside += (r2 < p0.rc2) ? 1 : 0;
            Real rr = sqrt_r(r2);
            if (MULTI) {
                const PairM<Real> &q = pm[ti * MAXT + (int)pj.w];
                const R4 g = q.geo;
                Real uu = clamp01(fma(rr, g.z, g.w));
                Real qq = fma(-uu, uu, Real(1));
                // c_c is not zero where i counts j
                qq = (q.cnt.x == Real(0) || ex) ? Real(0) : qq;
                chunk = fma(qq, qq, chunk);
            } else {
                Real uu = clamp01(fma(rr, p0.inv_dw, p0.nrl_dw));
                Real qq = fma(-uu, uu, Real(1));
                chunk = fma(qq, qq, chunk);
            }
            if (!SPLIT && ++e == CHUNK) {
                n += (double)chunk;
                chunk = Real(0);
                e = 0;
            }
        };
        if constexpr (SPLIT)
            for_each_neighbour_shared(B.nl, S_, i, B.nn[i], sub, ls, entry, [&]() {
                n = add_group(n, (double)chunk, ls);
                chunk = Real(0);
            });
        else for_each_neighbour(B.nl, S_, i, AHEAD && t == (int)threadIdx.x ? head : list_head(B, i), entry, []() {});
        evals += (unsigned long long)inside;
        if (SPLIT && sub) continue;
        B.nd[i] = n;
        bool win = false;
        // with FP32 pair arithmetic the window is widened by the margin: the particles
        // listed get their counts again in FP64 below, before anything reads them
        const double mg = sizeof(Real) == 4 ? COUNT_MARGIN : 0.0;
        if (MULTI) {
            // the switching factor depends on the pair: keep the count itself
            sA[i] = R2{(Real)n, Real(0)};
            for (int u = 0; u < R.ntypes; ++u) {
                const PairDev &pd = R.pair[ti * MAXT + u];
                if (pd.attract && n > pd.x1 - mg && n < pd.x2 + mg) win = true;
            }
        } else {
            sA[i] = R2{(Real)omega_d64(n, wx1, wx2), Real(0)};
            win = watt && n > wx1 - mg && n < wx2 + mg;
        }
        // the dU/dn pass visits only these: list them compactly in the brick's slots
        if (win) B.wlst[S.base + atomicAdd(&nwin, 1)] = (uint16_t)t;
        if (n_out) n_out[o_off + B.tag[i]] = n;
    }
    if (STATS) {
        evals = wave_sum(evals);
        if ((threadIdx.x % VBC_WAVE) == 0 && evals) atomicAdd(&ev_sum, evals);
    }
    __syncthreads();
    if (sizeof(Real) == 4) {
        // the listed entries are in global memory, written by this workgroup before the barrier
        const int nwv = nwin;
        // as many lanes per listed particle (32, 16 or 8) as one round of some threads allows: 32
        // take a list of up to 32 entries in one phase, 16 in two, 8 in four.  The lanes order
        // the sum, so their number follows the brick's particles and the replica alone, not the
        // workgroup: a count has the same bits at every workgroup size, alone and in a pool.
        // Longer lists are worth more lanes and a further round of a small workgroup (us for ten
        // steps and a frame: melt of 250,000, lists of 49, 1035 at a round of 256 and 1021 at
        // 512; dilute 10,000, lists of 3, 246 at 256 and 254 at 512; twenty tracked sets of 4000
        // alike 784 at 256 and 795 at 512, and 778 at the 128 threads that they have)
        const int round = R.recount_round;
        if (nwv > 0 && nwv * 32 <= round)
            recount_window<Real, MULTI, 32, 1>(B, P, R, b, S.total, S.base, nwv, X, n_out);
        else if (nwv > 0 && nwv * 16 <= round)
            recount_window<Real, MULTI, 16, 1>(B, P, R, b, S.total, S.base, nwv, X, n_out);
        else if (nwv > 0)
            recount_window<Real, MULTI, CHUNK, 1>(B, P, R, b, S.total, S.base, nwv, X, n_out);
    }
    if (threadIdx.x == 0) {
        B.wcnt[b] = nwin;
        if (STATS) B.bevals[b] += ev_sum;  // this workgroup is the only writer of brick b
        if (lb == 0) {
            if (STATS) B.stats[4 * r + 3] += 1ull;
            // in a time step the count pass opens the step: the step counter (the noise
            // counter of the Langevin O-step that the following force pass starts) advances
            if (advance) B.step[r] += 1ull;
        }
    }
    if (pend) thermo_add<1>(B, R, r);
}

template <class Real, bool MULTI, bool STATS, bool ONE, bool SPLIT>
__global__ void __attribute__((amdgpu_waves_per_eu(8))) k_count(Buffers B, Launch P, int cur, double *__restrict__ n_out, int advance, OneRep<ONE> R1)
{
    int b;
    if (brick_of_block(P, B, b)) count_brick<Real, MULTI, STATS, ONE, SPLIT, false>(B, P, cur, n_out, advance, R1, b);
}

template <class Real, bool MULTI, bool STATS>
__global__ void __launch_bounds__(DENSE_BLOCK) k_count_dense(Buffers B, Launch P, int cur, double *__restrict__ n_out, int advance)
{
    each_dense(P, B, [&](int b) {
        count_brick<Real, MULTI, STATS, false, false, true>(B, P, cur, n_out, advance, OneRep<false>{0}, b);
    });
}

// ---------------------------------------------------------------------------
// pass 2a: dU/dn for particles inside a switching window
// ---------------------------------------------------------------------------

// Waves per workgroup of the dU/dn pass; one workgroup per brick.
constexpr int EMBED_WAVES = 4;

// dU/dn of the window particles of brick b that fall to group g of ng groups of LPP lanes
// (particles g, g + ng, ...; see k_embed).  t_first: the first particle of this lane's
// group if already read, else -1.
template <int LPP, class Real, bool MULTI>
__device__ __forceinline__ void embed_brick(const Buffers &B, const Launch &P, const RepDev &R,
                                            const PairM<Real> *pm, int b, int total, int64_t base, int nw,
                                            int lane, int g, int ng, int t_first, int cur)
{
    using R4 = typename V4<Real>::t;
    // LPP lanes per window particle, EP entries of each list chunk per lane; neighbours are
    // gathered from global memory through the brick's staging map
    using R2 = typename V2<Real>::t;
    constexpr int EP = CHUNK / LPP;
    const int64_t S_ = P.nslots;
    R2 *sA = (R2 *)B.sA;
    const double *X = B.x[cur];
    const int32_t *sm = B.smap + (size_t)b * P.stage_cap;
    const uint8_t *wm = B.wmap + (size_t)b * P.stage_cap;
    const PairR<Real> p0 = pair_r<Real>(R.pair[0], R.rc2);
    const bool xr = R.excl_span > 0;
    const int e = lane % LPP;
    for (int k = g; k < nw; k += ng) {
        int t = (k == g && t_first >= 0) ? t_first : B.wlst[base + k];
        int64_t i = base + t;
        double n_i = B.nd[i];
        int ti = MULTI ? B.type[i] : 0;
        const double xi0 = X[3 * i], xi1 = X[3 * i + 1], xi2 = X[3 * i + 2];
        int nch = (B.nn[i] + CHUNK - 1) / CHUNK;
        double acc = 0.0;
        // four chunks at a time in phases (chunk words, staging map, positions, terms)
        // with no branch between the loads, so that the gathers of all four go out together;
        // rows past the list and the padding slot read valid memory and are masked.  The
        // first four rows are read before the list length arrives (rows below nchunk exist
        // for every slot).
        constexpr int CP = 4 / EP;  // chunks per phase
        uint4 qf[CP];
#pragma unroll
        for (int j = 0; j < CP; ++j) qf[j] = B.nl[(size_t)min(j, P.nchunk - 1) * S_ + i];
        for (int c0 = 0; c0 < nch; c0 += CP) {
            int uj[4], sj[4], wj[4];
            bool vj[4];
            uint4 qc[CP];
#pragma unroll
            for (int j = 0; j < CP; ++j)
                qc[j] = c0 == 0 ? qf[j] : B.nl[(size_t)min(c0 + j, P.nchunk - 1) * S_ + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int jc = j / EP, x = e + LPP * (j % EP);  // chunk, entry
                const uint4 q = qc[jc];
                const uint32_t wd = (x < 2) ? q.x : (x < 4) ? q.y : (x < 6) ? q.z : q.w;
                int u = (int)((wd >> (16 * (x & 1))) & 0xffffu);
                bool ok = c0 + jc < nch;
                if (MULTI && xr) {
                    ok = ok && !(u >> 15);  // excluded pair: no attraction between them
                    u &= 0x7fff;
                }
                vj[j] = ok && u < total;
                uj[j] = vj[j] ? u : 0;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sj[j] = sm[uj[j]];
                wj[j] = wm[uj[j]];
            }
            double xj[4][3];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                for (int a = 0; a < 3; ++a) xj[j][a] = X[3 * sj[j] + a];
            Real sjv[4];
            int tj[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sjv[j] = sA[sj[j]].x;
                tj[j] = MULTI ? B.type[sj[j]] : 0;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                Real dx = (Real)(xi0 - (xj[j][0] + R.L[0] * (double)unpack_w(wj[j], 0)));
                Real dy = (Real)(xi1 - (xj[j][1] + R.L[1] * (double)unpack_w(wj[j], 1)));
                Real dz = (Real)(xi2 - (xj[j][2] + R.L[2] * (double)unpack_w(wj[j], 2)));
                Real r2 = dx * dx + dy * dy + dz * dz;
                if (MULTI) {
                    // s'_ij(n_i) in FP64 by the pair's window; no attraction: E_a = 0
                    const PairM<Real> &q2 = pm[ti * MAXT + tj[j]];
                    const R4 qg = q2.geo;
                    const Real uu = fma(sqrt_r(r2), qg.x, qg.y);
                    const Real qq = fma(-uu, uu, Real(1));
                    if (vj[j] && qq > Real(0)) {
                        const double x1 = R.pair[ti * MAXT + tj[j]].x1;
                        acc += omega_dd64(n_i, x1, x1 + 1.0) *
                               (double)(omega_win<Real>(sjv[j], q2.core.w) * (-q2.cnt.w * qq * qq));
                    }
                } else {
                    Real uu = (sqrt_r(r2) - p0.m) * p0.inv_w;
                    Real qq = Real(1) - uu * uu;
                    if (vj[j] && qq > Real(0)) acc += (double)(sjv[j] * (-p0.E_a * qq * qq));
                }
            }
        }
        // fixed-order reduction over the lanes of the group
#pragma unroll
        for (int o = LPP / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, LPP);
        if (e == 0) {
            double A = MULTI ? acc : omega_dd64(n_i, R.pair[0].x1, R.pair[0].x2) * acc;
            sA[i].y = (Real)A;
        }
    }
}

// One workgroup of EMBED_WAVES waves per brick over the particles that the count pass
// listed as inside a switching window; most bricks hold a handful or none, and then only
// the first wave works.  No workgroup-wide synchronisation.
template <class Real, bool MULTI>
__global__ void k_embed(Buffers B, Launch P, int cur)
{
    __shared__ PairM<Real> ptab[EMBED_WAVES][MULTI ? MAXT * MAXT : 1];
    const int wv = threadIdx.x / VBC_WAVE, lane = threadIdx.x % VBC_WAVE;
    int b;
    if (!brick_of_block(P, B, b)) return;
    // the brick's owner, window count and staged count read together: most bricks have no
    // window particle and leave here; then the replica descriptor and the first window entry
    const int r = B.brick_rep[b];
    const int nw = B.wcnt[b];
    const int tot = B.stotal[b];
    // free brick, nothing in a window, or an overflowed brick
    if (r < 0 || nw == 0 || tot > P.stage_cap) return;
    const RepDev &R = B.reps[r];
    const int lb = b - R.b_off;
    const int64_t base = R.p_off + (int64_t)lb * R.bcap;
    const int t_first = B.wlst[base + lane / CHUNK];  // for eight lanes per particle
    // eight lanes per particle when the first wave takes all of the brick's window particles
    // at once; up to EMBED_WAVES x 8 of them, eight lanes each over every wave; with more,
    // four lanes each over every wave, so that up to EMBED_WAVES x 16 are in flight
    const bool one = nw <= VBC_WAVE / CHUNK;
    if (one && wv > 0) return;
    PairM<Real> *pm = ptab[wv];
    if (MULTI) {
        load_pairs_m<Real>(R, pm, lane);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (one) {
        embed_brick<CHUNK, Real, MULTI>(B, P, R, pm, b, tot, base, nw, lane, lane / CHUNK, VBC_WAVE / CHUNK,
                                        t_first, cur);
    } else if (nw <= EMBED_WAVES * (VBC_WAVE / CHUNK)) {
        // up to 32: eight lanes each over every wave, all of them in one round
        constexpr int G = VBC_WAVE / CHUNK;
        embed_brick<CHUNK, Real, MULTI>(B, P, R, pm, b, tot, base, nw, lane, wv * G + lane / CHUNK,
                                        EMBED_WAVES * G, -1, cur);
    } else {
        constexpr int G = VBC_WAVE / 4;  // groups of four lanes per wave
        embed_brick<4, Real, MULTI>(B, P, R, pm, b, tot, base, nw, lane, wv * G + lane / 4, EMBED_WAVES * G,
                                    -1, cur);
    }
}

// ---------------------------------------------------------------------------
// pass 2b: forces, energies, virial, fused integration
// ---------------------------------------------------------------------------

// Velocity / position update of one particle, in the same order of operations as the
// plain integrator (no contraction): closing half-kick of the previous step, then the
// opening half-kick and the drift of the next one.
__device__ __forceinline__ void integrate_one(const StepArgs &st, int mode, bool first_kick,
                                              const double F[3], double v[3], double x[3],
                                              uint64_t seed, uint64_t tag, uint64_t step)
{
#pragma clang fp contract(off)
    if (!first_kick)
        for (int a = 0; a < 3; ++a) v[a] = v[a] + st.hdt * F[a];
    if (mode == MODE_LAST) return;
    for (int a = 0; a < 3; ++a) v[a] = v[a] + st.hdt * F[a];
    if (st.kind == VBC_NVE) {
        for (int a = 0; a < 3; ++a) x[a] = x[a] + st.dt * v[a];
    } else {
        for (int a = 0; a < 3; ++a) x[a] = x[a] + st.hdt * v[a];
        double xi[3];
        langevin_noise(seed, tag, step, xi);
        for (int a = 0; a < 3; ++a) v[a] = st.c1 * v[a] + st.c2s * xi[a];
        for (int a = 0; a < 3; ++a) x[a] = x[a] + st.hdt * v[a];
    }
}

template <class Real, bool MULTI, bool THERMO, bool ONE, bool SPLIT, bool LARGE>
__device__ __forceinline__ void force_brick(const Buffers &B, const Launch &P, int cur, int mode, const StepArgs &st,
                                            double *__restrict__ F_out, double *__restrict__ e_out,
                                            const OneRep<ONE> &R1, int b)
{
    using R4 = typename V4<Real>::t;
    using R2 = typename V2<Real>::t;
    extern __shared__ __align__(32) unsigned char smem[];
    __shared__ PairR<Real> pt[1];
    __shared__ PairM<Real> pm[MULTI ? MAXT * MAXT : 1];
    __shared__ double red[8][1024 / VBC_WAVE];
    __shared__ int moved;
    const MapFirst mf = map_prefetch(B, b, P.stage_cap);
    const int r = ONE ? 0 : B.brick_rep[b];
    if (r < 0) return;
    const RepDev &R = rep_of<ONE>(R1, B, r);
    int lb = b - R.b_off;
    // staged per particle: position and, with one type, the switching factor s in .w plus
    // c_c A in a separate array (20 bytes in FP32); with several types the type in .w and
    // (s or n, A) beside it
    R4 *spos = (R4 *)smem;
    constexpr bool WHOLE = ONE && !SPLIT;  // as in the count pass
    const int cap = WHOLE ? P.stage_cap : P.lds_cap;
    R2 *ssa = (R2 *)(spos + cap + 1);
    Real *scA = (Real *)(spos + cap + 1);
    const int64_t S_ = P.nslots;
    const int64_t ntot = P.ntot;
    load_pairs<Real>(R, pt);
    if (MULTI) load_pairs_m<Real>(R, pm, threadIdx.x);
    if (threadIdx.x == 0) moved = 0;
    // every thread reads the header itself (as in the count pass); the staging barrier
    // orders pt and moved
    StageHdr S;
    pass_header(R, B, b, lb, P.stage_cap, S);
    if (!LARGE && !WHOLE && S.total > P.t_hi) return;
    const R2 *sA = (const R2 *)B.sA;
    if (S.overflow) {
        if (threadIdx.x == 0) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_STAGE_OVERFLOW);
        if (THERMO && threadIdx.x < 8) B.part[(size_t)b * 8 + threadIdx.x] = 0.0;
        if (THERMO && st.acc && lb == 0 && threadIdx.x == 0) B.tpend[r] = 1;
        return;
    }
    const double *X = B.x[cur];
    const Real cc0 = pair_r<Real>(R.pair[0], R.rc2).c_c;
    constexpr bool AHEAD = ONE && !SPLIT && !MULTI;
    ListHead head;
    if (AHEAD) head = list_head(B, S.base + min((int)threadIdx.x, R.bcap - 1));
    if (ONE || S.n_own > 0) stage_map4(B, b, P.stage_cap, S, mf, [&](int t, int src, int w, bool ok) {
        R4 p = local_pos<Real>(R, S, X, S_, src, w, MULTI ? B.type[src] : 0);
        const R2 sa = sA[src];
        if (!MULTI) p.w = sa.x;
        if (ok) {
            spos[t] = p;
            if (MULTI) ssa[t] = sa;
            else scA[t] = sa.y * cc0;  // one type: the chain-rule term needs only c_c A
        }
    });
    if (threadIdx.x == 0) {
        spos[S.total] = dummy_pos<R4>();
        if (MULTI) ssa[S.total] = R2{Real(0), Real(0)};
        else scA[S.total] = Real(0);
    }
    __syncthreads();

    const PairR<Real> p0 = pt[0];
    const bool xr = R.excl_span > 0;  // list entries carry the exclusion bit 15
    // read once: the global descriptor cannot be kept in registers across the stores below
    const int chain_len = R.chain_len;
    const double disp2 = R.disp2;
    const int64_t o_off = R.o_off;
    const uint64_t step = B.step[r];
    const uint64_t key = st.seed + R.seed;
    // e, -, Wxx, Wyy, Wzz, Wxy, Wxz, Wyz; the scalar virial W is the trace, formed per brick
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    bool bad = false, mv = false;
    const int ls = SPLIT ? P.split : 0, sub = SPLIT ? threadIdx.x & ((1 << ls) - 1) : 0;
    auto particle = [&](int t) __attribute__((always_inline)) {
        int64_t i = S.base + t;
        R4 pi = spos[t];
        const R2 sai = MULTI ? ssa[t] : R2{pi.w, scA[t]};
        int ti = MULTI ? (int)pi.w : 0;
        const Real cai = p0.c_a * sai.x;
        // ei: pair energies (several types), or with one type sum tc^2 and ea sum s_j q_a^2,
        // which E_r and E_a s_i scale once per particle
        // FP64 forces are summed chunk by chunk, the order that lanes sharing a list can keep
        constexpr bool CHUNKED = sizeof(Real) == 8;
        Real fx = 0, fy = 0, fz = 0, ei = 0, ea = 0;
        Real cx = 0, cy = 0, cz = 0;
        Real wxx = 0, wyy = 0, wzz = 0, wxy = 0, wxz = 0, wyz = 0;
        auto entry = [&](int u) {
            int ex = 0;  // pair excluded from counting and attraction (chain neighbours)
            if (MULTI && xr) {
                ex = u >> 15;
                u &= 0x7fff;
            }
            R4 pj = spos[u];
            Real dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
            Real r2 = dx * dx + dy * dy + dz * dz;
            Real phr, ep;
            if (MULTI) {
                // branch-free like the one-type path below, with the pair's constants in three
                // LDS reads; an excluded pair neither counts nor attracts
                const PairM<Real> &q = pm[ti * MAXT + (int)pj.w];
                const R4 qc = q.core, qg = q.geo, qn = q.cnt;
                const R2 saj = ssa[u];
                const Real rinv = rsqrt_r(r2 > Real(1e-30) ? r2 : Real(1e-30));
                const Real rr = r2 * rinv;
                const Real pr = fmin(fma(r2, qc.y, qc.x), Real(0));
                const Real uu = fma(rr, qg.x, qg.y);
                const Real qq = fmax(fma(-uu, uu, Real(1)), Real(0));
                Real psi = omega_win<Real>(sai.x, qc.w) * omega_win<Real>(saj.x, qc.w);
                Real asum = fma(qn.x, sai.y, qn.y * saj.y);
                if (xr && ex) psi = asum = Real(0);
                const Real uc = clamp01(fma(rr, qg.z, qg.w));
                const Real g = uc * fma(-uc, uc, Real(1));
                phr = fma(fma(asum, g, qc.z * psi * uu * qq), rinv, pr);
                // E_r (1 - r^2/r_r^2)^2 = (V_r'/r)^2 E_r / c_r^2
                ep = fma(pr * pr, qn.z, -(qn.w * psi * qq * qq));
            } else {
                // branch-free: beyond every cutoff (and for the padding slot) all three terms
                // vanish through the clamps.  phi/r = min(c_r + k_r r^2, 0)
                //   + [ c_a s_i s_j u_a q_a + (c_c A_i + c_c A_j) u_c (1 - u_c^2) ] / r
                const Real sj = pj.w, cAj = scA[u];
                Real rinv = rsqrt_r(r2 > Real(1e-30) ? r2 : Real(1e-30));
                Real rr = r2 * rinv;
                Real pr = fmin(fma(r2, p0.k_r, p0.c_r), Real(0));
                Real uu = fma(rr, p0.inv_w, p0.nm_w);
                Real qq = fmax(fma(-uu, uu, Real(1)), Real(0));
                Real uc = clamp01(fma(rr, p0.inv_dw, p0.nrl_dw));
                Real g = uc * fma(-uc, uc, Real(1));
                Real t = fma(sai.y + cAj, g, cai * sj * uu * qq);
                phr = fma(t, rinv, pr);
                if (THERMO) {
                    const Real tc = fmax(fma(-r2, p0.inv_rr2, Real(1)), Real(0));
                    ei = fma(tc, tc, ei);
                    ea = fma(sj * qq, qq, ea);
                }
            }
            if (CHUNKED) {
                cx -= phr * dx;
                cy -= phr * dy;
                cz -= phr * dz;
            } else {
                fx -= phr * dx;
                fy -= phr * dy;
                fz -= phr * dz;
            }
            if (THERMO) {
                if (MULTI) ei += ep;
                wxx -= phr * dx * dx;
                wyy -= phr * dy * dy;
                wzz -= phr * dz * dz;
                wxy -= phr * dx * dy;
                wxz -= phr * dx * dz;
                wyz -= phr * dy * dz;
            }
        };
        if constexpr (SPLIT) {
            static_assert(CHUNKED && !THERMO, "only forces are shared between lanes");
            for_each_neighbour_shared(B.nl, S_, i, B.nn[i], sub, ls, entry, [&]() {
                fx = add_group(fx, cx, ls);
                fy = add_group(fy, cy, ls);
                fz = add_group(fz, cz, ls);
                cx = cy = cz = Real(0);
            });
            if (sub) return;
        } else {
            for_each_neighbour(B.nl, S_, i, AHEAD && t == (int)threadIdx.x ? head : list_head(B, i), entry, [&]() {
                if (CHUNKED) {
                    fx += cx;
                    fy += cy;
                    fz += cz;
                    cx = cy = cz = Real(0);
                }
            });
        }
        double F[3] = {(double)fx, (double)fy, (double)fz};
        double eb = 0.0, wb[7] = {0, 0, 0, 0, 0, 0, 0};
        double xi_[3] = {X[3 * i], X[3 * i + 1], X[3 * i + 2]};
        int32_t tg = B.tag[i];
        if (chain_len > 1) {
            // harmonic bonds to the neighbouring beads of the same chain
            int bead = tg % chain_len;
            for (int side = -1; side <= 1; side += 2) {
                if ((side < 0 && bead == 0) || (side > 0 && bead == chain_len - 1)) continue;
                int64_t j = B.inv[o_off + tg + side];
                double d[3];
                for (int a = 0; a < 3; ++a) {
                    double tt = xi_[a] - X[3 * j + a];
                    d[a] = tt - R.L[a] * rint(tt / R.L[a]);
                }
                double rb = sqrt((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]);
                double dr = rb - R.r0_bond;
                double cf = rb > 0.0 ? R.k_bond * dr / rb : 0.0;
                for (int a = 0; a < 3; ++a) F[a] -= cf * d[a];
                if (THERMO) {
                    eb += 0.25 * R.k_bond * dr * dr;
                    wb[0] -= 0.5 * cf * rb * rb;
                    wb[1] -= 0.5 * cf * d[0] * d[0];
                    wb[2] -= 0.5 * cf * d[1] * d[1];
                    wb[3] -= 0.5 * cf * d[2] * d[2];
                    wb[4] -= 0.5 * cf * d[0] * d[1];
                    wb[5] -= 0.5 * cf * d[0] * d[2];
                    wb[6] -= 0.5 * cf * d[1] * d[2];
                }
            }
        }
        if (!(isfinite(F[0]) && isfinite(F[1]) && isfinite(F[2]))) bad = true;
        if (THERMO) {
            const Real e_pair = MULTI ? ei : p0.E_r * ei - p0.E_a * sai.x * ea;
            double e_i = 0.5 * (double)e_pair + eb;
            acc[0] += e_i;
            acc[2] += 0.5 * (double)wxx + wb[1];
            acc[3] += 0.5 * (double)wyy + wb[2];
            acc[4] += 0.5 * (double)wzz + wb[3];
            acc[5] += 0.5 * (double)wxy + wb[4];
            acc[6] += 0.5 * (double)wxz + wb[5];
            acc[7] += 0.5 * (double)wyz + wb[6];
            if (e_out) e_out[o_off + tg] = e_i;
        }
        if (mode == MODE_EVAL) {
            for (int a = 0; a < 3; ++a) B.Fst[a * S_ + i] = F[a];
            if (F_out)
                for (int a = 0; a < 3; ++a) F_out[a * ntot + o_off + tg] = F[a];
        } else {
            double vv[3] = {B.v[i], B.v[S_ + i], B.v[2 * S_ + i]};
            double xx[3] = {xi_[0], xi_[1], xi_[2]};
            integrate_one(st, mode, false, F, vv, xx, key, (uint64_t)tg, step);
            for (int a = 0; a < 3; ++a) B.v[a * S_ + i] = vv[a];
            if (mode == MODE_LAST) {
                for (int a = 0; a < 3; ++a) B.Fst[a * S_ + i] = F[a];
            } else {
                double *Xn = B.x[cur ^ 1];
                double d2 = 0.0;
                for (int a = 0; a < 3; ++a) {
                    Xn[3 * i + a] = xx[a];
                    double dd = xx[a] - B.xs[3 * i + a];
                    d2 += dd * dd;
                }
                if (d2 > disp2) mv = true;
            }
        }
    };
    if constexpr (THERMO) {
        // the sums of 64 consecutive particles (a wave's) are added in their order, round after
        // round of the workgroup: the same bits at every workgroup size.  The first round, with
        // which nearly every brick ends, stands by itself (an evaluation of 200,000 particles in
        // FP64: 175 us, 179 with it in the loop, 176 before); red holds the sums of as many
        // rounds as it has places for, so that few bricks meet a further barrier
        const int n_own = __builtin_amdgcn_readfirstlane(S.n_own);  // a scalar: barriers below
        const int wv = threadIdx.x / VBC_WAVE, ln = threadIdx.x % VBC_WAVE, nw = blockDim.x / VBC_WAVE;
        double s = 0.0;
        auto keep = [&](int at) __attribute__((always_inline)) {
            const double v = wave_sum8(acc);
            if ((ln & 7) == 0) red[ln >> 3][at + wv] = v;
        };
        auto add = [&](int n) __attribute__((always_inline)) {
            if (threadIdx.x == 1) {
                // W = W_xx + W_yy + W_zz, summed per wave in the same fixed order
                for (int w = 0; w < n; ++w) s += (red[2][w] + red[3][w]) + red[4][w];
            } else if (threadIdx.x < 8) {
                for (int w = 0; w < n; ++w) s += red[threadIdx.x][w];
            }
        };
        if ((int)threadIdx.x < n_own) particle(threadIdx.x);
        if (wv * VBC_WAVE < n_own) keep(0);
        int at = nw, done = 0;  // places of red given out, sums added
        for (int t0 = blockDim.x; t0 < n_own; t0 += blockDim.x) {
            if (at + nw > 1024 / VBC_WAVE) {
                __syncthreads();
                add(at);
                __syncthreads();
                done += at;
                at = 0;
            }
            if (t0 + wv * VBC_WAVE < n_own) {
                for (int k = 0; k < 8; ++k) acc[k] = 0.0;
                if (t0 + (int)threadIdx.x < n_own) particle(t0 + threadIdx.x);
                keep(at);
            }
            at += nw;
        }
        if (mv) moved = 1;
        __syncthreads();
        add((n_own + VBC_WAVE - 1) / VBC_WAVE - done);
        if (threadIdx.x < 8) B.part[(size_t)b * 8 + threadIdx.x] = s;
        // a time step's sums: added by the next count pass or the call's closing reduction
        if (st.acc && lb == 0 && threadIdx.x == 0) B.tpend[r] = 1;
    } else {
        for (int t = threadIdx.x >> ls; t < S.n_own; t += blockDim.x >> ls) particle(t);
        if (mv) moved = 1;
        __syncthreads();
    }
    if (bad) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_NONFINITE);
    if (threadIdx.x == 0 && moved) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_REBUILD);
}

template <class Real, bool MULTI, bool THERMO, bool ONE, bool SPLIT>
__global__ void k_force(Buffers B, Launch P, int cur, int mode, StepArgs st,
                        double *__restrict__ F_out, double *__restrict__ e_out, OneRep<ONE> R1)
{
    int b;
    if (brick_of_block(P, B, b))
        force_brick<Real, MULTI, THERMO, ONE, SPLIT, false>(B, P, cur, mode, st, F_out, e_out, R1, b);
}

template <class Real, bool MULTI, bool THERMO>
__global__ void __launch_bounds__(DENSE_BLOCK) k_force_dense(Buffers B, Launch P, int cur, int mode, StepArgs st,
                                                             double *__restrict__ F_out, double *__restrict__ e_out)
{
    each_dense(P, B, [&](int b) {
        force_brick<Real, MULTI, THERMO, false, false, true>(B, P, cur, mode, st, F_out, e_out, OneRep<false>{0}, b);
    });
}

// Opening half-kick and drift of the first step of a call, from the forces kept in Fst;
// one workgroup per brick.
__global__ void k_kick_drift(Buffers B, Launch P, int cur, StepArgs st)
{
    int b, r;
    if (!resolve_brick(P, B, b, r)) return;
    const RepDev &R = B.reps[r];
    const int64_t S_ = P.nslots;
    const int64_t base = R.p_off + (int64_t)(b - R.b_off) * R.bcap;
    const int nown = B.bcnt[0][b];
    const uint64_t key = st.seed + R.seed, step = B.step[r];
    bool far = false;
    for (int t = threadIdx.x; t < nown; t += blockDim.x) {
        int64_t i = base + t;
        double F[3], v[3], x[3];
        for (int a = 0; a < 3; ++a) {
            F[a] = B.Fst[a * S_ + i];
            v[a] = B.v[a * S_ + i];
            x[a] = B.x[cur][3 * i + a];
        }
        integrate_one(st, MODE_MID, true, F, v, x, key, (uint64_t)B.tag[i], step);
        double d2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            B.v[a * S_ + i] = v[a];
            B.x[cur ^ 1][3 * i + a] = x[a];
            double dd = x[a] - B.xs[3 * i + a];
            d2 += dd * dd;
        }
        far = far || d2 > R.disp2;
    }
    if (__syncthreads_or(far) && threadIdx.x == 0)
        atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_REBUILD);
}

// The eight sums of replica R's per-brick partial sums, in an order that does not depend on
// the workgroup's size (the count pass and the closing reduction run it with different
// sizes): lane l of the first wave adds bricks l, l + 64, ..., then the wave's lanes are
// added in the fixed order of wave_sum, whatever UN, the bricks each lane has in flight (1600
// bricks take 12.1 us with one, the latency of 25 dependent rounds; the count pass keeps one,
// to stay within its registers, in a workgroup that is not its last).  Called by the whole
// workgroup; thread k < 8 gets component k.
template <int UN>
__device__ __forceinline__ double replica_sum(const Buffers &B, const RepDev &R)
{
    __shared__ double red[8];
    if (threadIdx.x < VBC_WAVE) {
        double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const double *part = B.part + (size_t)R.b_off * 8;
        for (int b0 = threadIdx.x; b0 < R.nbrick; b0 += UN * VBC_WAVE) {
            // a brick past the end reads the lane's first one of the round and adds nothing
            double q[UN][8];
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int b = b0 + j * VBC_WAVE < R.nbrick ? b0 + j * VBC_WAVE : b0;
#pragma unroll
                for (int k = 0; k < 8; ++k) q[j][k] = part[(size_t)b * 8 + k];
            }
#pragma unroll
            for (int j = 0; j < UN; ++j)
                if (b0 + j * VBC_WAVE < R.nbrick)
                    for (int k = 0; k < 8; ++k) acc[k] += q[j][k];
        }
        for (int k = 0; k < 8; ++k) {
            const double v = wave_sum(acc[k]);
            if (threadIdx.x == 0) red[k] = v;
        }
    }
    __syncthreads();
    return threadIdx.x < 8 ? red[threadIdx.x] : 0.0;
}

// Per-replica totals from the per-brick partial sums, in brick order.
__global__ void k_reduce(Buffers B, int nrep, double *__restrict__ UW)
{
    int r = blockIdx.x;
    const RepDev &R = B.reps[r];
    const double s = replica_sum<4>(B, R);
    if (threadIdx.x < 8) UW[r * 8 + threadIdx.x] = s;
}

// A time step's energy and virial of replica r (kept as the last step's) added to its
// running sums from the per-brick sums its force pass left, and its step count raised by
// one; the pending mark cleared.  Called by a whole workgroup.
template <int UN>
__device__ __forceinline__ void thermo_add(const Buffers &B, const RepDev &R, int r)
{
    const double s = replica_sum<UN>(B, R);
    if (threadIdx.x < 8) {
        double *T = B.thermo + (size_t)r * THERMO_WORDS;
        T[1 + threadIdx.x] = s;
        T[9 + threadIdx.x] += s;
        if (threadIdx.x == 0) {
            T[0] += 1.0;
            B.tpend[r] = 0;
        }
    }
}

// At the end of a call with the sums on: the last step's sums of every replica with sums
// pending (a slot is live when its first brick is owned by it; retired descriptors stay
// behind).
__global__ void k_thermo_acc(Buffers B, int nrep)
{
    const int r = blockIdx.x;
    const RepDev &R = B.reps[r];
    if (!B.tpend[r]) return;
    if (R.nbrick <= 0 || B.brick_rep[R.b_off] != r) {
        if (threadIdx.x == 0) B.tpend[r] = 0;
        return;
    }
    thermo_add<4>(B, R, r);
}

__global__ void k_thermo_clear(Buffers B, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        B.thermo[i] = 0.0;
        if (i < n / THERMO_WORDS) B.tpend[i] = 0;
    }
}

// Export the list of one replica as tag pairs (inspection and tests).
__global__ void k_export_nlist(Buffers B, Launch P, int rep, int32_t *__restrict__ pairs,
                               int64_t cap, unsigned long long *__restrict__ count)
{
    __shared__ StageHdr S;
    const RepDev &R = B.reps[rep];
    int lb = blockIdx.x;
    if (lb >= R.nbrick) return;
    int b = R.b_off + lb;
    if (threadIdx.x == 0) pass_header(R, B, b, lb, P.stage_cap, S);
    __syncthreads();
    if (S.overflow) return;
    const int32_t *sm = B.smap + (size_t)b * P.stage_cap;
    for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
        int64_t i = S.base + t;
        for_each_neighbour(B.nl, P.nslots, i, B.nn[i], [&](int u) {
            if (R.excl_span > 0) u &= 0x7fff;
            if (u == S.total) return;  // padding
            unsigned long long k = atomicAdd(count, 1ull);
            if ((int64_t)k < cap) {
                pairs[2 * k] = B.tag[i];
                pairs[2 * k + 1] = B.tag[sm[u]];
            }
        });
    }
}

__global__ void k_zero_u64(unsigned long long *p) { *p = 0ull; }

__global__ void k_zero_i64(int64_t *p, int n)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) p[k] = 0;
}

// Squared minimum-image distance from the wrapped position wi of a particle to slot j, in
// FP64 with the operations of the plain definition (round-half-even image, no contraction):
// the bond criterion of the observables and of the cluster analysis.
// Both positions lie in [0, L), so |t| < L and the image index rint(t / L) is -1, 0 or 1;
// away from |t| = L / 2 the comparison t > L / 2 decides it exactly (the quotient is then
// far from 1/2), and only that band takes the division.
__device__ __forceinline__ double obs_r2(const RepDev &R, const double *__restrict__ X, int64_t S_,
                                         const double wi[3], int64_t j)
{
#pragma clang fp contract(off)
    double d[3];
    for (int a = 0; a < 3; ++a) {
        const double La = R.L[a];
        const double tt = wi[a] - wrap1(X[3 * j + a], La);
        const double at = fabs(tt);
        double k;
        if (at < 0.375 * La) k = 0.0;
        else if (at > 0.625 * La) k = tt > 0.0 ? 1.0 : -1.0;
        else k = rint(tt / La);
        d[a] = tt - La * k;
    }
    return (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
}

// Brick-local FP32 positions of every particle the brick staged at the last list build, and
// the dummy slot far away, in LDS as (x, y) | z | type, the types only with several of them:
// 12 bytes per particle with one type, which lets a third workgroup of a layout sized for
// condensation share the CU (the bond sweep of 500,000 particles: 102.6 -> 69.4 us together with
// reading a bond's slot only where it is needed).
struct Staged {
    float2 *xy;
    float *z;
    int32_t *type;  // several types only
};

__device__ __forceinline__ Staged carve_staged(unsigned char *smem, int stage_cap)
{
    Staged T;
    T.xy = (float2 *)smem;
    T.z = (float *)(T.xy + stage_cap + 1);
    T.type = (int32_t *)(T.z + stage_cap + 1);
    return T;
}

// All threads call this.
template <bool MULTI>
__device__ __forceinline__ void stage_bonds(const Buffers &B, const Launch &P, const RepDev &R,
                                            const StageHdr &S, int b, const double *X, const Staged &T,
                                            const MapFirst &first)
{
    stage_map4(B, b, P.stage_cap, S, first, [&](int t, int src, int w, bool ok) {
        const float4 p = local_pos<float>(R, S, X, P.nslots, src, w, 0);
        const int ty = MULTI ? B.type[src] : 0;
        if (ok) {
            T.xy[t] = make_float2(p.x, p.y);
            T.z[t] = p.z;
            if (MULTI) T.type[t] = ty;
        }
    });
    if (threadIdx.x == 0) {
        T.xy[S.total] = make_float2(1.0e6f, 1.0e6f);
        T.z[S.total] = 1.0e6f;
        if (MULTI) T.type[S.total] = 0;
    }
}

// Squared distance of staged particle u from (a, az).
__device__ __forceinline__ float staged_r2(const Staged &T, const float2 &a, float az, int u)
{
    const float2 q = T.xy[u];
    const float dx = a.x - q.x, dy = a.y - q.y, dz = az - T.z[u];
    return dx * dx + dy * dy + dz * dz;
}

// Threshold r^2 < c2 decided on the staged FP32 distance outside a band around c2 that is
// wider than the staging's rounding (its error in r^2 stays below 2e-5 for brick-local
// coordinates), and inside the band by the FP64 expression of the plain definition.
struct Band {
    float lo, hi;
    double c2;
};

__device__ __forceinline__ Band make_band(double c2)
{
    return Band{(float)(c2 * (1.0 - 2e-5) - 1e-4), (float)(c2 * (1.0 + 2e-5) + 1e-4), c2};
}

// r2f below the band is inside, above it outside; slot() (the neighbour's slot, read only in
// the band) decides the rest.
template <class F>
__device__ __forceinline__ bool within(float r2f, const Band &bd, const RepDev &R, const double *X,
                                       int64_t S_, int64_t i, F &&slot)
{
    if (r2f < bd.lo) return true;
    if (!(r2f < bd.hi)) return false;
    double wi[3];
    for (int a = 0; a < 3; ++a) wi[a] = wrap1(X[3 * i + a], R.L[a]);
    return obs_r2(R, X, S_, wi, slot()) < bd.c2;
}

// Observables of valency control: for every own particle the number of list neighbours
// within the attraction range and within the repulsive core of the pair, each threshold
// decided by `within` (exactly as the plain FP64 definition on the wrapped positions), plus
// per-replica sums {sum z, #(z > f), sum p}.  The list holds every pair within the
// interaction cutoff.
template <bool MULTI, bool LARGE>
__device__ __forceinline__ void observe_brick(const Buffers &B, const Launch &P, int cur, int32_t *__restrict__ z_out,
                                              int32_t *__restrict__ pen_out, int64_t *__restrict__ sums, int b)
{
    extern __shared__ __align__(16) unsigned char smem[];  // Staged
    __shared__ unsigned long long tot[3];
    const MapFirst mf = map_prefetch(B, b, P.stage_cap);
    const int r = B.brick_rep[b];
    if (r < 0) return;
    const RepDev &R = B.reps[r];
    const int lb = b - R.b_off;
    if (threadIdx.x == 0) tot[0] = tot[1] = tot[2] = 0ull;
    StageHdr S;
    pass_header(R, B, b, lb, P.stage_cap, S);
    if (S.overflow || (!LARGE && S.total > P.t_hi)) return;
    const int64_t S_ = P.nslots;
    const double *X = B.x[cur];
    const int32_t *sm = B.smap + (size_t)b * P.stage_cap;
    const Staged T = carve_staged(smem, P.lds_cap);
    stage_bonds<MULTI>(B, P, R, S, b, X, T, mf);
    __syncthreads();
    const bool xr = R.excl_span > 0;
    const Band ba0 = make_band(R.pair[0].ra2), br0 = make_band(R.pair[0].rr2);
    unsigned long long zs = 0, over = 0, ps = 0;
    for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
        const int64_t i = S.base + t;
        const float2 pi = T.xy[t];
        const float zi = T.z[t];
        const int ti = MULTI ? T.type[t] : 0;
        int z = 0, p = 0;
        for_each_neighbour(B.nl, S_, i, B.nn[i], [&](int u) {
            if (MULTI && xr) u &= 0x7fff;
            const float r2f = staged_r2(T, pi, zi, u);
            Band ba = ba0, br = br0;
            if (MULTI) {
                const PairDev &pd = R.pair[ti * MAXT + T.type[u]];
                ba = make_band(pd.ra2);
                br = make_band(pd.rr2);
            }
            if (!(r2f < ba.hi) && !(r2f < br.hi)) return;  // beyond both (and the padding)
            z += within(r2f, ba, R, X, S_, i, [&] { return (int64_t)sm[u]; }) ? 1 : 0;
            p += within(r2f, br, R, X, S_, i, [&] { return (int64_t)sm[u]; }) ? 1 : 0;
        });
        const int32_t tg = B.tag[i];
        if (z_out) z_out[R.o_off + tg] = z;
        if (pen_out) pen_out[R.o_off + tg] = p;
        zs += (unsigned long long)z;
        ps += (unsigned long long)p;
        over += ((double)z > R.pair[ti * MAXT + ti].f) ? 1ull : 0ull;
    }
    zs = wave_sum(zs);
    over = wave_sum(over);
    ps = wave_sum(ps);
    if ((threadIdx.x % VBC_WAVE) == 0) {
        atomicAdd(&tot[0], zs);
        atomicAdd(&tot[1], over);
        atomicAdd(&tot[2], ps);
    }
    __syncthreads();
    if (sums && threadIdx.x < 3 && tot[threadIdx.x])
        atomicAdd((unsigned long long *)&sums[3 * r + threadIdx.x], tot[threadIdx.x]);
}

template <bool MULTI>
__global__ void k_observe(Buffers B, Launch P, int cur, int32_t *__restrict__ z_out,
                          int32_t *__restrict__ pen_out, int64_t *__restrict__ sums)
{
    int b;
    if (brick_of_block(P, B, b)) observe_brick<MULTI, false>(B, P, cur, z_out, pen_out, sums, b);
}

template <bool MULTI>
__global__ void __launch_bounds__(DENSE_BLOCK) k_observe_dense(Buffers B, Launch P, int cur, int32_t *__restrict__ z_out,
                                                               int32_t *__restrict__ pen_out, int64_t *__restrict__ sums)
{
    each_dense(P, B, [&](int b) { observe_brick<MULTI, true>(B, P, cur, z_out, pen_out, sums, b); });
}

// ---------------------------------------------------------------------------
// clusters of the bond graph (Section 3): union-find over the slots
// ---------------------------------------------------------------------------
//
// parent[] forms a forest over the slots in which every pointer goes to a smaller slot:
// hooking links a root under a smaller root, and path halving only ever replaces a parent
// by one of its ancestors.  Every walk therefore ends, whatever other lanes do meanwhile,
// and the root of a cluster is its smallest slot.

__device__ __forceinline__ int32_t cc_ld(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void cc_st(int32_t *p, int32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t cc_find(int32_t *parent, int32_t x)
{
    while (true) {
        const int32_t p = cc_ld(parent + x);
        if (p == x) return x;
        const int32_t g = cc_ld(parent + p);
        if (g == p) return p;
        cc_st(parent + x, g);  // path halving
        x = g;
    }
}

__device__ __forceinline__ void cc_union(int32_t *parent, int32_t a, int32_t b)
{
    a = cc_find(parent, a);
    b = cc_find(parent, b);
    while (a != b) {
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t old = atomicCAS(parent + a, a, b);
        if (old == a) return;
        a = cc_find(parent, old);
        b = cc_find(parent, b);
    }
}

// LDS union-find over the own particles of one brick (their staged index is their index in
// the brick), with the same smaller-root rule.
__device__ __forceinline__ int32_t lcc_find(int32_t *lp, int32_t x)
{
    while (true) {
        const int32_t p = __hip_atomic_load(lp + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (p == x) return x;
        const int32_t g = __hip_atomic_load(lp + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (g == p) return p;
        __hip_atomic_store(lp + x, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        x = g;
    }
}

__device__ __forceinline__ void lcc_union(int32_t *lp, int32_t a, int32_t b)
{
    a = lcc_find(lp, a);
    b = lcc_find(lp, b);
    while (a != b) {
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t old = atomicCAS(lp + a, a, b);
        if (old == a) return;
        a = lcc_find(lp, old);
        b = lcc_find(lp, b);
    }
}

// Bonds that leave a brick, as (own slot, slot in the neighbouring brick) with the smaller
// slot first, recorded by the sweep of the bonds in the brick's share of a space that is free
// between list builds (xref, or xs of a replica that is stepped in one workgroup and keeps its
// reference positions in xref): up to three per slot.
__device__ __forceinline__ int2 *cross_bonds(const Buffers &B, const RepDev &R, int64_t base)
{
    return (int2 *)((R.resident ? B.xs : B.xref) + 3 * base);
}
__device__ __forceinline__ int cross_cap(const RepDev &R) { return 3 * R.bcap; }

// Bonds of every own particle (the z_i criterion of the observables) from its list.  Bonds
// between two own particles of the brick are joined in LDS first; the forest then starts from
// the brick's local components, each a star under its smallest slot, with the component's
// size, bond ends and smallest tag summed in LDS at that slot (size 0 marks the others).
// Bonds that leave the brick are recorded for the next kernel, so that the lists are swept
// once, not twice.  Also clears the statistics that the labelling adds to.
template <bool MULTI, bool LARGE>
__device__ __forceinline__ void cc_local_brick(const Buffers &B, const Launch &P, int cur, const ClusterWork &W, int b)
{
    extern __shared__ __align__(16) unsigned char smem[];  // Staged, then lp[bcap]
    __shared__ int ncross;
    const MapFirst mf = map_prefetch(B, b, P.stage_cap);
    const int r = B.brick_rep[b];
    if (r < 0) return;
    const RepDev &R = B.reps[r];
    const int lb = b - R.b_off;
    if (threadIdx.x == 0) ncross = 0;
    StageHdr S;
    pass_header(R, B, b, lb, P.stage_cap, S);
    if (!LARGE && S.total > P.t_hi) return;
    if (S.overflow) {
        // no lists: its particles stay single, uncounted, and may be joined from outside
        for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
            const int64_t i = S.base + t;
            W.parent[i] = (int32_t)i;
            W.size[i] = 0;
            W.ends[i] = 0u;
            W.mintag[i] = INT32_MAX;
        }
        return;
    }
    const int64_t S_ = P.nslots;
    const double *X = B.x[cur];
    const int32_t *sm = B.smap + (size_t)b * P.stage_cap;
    const Staged T = carve_staged(smem, P.lds_cap);
    int32_t *lp = T.type + (MULTI ? P.lds_cap + 1 : 0);
    stage_bonds<MULTI>(B, P, R, S, b, X, T, mf);
    for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) lp[t] = t;
    __syncthreads();
    const bool xr = R.excl_span > 0;
    const Band ba0 = make_band(R.pair[0].ra2);
    int2 *cross = cross_bonds(B, R, S.base);
    const int cap = cross_cap(R);
    for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
        const int64_t i = S.base + t;
        const float2 pi = T.xy[t];
        const float zi = T.z[t];
        const int ti = MULTI ? T.type[t] : 0;
        int z = 0;
        for_each_neighbour(B.nl, S_, i, B.nn[i], [&](int u) {
            if (MULTI && xr) u &= 0x7fff;
            const float r2f = staged_r2(T, pi, zi, u);
            const Band ba = MULTI ? make_band(R.pair[ti * MAXT + T.type[u]].ra2) : ba0;
            if (!(r2f < ba.hi)) return;  // also the padding
            if (!within(r2f, ba, R, X, S_, i, [&] { return (int64_t)sm[u]; })) return;
            ++z;
            if (u < S.n_own) {
                if (u > t) lcc_union(lp, t, u);
            } else {
                const int j = sm[u];
                if (j > (int)i) {
                    const int k = atomicAdd(&ncross, 1);
                    if (k < cap) cross[k] = make_int2((int)i, j);
                }
            }
        });
        W.z[i] = z;
    }
    __syncthreads();
    // the staged positions are no longer needed: their space takes the components' sums
    int32_t *csize = (int32_t *)smem, *cends = csize + S.n_own, *cmin = cends + S.n_own;
    for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
        csize[t] = cends[t] = 0;
        cmin[t] = INT32_MAX;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
        const int64_t i = S.base + t;
        const int root = lcc_find(lp, t);
        W.parent[i] = (int32_t)(S.base + root);
        atomicAdd(csize + root, 1);
        const int z = W.z[i];  // written by this thread
        if (z) atomicAdd(cends + root, z);
        atomicMin(cmin + root, B.tag[i]);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
        const int64_t i = S.base + t;
        W.size[i] = csize[t];
        W.ends[i] = (uint32_t)cends[t];
        W.mintag[i] = cmin[t];
    }
    if (threadIdx.x == 0) W.z[S.base] = ncross;  // bond counts are summed: their first word counts these
}

template <bool MULTI>
__global__ void k_cc_local(Buffers B, Launch P, int cur, ClusterWork W, int64_t *__restrict__ stats,
                           int64_t *__restrict__ hist, int64_t nhist)
{
    const int64_t g0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, gn = (int64_t)gridDim.x * blockDim.x;
    if (stats)
        for (int64_t k = g0; k < 5 * (int64_t)P.nrep; k += gn) stats[k] = 0;
    if (hist)
        for (int64_t k = g0; k < nhist; k += gn) hist[k] = 0;
    int b;
    if (brick_of_block(P, B, b)) cc_local_brick<MULTI, false>(B, P, cur, W, b);
}

template <bool MULTI>
__global__ void __launch_bounds__(DENSE_BLOCK) k_cc_local_dense(Buffers B, Launch P, int cur, ClusterWork W)
{
    each_dense(P, B, [&](int b) { cc_local_brick<MULTI, true>(B, P, cur, W, b); });
}

// Bonds that leave the brick join the global forest.  A bond is taken between the current
// parents of its ends (ancestors, so in the same clusters), and a workgroup joins each
// distinct pair of them once: a condensed brick has hundreds of bonds into a few dozen
// neighbouring components.  The set of pairs lives in LDS with open addressing; when it is
// full the join simply runs.  A brick with more such bonds than were recorded finds them
// again from its lists, by the plain FP64 definition.
constexpr int CC_SET = 512;

__global__ void k_cc_hook(Buffers B, Launch P, int cur, ClusterWork W)
{
    __shared__ unsigned long long set[CC_SET];
    int b, r;
    if (!resolve_brick(P, B, b, r)) return;
    const RepDev &R = B.reps[r];
    const int lb = b - R.b_off, n_own = B.bcnt[0][b];
    const int total = B.stotal[b];
    if (n_own == 0 || total > P.stage_cap) return;
    const int64_t base = R.p_off + (int64_t)lb * R.bcap;
    const int nc = W.z[base];
    for (int k = threadIdx.x; k < CC_SET; k += blockDim.x) set[k] = ~0ull;
    __syncthreads();
    auto join = [&](int i, int j) {
        int32_t pa = cc_ld(W.parent + i), pb = cc_ld(W.parent + j);
        if (pa == pb) return;
        if (pa > pb) {
            const int32_t tmp = pa;
            pa = pb;
            pb = tmp;
        }
        const unsigned long long key = ((unsigned long long)(uint32_t)pa << 32) | (uint32_t)pb;
        unsigned h = (unsigned)((key * 0x9E3779B97F4A7C15ull) >> 55) & (CC_SET - 1);
        for (int probe = 0; probe < 16; ++probe) {
            const unsigned long long prev = atomicCAS(set + h, ~0ull, key);
            if (prev == key) return;  // this pair is joined already
            if (prev == ~0ull) break;  // first of its pair
            h = (h + 1) & (CC_SET - 1);
        }
        cc_union(W.parent, pa, pb);
    };
    if (nc <= cross_cap(R)) {
        const int2 *cross = cross_bonds(B, R, base);
        for (int k = threadIdx.x; k < nc; k += blockDim.x) join(cross[k].x, cross[k].y);
        return;
    }
    const double *X = B.x[cur];
    const int32_t *sm = B.smap + (size_t)b * P.stage_cap;
    for (int t = threadIdx.x; t < n_own; t += blockDim.x) {
        const int64_t i = base + t;
        const int ti = B.type[i];
        double wi[3];
        for (int a = 0; a < 3; ++a) wi[a] = wrap1(X[3 * i + a], R.L[a]);
        for_each_neighbour(B.nl, P.nslots, i, B.nn[i], [&](int u) {
            if (R.excl_span > 0) u &= 0x7fff;
            if (u < n_own || u == total) return;  // inside the brick, or padding
            const int j = sm[u];
            if (j < (int)i || !(obs_r2(R, X, P.nslots, wi, j) < R.pair[ti * MAXT + B.type[j]].ra2)) return;
            join((int)i, j);
        });
    }
}

// Size, bond ends and smallest tag of every cluster, gathered at its root from the bricks'
// local components; each component's root keeps the cluster's root as parent for the
// labelling pass.  A workgroup first sums its components by cluster in an LDS table: the
// root of a percolating cluster then takes a few atomics per workgroup, and a small cluster
// one per brick it touches (one per particle: 247 us at 500,000 particles).
constexpr int CC_TAB = 256;

__global__ void k_cc_count(Buffers B, Launch P, ClusterWork W)
{
    __shared__ int32_t troot[CC_TAB], tsize[CC_TAB], tmin[CC_TAB];
    __shared__ uint32_t tends[CC_TAB];
    int b, r;
    if (!resolve_brick(P, B, b, r)) return;
    const RepDev &R = B.reps[r];
    const int n_own = B.bcnt[0][b];
    if (n_own == 0 || B.stotal[b] > P.stage_cap) return;
    const int64_t base = R.p_off + (int64_t)(b - R.b_off) * R.bcap;
    for (int k = threadIdx.x; k < CC_TAB; k += blockDim.x) {
        troot[k] = -1;
        tsize[k] = 0;
        tends[k] = 0u;
        tmin[k] = INT32_MAX;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < n_own; t += blockDim.x) {
        const int64_t i = base + t;
        const int32_t sz = W.size[i];
        if (sz == 0) continue;  // not a component's root
        // no path halving here: another thread's halving of slot i, from what it read before
        // the line below, could put an ancestor short of the root back
        int32_t root = (int32_t)i;
        for (int32_t p = cc_ld(W.parent + root); p != root; p = cc_ld(W.parent + root)) root = p;
        if (root == (int32_t)i) continue;
        cc_st(W.parent + i, root);
        const uint32_t en = W.ends[i];
        const int32_t mt = W.mintag[i];
        int h = (int)(((uint32_t)root * 0x9E3779B1u) >> 24) & (CC_TAB - 1);
        int at = -1;
        for (int probe = 0; probe < 8; ++probe) {
            const int32_t prev = atomicCAS(troot + h, -1, root);
            if (prev == -1 || prev == root) {
                at = h;
                break;
            }
            h = (h + 1) & (CC_TAB - 1);
        }
        if (at >= 0) {
            atomicAdd(tsize + at, sz);
            if (en) atomicAdd(tends + at, en);
            atomicMin(tmin + at, mt);
        } else {
            atomicAdd(W.size + root, sz);
            if (en) atomicAdd(W.ends + root, en);
            atomicMin(W.mintag + root, mt);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < CC_TAB; k += blockDim.x) {
        const int32_t root = troot[k];
        if (root < 0) continue;
        atomicAdd(W.size + root, tsize[k]);
        if (tends[k]) atomicAdd(W.ends + root, tends[k]);
        atomicMin(W.mintag + root, tmin[k]);
    }
}

// Per particle: its cluster's smallest tag.  Per root: the cluster's statistics and its
// histogram bins (all clusters, acyclic clusters), the latter summed in LDS first where they
// fit.  A workgroup takes a run of consecutive bricks and adds its sums to the replica's when
// the replica changes and at the end: all workgroups add to the same few words, and with a
// workgroup per brick and an atomic per cluster the pass took 88 us at 500,000 particles.
constexpr int CC_HIST = 2048;    // sizes a workgroup sums in LDS
constexpr int CC_GROUPS = 512;   // workgroups

__global__ void k_cc_label(Buffers B, Launch P, ClusterWork W, int32_t *__restrict__ label,
                           int64_t *__restrict__ stats, int64_t *__restrict__ hist, int hist_len)
{
    extern __shared__ uint32_t lh[];  // [2][hist_len] where hist_len <= CC_HIST
    __shared__ unsigned long long tot[5];
    const int T = P.list < 0 ? P.nb_launch : B.wl_n[P.list];
    const int per = (T + gridDim.x - 1) / gridDim.x;
    const int k0 = blockIdx.x * per, k1 = min(k0 + per, T);
    const bool inlds = hist && hist_len <= CC_HIST;
    if (threadIdx.x < 5) tot[threadIdx.x] = 0ull;
    if (inlds)
        for (int k = threadIdx.x; k < 2 * hist_len; k += blockDim.x) lh[k] = 0u;
    __syncthreads();
    unsigned long long nc = 0, cp = 0, bonds = 0, ncyc = 0, lg = 0;
    int rc = -1;  // the replica whose sums are open
    auto flush = [&](int r) {
        const unsigned long long v0 = wave_sum(nc), v2 = wave_sum(cp), v3 = wave_sum(bonds), v4 = wave_sum(ncyc);
        for (int o = VBC_WAVE / 2; o > 0; o >>= 1) {
            const unsigned long long v = __shfl_down(lg, o, VBC_WAVE);
            lg = v > lg ? v : lg;
        }
        if ((threadIdx.x % VBC_WAVE) == 0 && v0) {
            atomicAdd(&tot[0], v0);
            atomicMax(&tot[1], lg);
            atomicAdd(&tot[2], v2);
            atomicAdd(&tot[3], v3);
            atomicAdd(&tot[4], v4);
        }
        __syncthreads();
        if (inlds)
            for (int k = threadIdx.x; k < 2 * hist_len; k += blockDim.x)
                if (lh[k]) {
                    atomicAdd((unsigned long long *)(hist + (size_t)r * 2 * hist_len + k), (unsigned long long)lh[k]);
                    lh[k] = 0u;
                }
        if (threadIdx.x < 5) {
            unsigned long long *st = (unsigned long long *)(stats + 5 * (size_t)r) + threadIdx.x;
            const unsigned long long v = tot[threadIdx.x];
            if (stats && v) {
                if (threadIdx.x == 1) atomicMax(st, v);
                else atomicAdd(st, v);
            }
            tot[threadIdx.x] = 0ull;
        }
        __syncthreads();
        nc = cp = bonds = ncyc = lg = 0;
    };
    for (int k = k0; k < k1; ++k) {
        const int b = P.list < 0 ? P.b_lo + k : B.wl[P.list][k];
        const int r = B.brick_rep[b], n_own = B.bcnt[0][b];
        if (r < 0 || n_own == 0 || B.stotal[b] > P.stage_cap) continue;
        if (r != rc) {
            if (rc >= 0) flush(rc);
            rc = r;
        }
        const RepDev &R = B.reps[r];
        const int64_t base = R.p_off + (int64_t)(b - R.b_off) * R.bcap;
        int64_t *h = hist + (size_t)r * 2 * hist_len;
        for (int t = threadIdx.x; t < n_own; t += blockDim.x) {
            const int64_t i = base + t;
            // the particle's component root, whose parent is the cluster's root
            const int32_t root = W.parent[W.parent[i]];
            if (label) label[R.o_off + B.tag[i]] = W.mintag[root];
            if (root != (int32_t)i) continue;
            const unsigned long long sz = (unsigned long long)W.size[i];
            const unsigned long long e = (unsigned long long)(W.ends[i] / 2u);
            const bool cyc = e >= sz;
            nc += 1ull;
            bonds += e;
            if (cyc) {
                cp += sz;
                ncyc += 1ull;
            }
            lg = sz > lg ? sz : lg;
            if (hist) {
                const int bin = sz < (unsigned long long)hist_len ? (int)sz : 0;
                if (inlds) {
                    atomicAdd(lh + bin, 1u);
                    if (!cyc) atomicAdd(lh + hist_len + bin, 1u);
                } else {
                    atomicAdd((unsigned long long *)(h + bin), 1ull);
                    if (!cyc) atomicAdd((unsigned long long *)(h + hist_len + bin), 1ull);
                }
            }
        }
    }
    if (rc >= 0) flush(rc);
}

// ---------------------------------------------------------------------------
// bond lifetimes (Section 4): partners of every particle carried from sample to sample
// ---------------------------------------------------------------------------

// One sample of the bond tracker.  For every own particle the state (by caller index) holds
// up to M partner tags with the step each bond was first seen (-1: present when tracking
// began).  A stored partner that is no longer bonded is a broken bond: its lifetime goes to
// the replica's histogram (bin = lifetime / bin_steps, the last bin holds the longer ones),
// or to the censored count without a birth.  A bonded particle not stored is a new bond,
// born now.  Each event is counted at the end with the smaller tag, once per bond.
// stats per replica: {formed, broken with a lifetime, broken without one, partners that did
// not fit, bonds now}.
template <bool MULTI, bool LARGE>
__device__ __forceinline__ void bond_track_brick(const Buffers &B, const Launch &P, int cur, const BondTrack &T, int reset,
                                                 int64_t *__restrict__ hist, int hist_len, int64_t bin_steps,
                                                 int64_t *__restrict__ stats, int b)
{
    extern __shared__ __align__(16) unsigned char smem[];  // Staged
    __shared__ unsigned long long tot[5];
    const MapFirst mf = map_prefetch(B, b, P.stage_cap);
    const int r = B.brick_rep[b];
    if (r < 0) return;
    const RepDev &R = B.reps[r];
    const int lb = b - R.b_off;
    if (threadIdx.x < 5) tot[threadIdx.x] = 0ull;
    StageHdr S;
    pass_header(R, B, b, lb, P.stage_cap, S);
    if (S.overflow || (!LARGE && S.total > P.t_hi)) return;
    const int64_t S_ = P.nslots;
    const double *X = B.x[cur];
    const int32_t *sm = B.smap + (size_t)b * P.stage_cap;
    const Staged G = carve_staged(smem, P.lds_cap);
    stage_bonds<MULTI>(B, P, R, S, b, X, G, mf);
    __syncthreads();
    const bool xr = MULTI && R.excl_span > 0;
    const Band ba0 = make_band(R.pair[0].ra2);
    const int M = T.M;
    const int64_t now = (int64_t)B.step[r];
    unsigned long long formed = 0, broken = 0, cens = 0, over = 0, bonds = 0;
    for (int t = threadIdx.x; t < S.n_own; t += blockDim.x) {
        const int64_t i = S.base + t;
        const float2 pi = G.xy[t];
        const float zi = G.z[t];
        const int ti = MULTI ? G.type[t] : 0;
        const int32_t tg = B.tag[i];
        const int64_t c = R.o_off + tg;
        int32_t *ptag = T.tags + c * M;
        int64_t *pbirth = T.births + c * M;
        auto bonded = [&](int u) {
            const float r2f = staged_r2(G, pi, zi, u);
            const Band ba = MULTI ? make_band(R.pair[ti * MAXT + G.type[u]].ra2) : ba0;
            return r2f < ba.hi && within(r2f, ba, R, X, S_, i, [&] { return (int64_t)sm[u]; });
        };
        int n = 0;
        if (!reset) {
            // 1. which stored partners are still bonded
            const int n_old = min(max(T.count[c], 0), M);
            uint64_t keep = 0ull;
            for_each_neighbour(B.nl, S_, i, B.nn[i], [&](int u) {
                if (xr) u &= 0x7fff;
                if (!bonded(u)) return;
                const int32_t tj = B.tag[sm[u]];
                for (int k = 0; k < n_old; ++k)
                    if (ptag[k] == tj) {
                        keep |= 1ull << k;
                        break;
                    }
            });
            // 2. broken bonds leave, the others close up in order
            for (int k = 0; k < n_old; ++k) {
                const int32_t tk = ptag[k];
                const int64_t bk = pbirth[k];
                if ((keep >> k) & 1ull) {
                    ptag[n] = tk;
                    pbirth[n] = bk;
                    ++n;
                } else if (tg < tk) {
                    if (bk >= 0) {
                        ++broken;
                        if (hist) {
                            const int64_t bin = (now - bk) / bin_steps;
                            atomicAdd((unsigned long long *)(hist + (size_t)r * hist_len +
                                                             (bin < hist_len - 1 ? bin : hist_len - 1)),
                                      1ull);
                        }
                    } else {
                        ++cens;
                    }
                }
            }
        }
        // 3. bonds not stored are new (at a reset: present from the start, birth unknown)
        const int n_keep = n;
        for_each_neighbour(B.nl, S_, i, B.nn[i], [&](int u) {
            if (xr) u &= 0x7fff;
            if (!bonded(u)) return;
            const int32_t tj = B.tag[sm[u]];
            if (tg < tj) ++bonds;
            for (int k = 0; k < n_keep; ++k)
                if (ptag[k] == tj) return;
            if (n < M) {
                ptag[n] = tj;
                pbirth[n] = reset ? (int64_t)-1 : now;
                ++n;
                if (!reset && tg < tj) ++formed;
            } else {
                ++over;
            }
        });
        T.count[c] = n;
    }
    formed = wave_sum(formed);
    broken = wave_sum(broken);
    cens = wave_sum(cens);
    over = wave_sum(over);
    bonds = wave_sum(bonds);
    if ((threadIdx.x % VBC_WAVE) == 0) {
        atomicAdd(&tot[0], formed);
        atomicAdd(&tot[1], broken);
        atomicAdd(&tot[2], cens);
        atomicAdd(&tot[3], over);
        atomicAdd(&tot[4], bonds);
    }
    __syncthreads();
    if (stats && threadIdx.x < 5 && tot[threadIdx.x])
        atomicAdd((unsigned long long *)(stats + 5 * (size_t)r + threadIdx.x), tot[threadIdx.x]);
}

template <bool MULTI>
__global__ void k_bond_track(Buffers B, Launch P, int cur, BondTrack T, int reset,
                             int64_t *__restrict__ hist, int hist_len, int64_t bin_steps,
                             int64_t *__restrict__ stats)
{
    int b;
    if (brick_of_block(P, B, b)) bond_track_brick<MULTI, false>(B, P, cur, T, reset, hist, hist_len, bin_steps, stats, b);
}

template <bool MULTI>
__global__ void __launch_bounds__(DENSE_BLOCK) k_bond_track_dense(Buffers B, Launch P, int cur, BondTrack T, int reset,
                                                                  int64_t *__restrict__ hist, int hist_len,
                                                                  int64_t bin_steps, int64_t *__restrict__ stats)
{
    each_dense(P, B, [&](int b) {
        bond_track_brick<MULTI, true>(B, P, cur, T, reset, hist, hist_len, bin_steps, stats, b);
    });
}

// ---------------------------------------------------------------------------
// resident steps of small replicas
// ---------------------------------------------------------------------------

// A set of small replicas takes a step of brick kernels at the pace of its many small bricks:
// 32 replicas of 1000 particles laid out for condensation are 6912 bricks of five particles,
// whose reserved LDS leaves two workgroups of two waves on a CU (190 us a step), and some
// replica's list is due in nearly every step.  The steps of such a set run with one workgroup
// per replica instead: its positions and switching factors stay in LDS, a barrier takes the
// place of a launch, and one launch does many steps for all replicas (that set: 20 us a step
// from a uniform start, 65 once some replicas have collapsed into droplets with lists of a
// hundred neighbours; then one CU's VALU issue on the densest replica is the bound).
//
// Between calls the particles stand in caller order (slot p_off + tag, positions wrapped
// every step) with their forces (Fst), velocities, the positions of the last list build
// (xref) and the list (nl, nn: tags in 16 bits, eight per chunk).  An analysis or a force
// evaluation in between takes the replica into the brick layout, which leaves xref alone; the
// next step then builds the same list again from xref and the same forces, so that the
// trajectory does not depend on it.  The list orders neighbours by cell of a grid of at least
// the list radius and by tag inside a cell, so it depends on xref alone, and every sum here is
// per particle in list order or over 64 consecutive tags: neither the workgroup's size nor
// the other replicas change a bit.
//
// FP32 pair arithmetic: positions are 64-bit fractions of the box, and a distance starts from
// the wrapped integer difference of their upper halves: the minimum image without a test, and
// an error of L 2^-32 where a staged FP32 coordinate has up to 5e-7.  The FP64 recount of
// particles near a switching window takes the whole 64 bits, and so does dU/dn, whose
// distances are rounded once (a box of 500: rms force error of window particles 3.6e-7 with
// upper halves, 3.3e-7 so, 7.9e-7 by bricks; same time).  The list takes every pair below the list radius: its FP32 test
// allows a millionth more than that, so that it may hold a pair that the bricks' lists do not,
// beyond every cutoff.
//
// A thread owns the particle of its index: position, velocity, force and reference position
// stay in registers through a call, and only the list is read from memory.
constexpr double RES_MAX_L = 512.0;

template <class Real> struct ResLds;

template <> struct ResLds<float> {
    int2 *xy, *zs;       // upper halves of the fractions; s beside z
    float *A;            // c_c dU/dn
    uint32_t *lo[3];     // lower halves
    int4 *sorted;        // list build: (x, y, z, tag) by cell, then by tag
    int *cell;           // [n + 2] list build: end of each cell
    uint16_t *order;     // [n] list build: members; then the window particles
    static size_t bytes(int n) { return (size_t)n * (32 + 16 + 4 + 2) + 64; }
    __device__ void carve(unsigned char *p, int n)
    {
        sorted = (int4 *)p;
        xy = (int2 *)(sorted + n);
        zs = xy + n;
        A = (float *)(zs + n);
        for (int a = 0; a < 3; ++a) lo[a] = (uint32_t *)(A + (a + 1) * n);
        cell = (int *)(lo[2] + n);
        order = (uint16_t *)(cell + n + 2);
    }
    struct Pos { int x, y, z; };
    struct Scale { float h[3]; };  // L 2^-32
    static __device__ Scale scale(const double L[3])
    {
        return Scale{{(float)(L[0] * 0x1p-32), (float)(L[1] * 0x1p-32), (float)(L[2] * 0x1p-32)}};
    }
    __device__ void put(int k, const double x[3], const double iL[3])
    {
        uint32_t hi[3];
        for (int a = 0; a < 3; ++a) {
            double f = x[a] * iL[a];
            f = f < 1.0 ? f * 0x1p32 : 0.0;  // x < L, but the product may round up to 1
            const double fl = floor(f);
            hi[a] = (uint32_t)fl;
            lo[a][k] = (uint32_t)((f - fl) * 0x1p32);
        }
        xy[k] = make_int2((int)hi[0], (int)hi[1]);
        zs[k].x = (int)hi[2];
    }
    __device__ Pos own(int k) const { return Pos{xy[k].x, xy[k].y, zs[k].x}; }
    __device__ void sort_in(int q, int k) { sorted[q] = make_int4(xy[k].x, xy[k].y, zs[k].x, k); }
    static __device__ int cell_axis(const Pos &p, int a, int g, const double[3])
    {
        return (int)__umulhi((uint32_t)(a == 0 ? p.x : a == 1 ? p.y : p.z), (uint32_t)g);
    }
    static __device__ void sub(const Pos &p, int x, int y, int z, const Scale &H, float d[3])
    {
        d[0] = (float)(int)((uint32_t)p.x - (uint32_t)x) * H.h[0];
        d[1] = (float)(int)((uint32_t)p.y - (uint32_t)y) * H.h[1];
        d[2] = (float)(int)((uint32_t)p.z - (uint32_t)z) * H.h[2];
    }
    // d = x_i - x_j, minimum image
    __device__ void diff(const Pos &p, int j, const Scale &H, float d[3]) const
    {
        const int2 q = xy[j];
        sub(p, q.x, q.y, zs[j].x, H, d);
    }
    __device__ void diff_s(const Pos &p, int j, const Scale &H, float d[3], float &s) const
    {
        const int2 q = xy[j], r = zs[j];
        sub(p, q.x, q.y, r.x, H, d);
        s = __int_as_float(r.y);
    }
    __device__ int diff_sorted(const Pos &p, int q, const Scale &H, float d[3]) const
    {
        const int4 v = sorted[q];
        sub(p, v.x, v.y, v.z, H, d);
        return v.w;
    }
    // d = x_i - x_j in FP64 from the whole fractions, minimum image
    __device__ void diff64(int i, int j, const double L[3], double d[3]) const
    {
        const uint32_t hi[3] = {(uint32_t)xy[i].x, (uint32_t)xy[i].y, (uint32_t)zs[i].x};
        const uint32_t hj[3] = {(uint32_t)xy[j].x, (uint32_t)xy[j].y, (uint32_t)zs[j].x};
        for (int a = 0; a < 3; ++a) {
            const uint64_t u = (((uint64_t)hi[a] << 32) | lo[a][i]) - (((uint64_t)hj[a] << 32) | lo[a][j]);
            const double f = (double)(int)(uint32_t)(u >> 32) + (double)(uint32_t)u * 0x1p-32;
            d[a] = f * (L[a] * 0x1p-32);
        }
    }
    __device__ double r2_64(int i, int j, const double L[3]) const
    {
        double d[3];
        diff64(i, j, L, d);
        return (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
    }
    // the distance rounded once, with the neighbour's s, for the window particle i at p
    __device__ void diff_w(int i, const Pos &, int j, const Scale &, const double L[3], float d[3], float &s) const
    {
        double q[3];
        diff64(i, j, L, q);
        for (int a = 0; a < 3; ++a) d[a] = (float)q[a];
        s = __int_as_float(zs[j].y);
    }
    __device__ void set_s(int k, float v) { zs[k].y = __float_as_int(v); }
    __device__ float get_s(int k) const { return __int_as_float(zs[k].y); }
};

template <> struct ResLds<double> {
    double *x[3], *s, *A;
    int *tag;            // list build: tags by cell, then by tag
    int *cell;
    uint16_t *order;
    static size_t bytes(int n) { return (size_t)n * (40 + 4 + 4 + 2) + 64; }
    __device__ void carve(unsigned char *p, int n)
    {
        for (int a = 0; a < 3; ++a) x[a] = (double *)p + a * n;
        s = x[2] + n;
        A = s + n;
        tag = (int *)(A + n);
        cell = tag + n;
        order = (uint16_t *)(cell + n + 2);
    }
    struct Pos { double x, y, z; };
    struct Scale { double L[3], iL[3]; };
    static __device__ Scale scale(const double L[3])
    {
        return Scale{{L[0], L[1], L[2]}, {1.0 / L[0], 1.0 / L[1], 1.0 / L[2]}};
    }
    __device__ void put(int k, const double q[3], const double[3])
    {
        for (int a = 0; a < 3; ++a) x[a][k] = q[a];
    }
    __device__ Pos own(int k) const { return Pos{x[0][k], x[1][k], x[2][k]}; }
    __device__ void sort_in(int q, int k) { tag[q] = k; }
    static __device__ int cell_axis(const Pos &p, int a, int g, const double iL[3])
    {
        const int c = (int)((a == 0 ? p.x : a == 1 ? p.y : p.z) * iL[a] * (double)g);
        return c < 0 ? 0 : (c >= g ? g - 1 : c);
    }
    __device__ void diff(const Pos &p, int j, const Scale &H, double d[3]) const
    {
        d[0] = p.x - x[0][j];
        d[1] = p.y - x[1][j];
        d[2] = p.z - x[2][j];
        for (int a = 0; a < 3; ++a) d[a] = fma(-H.L[a], rint(d[a] * H.iL[a]), d[a]);
    }
    __device__ void diff_s(const Pos &p, int j, const Scale &H, double d[3], double &sj) const
    {
        diff(p, j, H, d);
        sj = s[j];
    }
    __device__ void diff_w(int, const Pos &p, int j, const Scale &H, const double[3], double d[3], double &sj) const
    {
        diff_s(p, j, H, d, sj);
    }
    __device__ int diff_sorted(const Pos &p, int q, const Scale &H, double d[3]) const
    {
        const int j = tag[q];
        diff(p, j, H, d);
        return j;
    }
    __device__ void set_s(int k, double v) { s[k] = v; }
    __device__ double get_s(int k) const { return s[k]; }
};

// Visit the nn list entries of the particle at slot i, in order; fn(j).
template <class F>
__device__ __forceinline__ void res_list(const uint4 *nl, int64_t S_, int64_t i, int nn, F &&fn)
{
    const uint4 *lp = nl + i;
    const int nfull = nn / CHUNK, rest = nn % CHUNK;
    uint4 q = nn > 0 ? lp[0] : make_uint4(0u, 0u, 0u, 0u);
    for (int c = 0; c < nfull; ++c) {
        const uint4 qn = (c + 1) * CHUNK < nn ? lp[(size_t)(c + 1) * S_] : q;
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < CHUNK; ++e) fn((int)((w[e >> 1] >> (16 * (e & 1))) & 0xffffu));
        q = qn;
    }
    if (rest) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < CHUNK - 1; ++e)
            if (e < rest) fn((int)((w[e >> 1] >> (16 * (e & 1))) & 0xffffu));
    }
}

template <class Real, bool THERMO>
__global__ void __launch_bounds__(RES_MAX_N) k_resident(Buffers B, Launch P, int cur, int nsteps, int k0,
                                                        int max_n, StepArgs st)
{
    extern __shared__ __align__(32) unsigned char smem[];
    __shared__ int nwin, wsum[RES_MAX_N / VBC_WAVE];
    __shared__ unsigned long long evals_s, ent_s;
    __shared__ double red[8][RES_MAX_N / VBC_WAVE];
    const int r = blockIdx.x;
    const RepDev &R = B.reps[r];
    const int n = (int)R.n;
    // an empty slot; a larger replica is not reached: the launch takes the largest of the set
    if (!R.resident || n <= 0 || n > max_n) return;
    const int k = threadIdx.x, nt = blockDim.x, wv = k / VBC_WAVE, ln = k % VBC_WAVE;
    const bool own = k < n;
    const int64_t S_ = P.nslots, base = R.p_off, i = base + k;
    // every condition around a barrier is made a scalar: the compiler takes what it loads into
    // vector registers as different per lane, and splits a loop with a barrier in it between the
    // lanes that leave and those that stay
    const uint32_t fl = (uint32_t)__builtin_amdgcn_readfirstlane((int)B.flags[r]);
    auto any_thread = [](bool v) { return __builtin_amdgcn_readfirstlane(__syncthreads_or(v)) != 0; };
    const double L[3] = {R.L[0], R.L[1], R.L[2]};
    const double iL[3] = {1.0 / L[0], 1.0 / L[1], 1.0 / L[2]};
    const double disp2 = R.disp2;
    const uint64_t key = st.seed + R.seed;
    using Lds = ResLds<Real>;
    Lds T;
    T.carve(smem, max_n);
    const typename Lds::Scale H = Lds::scale(L);
    const PairR<Real> p0 = pair_r<Real>(R.pair[0], R.rc2);
    const PairDev &pd = R.pair[0];
    const double wx1 = pd.x1, wx2 = pd.x2;
    const bool watt = pd.attract;
    double *X = B.x[cur];
    bool bad = false;

    // ---- the state: from the brick layout by way of the next layout's space, or in place ----
    double x[3] = {0, 0, 0}, v[3] = {0, 0, 0}, xr[3] = {0, 0, 0}, F[3] = {0, 0, 0};
    if (!(fl & FLAG_FULL)) {
        for (int lb = wv; lb < R.nbrick; lb += nt / VBC_WAVE) {
            const int cnt = B.bcnt[0][R.b_off + lb];
            for (int t = ln; t < cnt; t += VBC_WAVE) {
                const int64_t j = base + (int64_t)lb * R.bcap + t, d = base + B.tag[j];
                for (int a = 0; a < 3; ++a) {
                    B.xs[3 * d + a] = X[3 * j + a];
                    B.vs[a * S_ + d] = B.v[a * S_ + j];
                }
            }
        }
        __syncthreads();
    }
    if (own) {
        for (int a = 0; a < 3; ++a) {
            double t = (fl & FLAG_FULL) ? X[3 * i + a] : B.xs[3 * i + a];
            if (!isfinite(t)) {
                bad = true;
                t = 0.0;
            }
            x[a] = wrap1(t, L[a]);
            v[a] = (fl & FLAG_FULL) ? B.v[a * S_ + i] : B.vs[a * S_ + i];
            F[a] = B.Fst[a * S_ + i];
            xr[a] = B.xref[a * S_ + i];
        }
        B.tag[i] = k;
    }

    uint64_t step = B.step[r];
    const bool need_eval = !(fl & FLAG_RES);
    bool moved = false;  // the list is due (scalar)
    int nn = own ? (int)B.nn[i] : 0;

    // after a drift: wrap, and whether the particle has left its buffer
    auto drifted = [&]() {
        double d2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            x[a] = wrap1(x[a], L[a]);
            if (!isfinite(x[a])) {
                bad = true;
                x[a] = 0.0;
            }
            double dd = x[a] - xr[a];
            dd -= L[a] * rint(dd * iL[a]);
            d2 += dd * dd;
        }
        return d2 > disp2;
    };

    if (!need_eval) {
        bool mv = false;
        if (own) {
            integrate_one(st, MODE_MID, true, F, v, x, key, (uint64_t)k, step);
            mv = drifted();
        }
        moved = any_thread(mv);
    }

    // step -1 evaluates the forces that the opening half-kick needs where none are stored; step
    // -2 makes a list lost to the brick layout again from its own reference positions
    const int m0 = need_eval ? ((fl & FLAG_XREF) ? -2 : -1) : 0;
    for (int m = m0; m < nsteps; ++m) {
        // ---- positions into LDS; a list when one is due ----
        if (own) T.put(k, m == -2 ? xr : x, iL);
        if (k == 0) {
            nwin = 0;
            evals_s = 0ull;
            ent_s = 0ull;
        }
        __syncthreads();
        if ((need_eval && m == m0) || moved) {
            moved = false;
            const typename Lds::Pos pi = own ? T.own(k) : typename Lds::Pos{};
            if (m > -2 && own) {
                bool lost = false;
                for (int a = 0; a < 3; ++a) {
                    // further than one cell since the last build: unstable dynamics
                    const int dc = abs(cell_of(x[a], R.h[a], R.nc[a]) - cell_of(xr[a], R.h[a], R.nc[a]));
                    if (m >= 0 && min(dc, R.nc[a] - dc) > 1) lost = true;
                    xr[a] = x[a];
                }
                if (lost) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_LOST);
            }
            // cells: at most one per particle, none smaller than the list radius; in a small
            // system every particle is a candidate, in one cell
            const bool all = n < 128;
            int g[3] = {1, 1, 1};
            if (!all) {
                int c = 3;
                while (c < 10 && (c + 1) * (c + 1) * (c + 1) <= n) ++c;
                for (int a = 0; a < 3; ++a) g[a] = min(c, R.nc[a]);
            }
            const int ncell = g[0] * g[1] * g[2];
            const int cx = all ? 0 : Lds::cell_axis(pi, 0, g[0], iL), cy = all ? 0 : Lds::cell_axis(pi, 1, g[1], iL),
                      cz = all ? 0 : Lds::cell_axis(pi, 2, g[2], iL);
            const int cid = cx + g[0] * (cy + g[1] * cz);
            if (k < ncell) T.cell[k] = 0;  // ncell <= n <= threads
            __syncthreads();
            if (own) atomicAdd(&T.cell[cid], 1);
            __syncthreads();
            {
                const int c = k < ncell ? T.cell[k] : 0;
                int incl = c;
#pragma unroll
                for (int o = 1; o < VBC_WAVE; o <<= 1) {
                    const int t = __shfl_up(incl, o, VBC_WAVE);
                    if (ln >= o) incl += t;
                }
                if (ln == VBC_WAVE - 1) wsum[wv] = incl;
                __syncthreads();
                int off = incl - c;
                for (int w = 0; w < wv; ++w) off += wsum[w];
                if (k < ncell) T.cell[k] = off;
            }
            __syncthreads();
            // members in any order (a cell's counter runs to its end), then ranked by tag
            if (own) T.order[atomicAdd(&T.cell[cid], 1)] = (uint16_t)k;
            __syncthreads();
            // cell c now ends at cell[c], where the next one starts
            auto begin = [&](int c) { return c ? T.cell[c - 1] : 0; };
            if (own) {
                const int lo = begin(cid), hi = T.cell[cid];
                int rank = lo;
                for (int j = lo; j < hi; ++j) rank += (int)T.order[j] < k ? 1 : 0;
                T.sort_in(rank, k);
            }
            __syncthreads();
            const Real rl2 = (Real)(R.rlist2 * (1.0 + 1e-6));
            const int kmax = P.k_max;
            bool ovf = false;
            if (own) {
                int e = 0;
                nn = 0;
                uint32_t b0 = 0u, b1 = 0u, b2 = 0u, b3 = 0u;
                uint4 *wp = B.nl + i;
                auto chunk = [&] {  // the oldest entry first
                    return make_uint4((b3 >> 16) | (b3 << 16), (b2 >> 16) | (b2 << 16), (b1 >> 16) | (b1 << 16),
                                      (b0 >> 16) | (b0 << 16));
                };
                auto push = [&](uint32_t j) {
                    b3 = __builtin_amdgcn_alignbit(b3, b2, 16);
                    b2 = __builtin_amdgcn_alignbit(b2, b1, 16);
                    b1 = __builtin_amdgcn_alignbit(b1, b0, 16);
                    b0 = (b0 << 16) | j;
                };
                // segments of up to 32 candidates: a tight loop marks those within the radius, a
                // second one appends only the marked (as the list build of the bricks)
                auto visit = [&](int lo, int hi) {
                    for (int q0 = lo; q0 < hi; q0 += 32) {
                        const int cnt = min(32, hi - q0);
                        uint32_t near = 0u;
                        for (int q = 0; q < cnt; ++q) {
                            Real d[3];
                            const int j = T.diff_sorted(pi, q0 + q, H, d);
                            const Real r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                            near |= (r2 < rl2 && j != k) ? 1u << q : 0u;
                        }
                        while (near) {
                            const int q = __builtin_ctz(near);
                            near &= near - 1u;
                            uint32_t j;
                            if constexpr (sizeof(Real) == 4) j = (uint32_t)T.sorted[q0 + q].w;
                            else j = (uint32_t)T.tag[q0 + q];
                            push(j);
                            ++nn;
                            if (++e == CHUNK) {
                                if (nn <= kmax) *wp = chunk();
                                wp += S_;
                                e = 0;
                            }
                        }
                    }
                };
                if (all) {
                    visit(0, n);
                } else {
                    for (int dz = -1; dz <= 1; ++dz)
                        for (int dy = -1; dy <= 1; ++dy) {
                            const int z = cz + dz + (cz + dz < 0 ? g[2] : 0) - (cz + dz >= g[2] ? g[2] : 0);
                            const int y = cy + dy + (cy + dy < 0 ? g[1] : 0) - (cy + dy >= g[1] ? g[1] : 0);
                            const int row = g[0] * (y + g[1] * z);
                            // three cells along x: one range, or two where the row wraps
                            visit(begin(row + max(cx - 1, 0)), T.cell[row + min(cx + 1, g[0] - 1)]);
                            if (cx == 0) visit(begin(row + g[0] - 1), T.cell[row + g[0] - 1]);
                            if (cx == g[0] - 1) visit(begin(row), T.cell[row]);
                        }
                }
                if (e && nn <= kmax) {
                    for (; e < CHUNK; ++e) push(0u);
                    *wp = chunk();
                }
                if (nn > kmax) {
                    ovf = true;
                    nn = kmax;
                }
                B.nn[i] = (uint16_t)nn;
            }
            if (ovf) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_NLIST_OVERFLOW);
            const unsigned long long entries = wave_sum((unsigned long long)nn);
            if (ln == 0 && entries) atomicAdd(&ent_s, entries);
            for (int lb = k; lb < R.nbrick; lb += nt) B.bentries[R.b_off + lb] = 0u;
            __syncthreads();
            if (k == 0) {
                B.bentries[R.b_off] = (uint32_t)ent_s;
                if (m > -2) B.stats[4 * r + 0] += 1ull;  // not for the same list made again
            }
        }
        if (m == -2) continue;

        // ---- counts ----
        const bool stats = m < 0 || (k0 + m) % 8 == 0;
        const typename Lds::Pos pi = own ? T.own(k) : typename Lds::Pos{};
        int inside = 0;
        if (own) {
            double nc = 0.0;
            Real part = Real(0);
            int e = 0;
            res_list(B.nl, S_, i, nn, [&](int j) {
                Real d[3];
                T.diff(pi, j, H, d);
                const Real r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                if (stats) inside += r2 < p0.rc2 ? 1 : 0;
                const Real uu = clamp01(fma(sqrt_r(r2), p0.inv_dw, p0.nrl_dw));
                const Real qq = fma(-uu, uu, Real(1));
                part = fma(qq, qq, part);
                if (++e == CHUNK) {
                    nc += (double)part;
                    part = Real(0);
                    e = 0;
                }
            });
            nc += (double)part;
            const double mg = sizeof(Real) == 4 ? COUNT_MARGIN : 0.0;
            T.A[k] = Real(0);
            if (watt && nc > wx1 - mg && nc < wx2 + mg) {
                T.order[atomicAdd(&nwin, 1)] = (uint16_t)k;
                B.nd[i] = nc;
            }
            T.set_s(k, (Real)omega_d64(nc, wx1, wx2));
        }
        if (stats) {
            const int ev = wave_sum(inside);
            if (ln == 0 && ev) atomicAdd(&evals_s, (unsigned long long)ev);
        }
        __syncthreads();
        const int nw = __builtin_amdgcn_readfirstlane(nwin);
        if (m >= 0) ++step;
        if (stats && k == 0) {
            B.bevals[R.b_off] += evals_s;
            B.stats[4 * r + 3] += 1ull;
        }

        // ---- particles in a switching window, eight lanes each: recount, dU/dn ----
        if (nw > 0) {
            const int e = k % CHUNK, grp = k / CHUNK, ng = nt / CHUNK;
            if constexpr (sizeof(Real) == 4) {
                for (int w = grp; w < nw; w += ng) {
                    const int kw = T.order[w], nj = B.nn[base + kw];
                    double acc = 0.0;
                    for (int c = 0; c * CHUNK < nj; ++c)
                        if (c * CHUNK + e < nj) {
                            const int j = ((const uint16_t *)(B.nl + (size_t)c * S_ + base + kw))[e];
                            acc += count_term64(T.r2_64(kw, j, L), pd);
                        }
#pragma unroll
                    for (int o = CHUNK / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, CHUNK);
                    if (e == 0) {
                        B.nd[base + kw] = acc;
                        T.set_s(kw, (Real)omega_d64(acc, wx1, wx2));
                    }
                }
                __syncthreads();
            }
            for (int w = grp; w < nw; w += ng) {
                const int kw = T.order[w], nj = B.nn[base + kw];
                const typename Lds::Pos pw = T.own(kw);
                double acc = 0.0;
                for (int c = 0; c * CHUNK < nj; ++c)
                    if (c * CHUNK + e < nj) {
                        const int j = ((const uint16_t *)(B.nl + (size_t)c * S_ + base + kw))[e];
                        Real d[3], sj;
                        T.diff_w(kw, pw, j, H, L, d, sj);
                        const Real r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                        const Real uu = (sqrt_r(r2) - p0.m) * p0.inv_w;
                        const Real qq = Real(1) - uu * uu;
                        if (qq > Real(0)) acc += (double)(sj * (-p0.E_a * qq * qq));
                    }
#pragma unroll
                for (int o = CHUNK / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, CHUNK);
                if (e == 0) T.A[kw] = (Real)(omega_dd64(B.nd[base + kw], wx1, wx2) * acc) * p0.c_c;
            }
            __syncthreads();
        }

        // ---- forces and the integrator ----
        const int mode = m < 0 ? MODE_MID : (m == nsteps - 1 ? MODE_LAST : MODE_MID);
        bool mv = false;
        double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (own) {
            const Real si = T.get_s(k), cAi = T.A[k], cai = p0.c_a * si;
            Real fx = 0, fy = 0, fz = 0, ei = 0, ea = 0;
            Real wxx = 0, wyy = 0, wzz = 0, wxy = 0, wxz = 0, wyz = 0;
            // the terms of k_force's one-type path
            res_list(B.nl, S_, i, nn, [&](int j) {
                Real d[3], sj;
                T.diff_s(pi, j, H, d, sj);
                const Real cAj = T.A[j];
                const Real r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                const Real rinv = rsqrt_r(r2 > Real(1e-30) ? r2 : Real(1e-30));
                const Real rr = r2 * rinv;
                const Real pr = fmin(fma(r2, p0.k_r, p0.c_r), Real(0));
                const Real uu = fma(rr, p0.inv_w, p0.nm_w);
                const Real qq = fmax(fma(-uu, uu, Real(1)), Real(0));
                const Real uc = clamp01(fma(rr, p0.inv_dw, p0.nrl_dw));
                const Real gg = uc * fma(-uc, uc, Real(1));
                const Real t = fma(cAi + cAj, gg, cai * sj * uu * qq);
                const Real phr = fma(t, rinv, pr);
                fx -= phr * d[0];
                fy -= phr * d[1];
                fz -= phr * d[2];
                if (THERMO) {
                    const Real tc = fmax(fma(-r2, p0.inv_rr2, Real(1)), Real(0));
                    ei = fma(tc, tc, ei);
                    ea = fma(sj * qq, qq, ea);
                    wxx -= phr * d[0] * d[0];
                    wyy -= phr * d[1] * d[1];
                    wzz -= phr * d[2] * d[2];
                    wxy -= phr * d[0] * d[1];
                    wxz -= phr * d[0] * d[2];
                    wyz -= phr * d[1] * d[2];
                }
            });
            F[0] = (double)fx;
            F[1] = (double)fy;
            F[2] = (double)fz;
            if (!(isfinite(F[0]) && isfinite(F[1]) && isfinite(F[2]))) bad = true;
            if (THERMO) {
                acc[0] = 0.5 * (double)(p0.E_r * ei - p0.E_a * si * ea);
                acc[2] = 0.5 * (double)wxx;
                acc[3] = 0.5 * (double)wyy;
                acc[4] = 0.5 * (double)wzz;
                acc[5] = 0.5 * (double)wxy;
                acc[6] = 0.5 * (double)wxz;
                acc[7] = 0.5 * (double)wyz;
            }
            integrate_one(st, mode, m < 0, F, v, x, key, (uint64_t)k, step);
            if (mode != MODE_LAST) mv = drifted();
        }
        if (THERMO) {
            const double w = wave_sum8(acc);
            if ((ln & 7) == 0) red[ln >> 3][wv] = w;
        }
        moved = any_thread(mv);
        if (THERMO && m >= 0 && k < 8) {
            // 64 consecutive tags at a time, whatever the workgroup's size
            const int nb = (n + VBC_WAVE - 1) / VBC_WAVE;
            double sum = 0.0;
            if (k == 1) {
                for (int w = 0; w < nb; ++w) sum += (red[2][w] + red[3][w]) + red[4][w];
            } else {
                for (int w = 0; w < nb; ++w) sum += red[k][w];
            }
            double *A = B.thermo + (size_t)r * THERMO_WORDS;
            A[1 + k] = sum;
            A[9 + k] += sum;
            if (k == 0) A[0] += 1.0;
        }
    }
    if (own)
        for (int a = 0; a < 3; ++a) {
            X[3 * i + a] = x[a];
            B.v[a * S_ + i] = v[a];
            B.Fst[a * S_ + i] = F[a];
            B.xref[a * S_ + i] = xr[a];
        }
    if (bad) atomicOr(&B.flags[r], (uint32_t)VBC_FLAG_NONFINITE);
    if (k == 0) {
        B.step[r] = step;
        atomicAnd(&B.flags[r], ~(uint32_t)VBC_FLAG_REBUILD);
        atomicOr(&B.flags[r], (uint32_t)(FLAG_FULL | FLAG_RES | FLAG_XREF));
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static inline unsigned blocks_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }
// Waves of a list build's workgroup, and the LDS up to which its output windows may grow it
// (two workgroups on a CU); LDS_MAX: what one workgroup can have, less the static part.
constexpr int LIST_WAVES = 12, LIST_WAVES_ALONE = 16;
constexpr size_t LIST_LDS = 80 * 1024 - 256, LDS_MAX = 160 * 1024 - 256;

static inline unsigned dense_grid(int nb, size_t lds)
{
    const int n = std::max(1, std::min(8, (int)((LDS_MAX + 256) / (lds + 1024))));
    return (unsigned)std::min(nb, std::max(256 * n, (nb + VBC_WAVE - 1) / VBC_WAVE));
}
static inline unsigned brick_grid(int nb) { return (unsigned)(((nb + 7) / 8) * 8); }

static size_t tabs_bytes(const Launch &P)
{
    int nh_cap = (P.nh_max + 3) & ~3;
    return ((size_t)5 * nh_cap * sizeof(int) + 31) & ~(size_t)31;
}

static size_t sort_bytes(const Launch &P)
{
    return (size_t)4 * P.bcap_max * sizeof(int) + (size_t)3 * P.ncb_max * sizeof(int);
}

size_t lds_bytes_sort(const Launch &P) { return tabs_bytes(P) + sort_bytes(P); }
// the list build without its output windows: tables, grid-order positions (16 B), cell
// offsets, grid -> staging order (2 B)
static size_t nlist_stage_bytes(const Launch &P)
{
    const size_t nh_cap = (size_t)((P.nh_max + 3) & ~3);
    return tabs_bytes(P) + (size_t)(P.lds_cap + SCAN_UNROLL) * 16 + (nh_cap + 4) * sizeof(int) +
           (size_t)P.lds_cap * 2;
}
static size_t nlist_wave_bytes(int win) { return (size_t)NL_PPW * (win + CHUNK) * sizeof(uint16_t); }
size_t lds_bytes_nlist(const Launch &P)
{
    return nlist_stage_bytes(P) + (size_t)(P.list_block / VBC_WAVE) * nlist_wave_bytes(P.list_win);
}
// what the handle's check asks for: the build has hardly any static LDS, and one wave's
// smallest window fits into the room that the check leaves for it
size_t lds_need_nlist(const Launch &P)
{
    return std::max(nlist_stage_bytes(P), lds_bytes_nlist(P) - nlist_wave_bytes(32));
}

// Lanes per particle (2^split) of the FP64 count and force passes of a single replica.  A small
// or mid-sized system leaves each SIMD a wave or two, and the pass then takes the length of one
// particle's chain of list chunks (with FP64 square roots and divisions); two or four lanes take
// every second or fourth chunk, and the staging is spread over as many more threads.  The
// chunks' sums are added in the list's order, so results do not depend on the lanes.  Us a step at density 0.3 with one, two, four lanes:
// 1000 particles 27.3, 25.8, 24.6; 20,000 28.9, 27.1, 25.9; 100,000 67.7, 63.0, 61.8;
// 200,000 85.1, 75.5, 92.7.  At density 0.5 (four waves a brick) 20,000 32.1, 31.2, 33.5 and
// 50,000 40.0, 41.5, 47.9.  Lists of less than a chunk have nothing to share (22.7, 22.0, 23.4
// at 10,000 and 0.05).  FP32 passes gain 3 % at most and lose 2 % at density 0.5; the force
// pass with energies holds too many registers for the extra waves (31.9 to 32.0).
void split_shape(Launch &P)
{
    auto fits = [&](int l, int threads, int64_t waves) {
        return (P.block << l) <= threads && (int64_t)P.nbrick_tot * ((P.block << l) / VBC_WAVE) <= waves;
    };
    P.split = 0;
    if (P.precision != VBC_FP64 || P.k_mean < CHUNK) return;
    if (fits(2, 768, 12288)) P.split = 2;
    else if (fits(1, 384, INT64_MAX) || fits(1, 768, 2048)) P.split = 1;
}

// The list build's workgroup: a wave for each 21 particles of a mean brick, and one for
// fluctuations, up to twelve (two such workgroups fill a CU's registers), fewer where the
// windows would take a second workgroup's LDS.  Where the staging alone leaves room for one
// workgroup only, as many waves as it can use.  (Passes of ten steps or a tick, us: a million
// particles, 455 a brick, 1389 with twelve waves, 1484 with six; twenty systems of 4000, 52 a
// brick, 1150 with three, 1206 with two; a pool laid out for density 1, 416 a brick, 1066 with
// sixteen, 1095 with eleven, 1254 with four.)  The windows hold a mean list and three standard
// deviations, in whole chunks between 32 and 64 entries.
void list_shape(Launch &P)
{
    const int win = (int)(P.k_mean + 3.0 * std::sqrt(P.k_mean) + CHUNK) & ~(CHUNK - 1);
    const size_t base = nlist_stage_bytes(P);
    P.list_win = std::max(32, std::min(64, win));
    const size_t wb = nlist_wave_bytes(P.list_win);
    const int want = std::max(1, std::min(LIST_WAVES_ALONE, (int)(P.own_mean / NL_PPW + 1.5)));
    int waves = std::min(want, LIST_WAVES);
    while (waves > 1 && base + waves * wb > LIST_LDS) --waves;
    if (3 * waves < 2 * std::min(want, LIST_WAVES)) waves = want;
    while (waves > 1 && base + waves * wb > LDS_MAX) --waves;
    if (base + waves * wb > LDS_MAX) P.list_win = 32;
    P.list_block = waves * VBC_WAVE;
}
size_t lds_bytes_count(const Launch &P)
{
    return (size_t)(P.lds_cap + 1) * (P.precision == VBC_FP64 ? 32 : (P.multi ? 16 : 12));
}
size_t lds_bytes_embed(const Launch &P) { (void)P; return 0; }
// bond tests (observables, clusters, bond tracker): FP32 staging, and the brick's forest
static size_t staged_bytes(const Launch &P) { return (size_t)(P.lds_cap + 1) * (P.multi ? 16 : 12); }
size_t lds_bytes_bonds(const Launch &P)
{
    return staged_bytes(P) + (size_t)P.bcap_max * sizeof(int32_t) + 16;
}
size_t lds_bytes_force(const Launch &P)
{
    const size_t real = P.precision == VBC_FP64 ? 8 : 4;
    return (size_t)(P.lds_cap + 1) * real * (P.multi ? 6 : 5);
}

// Whether a pass is two launches (parts).  A layout that holds local densities far above the
// mean reserves LDS for them in every workgroup, so that one to three workgroups of a few waves
// stand on a CU and a pass takes many rounds of the chip.  The bricks of usual density (as many
// staged as a layout without a stated maximum has room for) go first, with LDS for those, then
// the others.  Worth it where it saves rounds enough: an idle second launch costs 1.6 us and
// its bricks wait for the first.  The force pass gains from half a round (30,000 particles at
// density 0.05 27.6 and 26.1 us a step; with none saved, FP64 at 0.3, 60.3 and 61.9), the count
// pass from one (0.7 saved: 88.6 and 90.1), the list pass, not due in most steps, from two (1.9
// saved: 49.2 and 51.1).  The waves a CU can hold follow the kernels' registers: of one type 8
// per SIMD in the count pass and the bond analyses (the tracker 6), 6 in the FP32 and 5 in the
// FP64 force pass, 6 in the list build.  Laid out for density 1, all passes in one and two launches:
// 100,000 particles at 0.05 59.2 and 39.9 (FP64 128 and 62), 400,000 199.6 and 95.1, 200,000
// at 0.15 72.3 and 60.0; ten steps of twenty tracked systems of 4000 at 0.05 1151 and 766, a
// tick of a pool of 24 at 0.3 1057 and 872.
void part_shape(Launch &P)
{
    const int small = P.cap_usual;
    P.small_count = P.small_force = P.small_list = P.small_bonds = 0;
    if (small <= 0 || small >= P.stage_cap) return;
    auto rounds = [&](int64_t nb, size_t lds, int threads, int waves_cu) {
        const int64_t n = std::min<int64_t>((LDS_MAX + 256) / (lds + 1024), waves_cu / (threads / VBC_WAVE));
        return std::max(1.0, (double)nb / (double)(256 * std::max<int64_t>(n, 1)));
    };
    Launch F = P, Q = P;
    Q.lds_cap = small;
    const int64_t nb = P.nbrick_tot;
    const int threads = P.block << (P.one ? P.split : 0);
    auto saves = [&](int64_t n, size_t (*lds)(const Launch &), int tf, int tq, int waves, double least) {
        return rounds(n, lds(F), tf, waves) - rounds(n, lds(Q), tq, waves) >= least ? small : 0;
    };
    P.small_count = saves(nb, lds_bytes_count, threads, threads, 32, 1.0);
    P.small_force = saves(nb, lds_bytes_force, threads, threads, P.precision == VBC_FP64 ? 20 : 24, 0.5);
    P.small_bonds = saves(nb, lds_bytes_bonds, P.block, P.block, 32, 1.0);
    list_shape(F);
    list_shape(Q);
    // of several replicas, some are due for a build at a time
    P.small_list = saves(P.lists ? (nb + 1) / 2 : nb, lds_bytes_nlist, F.list_block, Q.list_block, 24, 2.0);
}

namespace {
thread_local hipEvent_t g_ev_start = nullptr, g_ev_stop = nullptr;
thread_local int g_ev_used = 0;
thread_local hipError_t g_ev_err = hipSuccess;

// A launch of a timed pass: through hipExtLaunchKernel while timing events are set (its
// error, if any, is kept for launch_events_used's caller), else the plain launch.
template <typename... P, typename... A>
inline void tlaunch(void (*k)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t s, A... a)
{
    if (g_ev_stop) {
        std::tuple<std::decay_t<P>...> args(a...);
        void *ptrs[sizeof...(P) > 0 ? sizeof...(P) : 1];
        std::apply(
            [&](auto &...x) {
                int n = 0;
                ((ptrs[n++] = (void *)&x), ...);
            },
            args);
        const hipError_t e = hipExtLaunchKernel((const void *)k, grid, block, ptrs, lds, s, g_ev_start,
                                                g_ev_stop, 0);
        if (e != hipSuccess && g_ev_err == hipSuccess) g_ev_err = e;
        g_ev_start = nullptr;
        ++g_ev_used;
    } else {
        k<<<grid, block, lds, s>>>(a...);
    }
}
}  // namespace

void set_launch_events(hipEvent_t start, hipEvent_t stop)
{
    g_ev_start = start;
    g_ev_stop = stop;
    g_ev_used = 0;
    g_ev_err = hipSuccess;
}

int launch_events_used() { return g_ev_used; }

hipError_t launch_events_error() { return g_ev_err; }

hipError_t launch_set_state(const Buffers &B, const Launch &P, int cur, int r, int64_t n,
                            const double *x, const double *v, const int32_t *type,
                            int64_t in_off, int64_t in_stride, uint64_t step0, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_set_state<<<blocks_for(n, 256), 256, 0, s>>>(B, P.nslots, cur, r, in_off, in_stride, x, v,
                                                    type, step0);
    return hipGetLastError();
}

// Particles for which the state is read by way of records: enough that the scattered lines
// are what takes the time, and no more than keep the records, their sources and the caller's
// arrays (148 bytes a particle) in the 256 MB last-level cache.  Us, in one pass and in two:
// 200,000 17.0 and 18.0, 400,000 34.7 and 29.5, 1,000,000 82.9 and 60.6, 2,000,000 164 and 202.
constexpr int64_t RECORDS_MIN = 300000, RECORDS_MAX = 1700000;

hipError_t launch_get_state(const Buffers &B, const Launch &P, int cur, int r, int64_t n, int64_t nslot,
                            int64_t out_off, int64_t out_stride, double *x, double *v,
                            hipStream_t s)
{
    if (nslot <= 0) return hipSuccess;
    if (n >= RECORDS_MIN && n <= RECORDS_MAX && x && v) {
        k_get_records<<<blocks_for(nslot, 256), 256, 0, s>>>(B, P.nslots, cur, r);
        k_put_records<<<blocks_for(n, 256), 256, 0, s>>>(B, r, out_off, out_stride, x, v);
        return hipGetLastError();
    }
    k_get_state<<<blocks_for(nslot, 256), 256, 0, s>>>(B, P.nslots, cur, r, out_off, out_stride,
                                                        x, v);
    return hipGetLastError();
}

hipError_t launch_set_state_all(const Buffers &B, const Launch &P, int cur, const double *x, const double *v,
                                const int32_t *type, uint64_t step0, hipStream_t s)
{
    // one wave per brick where bricks are small
    k_set_state_all<<<P.nbrick_tot, P.bcap_max <= 128 ? VBC_WAVE : 256, 0, s>>>(B, P.nslots, cur, P.ntot, x, v, type, step0);
    return hipGetLastError();
}

hipError_t launch_get_state_all(const Buffers &B, const Launch &P, int cur, double *x, double *v, hipStream_t s)
{
    k_get_state_all<<<P.nbrick_tot, P.bcap_max <= 128 ? VBC_WAVE : 256, 0, s>>>(B, P.nslots, cur, P.ntot, x, v);
    return hipGetLastError();
}

hipError_t launch_flags(const Buffers &B, int r_lo, int r_n, uint32_t bits, bool set,
                        hipStream_t s)
{
    if (r_n <= 0) return hipSuccess;
    k_flags<<<blocks_for(r_n, 64), 64, 0, s>>>(B, r_lo, r_n, bits, set ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_admit(const Buffers &B, int r, int64_t nthreads, hipStream_t s)
{
    k_admit<<<blocks_for(std::max<int64_t>(nthreads, 1), 256), 256, 0, s>>>(B, r);
    return hipGetLastError();
}

hipError_t launch_retire(const Buffers &B, int r, int b_off, int nbrick, hipStream_t s)
{
    k_retire<<<blocks_for(std::max(nbrick, 1), 256), 256, 0, s>>>(B, r, b_off, nbrick);
    return hipGetLastError();
}

hipError_t launch_stamp(const Buffers &B, hipStream_t s)
{
    k_stamp<<<1, 1, 0, s>>>(B, (uint32_t)(STAMP_CAP - 1));
    return hipGetLastError();
}

// A pass over P's bricks in one launch, or in two: with LDS for `small` staged particles over the
// bricks that have no more, then with the full capacity over the others.
template <class F>
static void parts(const Launch &P, int small, F &&launch)
{
    if (!small) return launch(P);
    Launch Q = P;
    Q.lds_cap = Q.t_hi = small;
    launch(Q);
    Q = P;
    Q.t_lo = small;
    launch(Q);
}

static void launch_nlist(const Buffers &B, const Launch &P, int cur, hipStream_t s)
{
    parts(P, P.small_list, [&](Launch Q) {
        list_shape(Q);
        if (Q.t_lo >= 0) Q.list_block = std::min(Q.list_block, DENSE_BLOCK);
        if (Q.t_lo >= 0) tlaunch(k_nlist_dense, dense_grid(Q.nb_launch, lds_bytes_nlist(Q)), Q.list_block, lds_bytes_nlist(Q), s, B, Q, cur);
        else tlaunch(k_nlist, brick_grid(Q.nb_launch), Q.list_block, lds_bytes_nlist(Q), s, B, Q, cur);
    });
}

// Full build of replica r (P covering its bricks) if its input is unsorted: bin and sort it
// from caller order, then build its list.  k_resort skips FULL replicas, so the same kernel as
// in an incremental rebuild serves (due: a replica that is only due for a rebuild has no next
// layout yet).
hipError_t launch_full_build(const Buffers &B, const Launch &P, int cur, int r, int64_t n,
                             hipStream_t s)
{
    Launch Q = P;
    Q.due = FLAG_FULL;
    if (n > 0) tlaunch(k_gbin, blocks_for(n, 256), 256, 0, s, B, Q.nslots, cur, r);
    tlaunch(k_gsort, brick_grid(Q.nb_launch), Q.block, sort_bytes(Q), s, B, Q, cur);
    launch_nlist(B, Q, cur, s);
    tlaunch(k_full_done, 1, 64, 0, s, B, r, 1);
    return hipGetLastError();
}

// Full builds of every replica with unsorted input, over all bricks at once.
hipError_t launch_full_build_all(const Buffers &B, const Launch &P, int cur, hipStream_t s)
{
    Launch Q = P;
    Q.b_lo = 0;
    Q.nb_launch = P.nbrick_tot;
    Q.list = -1;
    Q.due = FLAG_FULL;
    tlaunch(k_gbin_all, P.nbrick_tot, P.bcap_max <= 128 ? VBC_WAVE : 256, 0, s, B, cur);
    tlaunch(k_gsort, brick_grid(Q.nb_launch), Q.block, sort_bytes(Q), s, B, Q, cur);
    launch_nlist(B, Q, cur, s);
    tlaunch(k_full_done, blocks_for(P.nrep, 256), 256, 0, s, B, 0, P.nrep);
    return hipGetLastError();
}

static void launch_worklist(const Buffers &B, const Launch &P, hipStream_t s)
{
    const int groups = std::min(64, (P.nbrick_tot + WL_PER_GROUP - 1) / WL_PER_GROUP);
    tlaunch(k_worklist, groups, 1024, 0, s, B, P.nrep, P.list == 0 ? 0 : 1);
}

// Incremental rebuild of the replicas whose REBUILD flag is set.  A launch over all bricks of
// several replica slots first makes the step's work lists and visits only the bricks of those
// replicas.
hipError_t launch_rebuild(const Buffers &B, const Launch &P, int cur, hipStream_t s)
{
    Launch Q = P;
    if (P.lists) {
        launch_worklist(B, P, s);
        Q.list = 1;
    }
    tlaunch(k_resort, brick_grid(Q.nb_launch), Q.block, lds_bytes_sort(Q), s, B, Q, cur);
    launch_nlist(B, Q, cur, s);
    return hipGetLastError();
}

template <class Real, bool MULTI, bool STATS>
static void launch_count_t(const Buffers &B, const Launch &P, int cur, double *n_out, int advance, hipStream_t s)
{
    const size_t lds = lds_bytes_count(P);
    const unsigned g = brick_grid(P.nb_launch);
    if (P.t_lo >= 0) tlaunch(k_count_dense<Real, MULTI, STATS>, dense_grid(P.nb_launch, lds), std::min(P.block, DENSE_BLOCK), lds, s, B, P, cur, n_out, advance);
    else if (!P.one || (P.t_hi != INT32_MAX && !P.split)) tlaunch(k_count<Real, MULTI, STATS, false, false>, g, P.block, lds, s, B, P, cur, n_out, advance, OneRep<false>{0});
    else if (!P.split) tlaunch(k_count<Real, MULTI, STATS, true, false>, g, P.block, lds, s, B, P, cur, n_out, advance, OneRep<true>{*P.one});
    else if constexpr (sizeof(Real) == 8)
        tlaunch(k_count<Real, MULTI, STATS, true, true>, g, P.block << P.split, lds, s, B, P, cur, n_out, advance, OneRep<true>{*P.one});
}

template <class Real, bool MULTI>
static void launch_count_t(const Buffers &B, const Launch &P, int cur, double *n_out, int advance,
                           bool stats, hipStream_t s)
{
    if (stats) launch_count_t<Real, MULTI, true>(B, P, cur, n_out, advance, s);
    else launch_count_t<Real, MULTI, false>(B, P, cur, n_out, advance, s);
}

hipError_t launch_count(const Buffers &B, const Launch &P, int cur, double *n_out, int advance,
                        bool stats, hipStream_t s)
{
    parts(P, P.small_count, [&](const Launch &Q) {
        if (Q.precision == VBC_FP64) {
            if (Q.multi) launch_count_t<double, true>(B, Q, cur, n_out, advance, stats, s);
            else launch_count_t<double, false>(B, Q, cur, n_out, advance, stats, s);
        } else {
            if (Q.multi) launch_count_t<float, true>(B, Q, cur, n_out, advance, stats, s);
            else launch_count_t<float, false>(B, Q, cur, n_out, advance, stats, s);
        }
    });
    return hipGetLastError();
}

hipError_t launch_embed(const Buffers &B, const Launch &P, int cur, hipStream_t s)
{
    unsigned g = brick_grid(P.nb_launch);
    bool multi = P.multi != 0;
    const int bs = EMBED_WAVES * VBC_WAVE;
    size_t lds = 0;
    if (P.precision == VBC_FP64) {
        if (multi) tlaunch(k_embed<double, true>, g, bs, lds, s, B, P, cur);
        else tlaunch(k_embed<double, false>, g, bs, lds, s, B, P, cur);
    } else {
        if (multi) tlaunch(k_embed<float, true>, g, bs, lds, s, B, P, cur);
        else tlaunch(k_embed<float, false>, g, bs, lds, s, B, P, cur);
    }
    return hipGetLastError();
}

template <class Real, bool MULTI, bool THERMO>
static void launch_force_t(const Buffers &B, const Launch &P, int cur, Mode mode, const StepArgs &st,
                           double *F_out, double *e_out, hipStream_t s)
{
    const size_t lds = lds_bytes_force(P);
    const unsigned g = brick_grid(P.nb_launch);
    const int m = (int)mode;
    if (P.t_lo >= 0) tlaunch(k_force_dense<Real, MULTI, THERMO>, dense_grid(P.nb_launch, lds), std::min(P.block, DENSE_BLOCK), lds, s, B, P, cur, m, st, F_out, e_out);
    else if (!P.one || (P.t_hi != INT32_MAX && (THERMO || !P.split))) tlaunch(k_force<Real, MULTI, THERMO, false, false>, g, P.block, lds, s, B, P, cur, m, st, F_out, e_out, OneRep<false>{0});
    else if (THERMO || !P.split) tlaunch(k_force<Real, MULTI, THERMO, true, false>, g, P.block, lds, s, B, P, cur, m, st, F_out, e_out, OneRep<true>{*P.one});
    else if constexpr (sizeof(Real) == 8 && !THERMO)
        tlaunch(k_force<Real, MULTI, false, true, true>, g, P.block << P.split, lds, s, B, P, cur, m, st, F_out, e_out, OneRep<true>{*P.one});
}

template <class Real, bool MULTI>
static void launch_force_t(const Buffers &B, const Launch &P, int cur, Mode mode, bool thermo,
                           const StepArgs &st, double *F_out, double *e_out, hipStream_t s)
{
    if (thermo) launch_force_t<Real, MULTI, true>(B, P, cur, mode, st, F_out, e_out, s);
    else launch_force_t<Real, MULTI, false>(B, P, cur, mode, st, F_out, e_out, s);
}

hipError_t launch_force(const Buffers &B, const Launch &P, int cur, Mode mode, bool thermo,
                        const StepArgs &st, double *F_out, double *e_out, hipStream_t s)
{
    parts(P, P.small_force, [&](const Launch &Q) {
        if (Q.precision == VBC_FP64) {
            if (Q.multi) launch_force_t<double, true>(B, Q, cur, mode, thermo, st, F_out, e_out, s);
            else launch_force_t<double, false>(B, Q, cur, mode, thermo, st, F_out, e_out, s);
        } else {
            if (Q.multi) launch_force_t<float, true>(B, Q, cur, mode, thermo, st, F_out, e_out, s);
            else launch_force_t<float, false>(B, Q, cur, mode, thermo, st, F_out, e_out, s);
        }
    });
    return hipGetLastError();
}

hipError_t launch_thermo_acc(const Buffers &B, const Launch &P, hipStream_t s)
{
    k_thermo_acc<<<P.nrep, 256, 0, s>>>(B, P.nrep);
    return hipGetLastError();
}

hipError_t launch_thermo_clear(const Buffers &B, int nrep, hipStream_t s)
{
    const int n = nrep * THERMO_WORDS;
    k_thermo_clear<<<blocks_for(n, 256), 256, 0, s>>>(B, n);
    return hipGetLastError();
}

hipError_t launch_reduce(const Buffers &B, const Launch &P, double *UW, hipStream_t s)
{
    k_reduce<<<P.nrep, 256, 0, s>>>(B, P.nrep, UW);
    return hipGetLastError();
}

hipError_t launch_kick_drift(const Buffers &B, const Launch &P, int cur, const StepArgs &st,
                             hipStream_t s)
{
    if (P.list == 0) launch_worklist(B, P, s);
    k_kick_drift<<<brick_grid(P.nb_launch), 256, 0, s>>>(B, P, cur, st);
    return hipGetLastError();
}

// Whether a replica can take its steps in one workgroup (k_resident): one type that counts
// every neighbour, no chains, and small enough for its LDS.
bool resident_can(const RepDev &R)
{
    if (R.ntypes != 1 || R.chain_len || !(R.mask[0] & 1u)) return false;
    if (R.n > RES_MAX_N) return false;
    for (int a = 0; a < 3; ++a)
        if (!(R.L[a] <= RES_MAX_L)) return false;
    return true;
}

hipError_t launch_resident(const Buffers &B, const Launch &P, int cur, int nsteps, int k0, int max_n,
                           const StepArgs &st, hipStream_t s)
{
    const int bs = std::max(128, (max_n + VBC_WAVE - 1) / VBC_WAVE * VBC_WAVE);  // a thread per particle
    const bool fp64 = P.precision == VBC_FP64;
    const size_t lds = fp64 ? ResLds<double>::bytes(max_n) : ResLds<float>::bytes(max_n);
    if (fp64) {
        if (st.acc) k_resident<double, true><<<P.nrep, bs, lds, s>>>(B, P, cur, nsteps, k0, max_n, st);
        else k_resident<double, false><<<P.nrep, bs, lds, s>>>(B, P, cur, nsteps, k0, max_n, st);
    } else {
        if (st.acc) k_resident<float, true><<<P.nrep, bs, lds, s>>>(B, P, cur, nsteps, k0, max_n, st);
        else k_resident<float, false><<<P.nrep, bs, lds, s>>>(B, P, cur, nsteps, k0, max_n, st);
    }
    return hipGetLastError();
}

hipError_t launch_observe(const Buffers &B, const Launch &P, int cur, int32_t *z_out,
                          int32_t *pen_out, int64_t *sums, hipStream_t s)
{
    if (sums) k_zero_i64<<<blocks_for(3 * P.nrep, 256), 256, 0, s>>>(sums, 3 * P.nrep);
    parts(P, P.small_bonds, [&](const Launch &Q) {
        const bool dense = Q.t_lo >= 0;
        const unsigned g = dense ? dense_grid(Q.nb_launch, staged_bytes(Q)) : brick_grid(Q.nb_launch);
        const int bs = dense ? std::min(Q.block, DENSE_BLOCK) : Q.block;
        auto k = dense ? (Q.multi ? k_observe_dense<true> : k_observe_dense<false>)
                       : (Q.multi ? k_observe<true> : k_observe<false>);
        k<<<g, bs, staged_bytes(Q), s>>>(B, Q, cur, z_out, pen_out, sums);
    });
    return hipGetLastError();
}

hipError_t launch_clusters(const Buffers &B, const Launch &P, int cur, const ClusterWork &W,
                           int32_t *label, int64_t *stats, int64_t *hist, int hist_len, hipStream_t s)
{
    const unsigned g = brick_grid(P.nb_launch);
    const int64_t nhist = 2 * (int64_t)P.nrep * hist_len;
    parts(P, P.small_bonds, [&](const Launch &Q) {
        const size_t lds = lds_bytes_bonds(Q);
        if (Q.t_lo >= 0) {
            auto k = Q.multi ? k_cc_local_dense<true> : k_cc_local_dense<false>;
            k<<<dense_grid(Q.nb_launch, lds), std::min(Q.block, DENSE_BLOCK), lds, s>>>(B, Q, cur, W);
        } else {
            auto k = Q.multi ? k_cc_local<true> : k_cc_local<false>;
            k<<<g, Q.block, lds, s>>>(B, Q, cur, W, stats, hist, nhist);
        }
    });
    k_cc_hook<<<g, 256, 0, s>>>(B, P, cur, W);
    k_cc_count<<<g, 256, 0, s>>>(B, P, W);
    const size_t lh = hist && hist_len <= CC_HIST ? (size_t)2 * hist_len * sizeof(uint32_t) : 0;
    k_cc_label<<<std::min<unsigned>(g, CC_GROUPS), 256, lh, s>>>(B, P, W, label, stats, hist, hist_len);
    return hipGetLastError();
}

hipError_t launch_bond_track(const Buffers &B, const Launch &P, int cur, const BondTrack &T, int reset,
                             int64_t *hist, int hist_len, int64_t bin_steps, int64_t *stats, hipStream_t s)
{
    if (reset && stats) k_zero_i64<<<blocks_for(5 * P.nrep, 256), 256, 0, s>>>(stats, 5 * P.nrep);
    if (reset && hist) k_zero_i64<<<blocks_for((int64_t)P.nrep * hist_len, 256), 256, 0, s>>>(hist, P.nrep * hist_len);
    parts(P, P.small_bonds, [&](const Launch &Q) {
        const bool dense = Q.t_lo >= 0;
        const unsigned g = dense ? dense_grid(Q.nb_launch, staged_bytes(Q)) : brick_grid(Q.nb_launch);
        const int bs = dense ? std::min(Q.block, DENSE_BLOCK) : Q.block;
        auto k = dense ? (Q.multi ? k_bond_track_dense<true> : k_bond_track_dense<false>)
                       : (Q.multi ? k_bond_track<true> : k_bond_track<false>);
        k<<<g, bs, staged_bytes(Q), s>>>(B, Q, cur, T, reset, hist, hist_len, bin_steps, stats);
    });
    return hipGetLastError();
}

hipError_t launch_export_nlist(const Buffers &B, const Launch &P, int rep, int nbrick,
                               int32_t *pairs, int64_t cap, int64_t *count, hipStream_t s)
{
    unsigned long long *c = (unsigned long long *)count;
    k_zero_u64<<<1, 1, 0, s>>>(c);
    if (nbrick > 0)
        k_export_nlist<<<nbrick, P.block, 0, s>>>(B, P, rep, pairs, cap, c);
    return hipGetLastError();
}

}  // namespace vbc
