// empp_dev.h -- device-side types and helpers shared by the HIP kernels of
// libempp.so.  gfx950 only; compiled with hipcc --offload-arch=gfx950.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace empp {

// CODATA 2018 (c, e, m_e exact or recommended; mu0 recommended).
constexpr double kC_LIGHT = 299792458.0;
constexpr double kMU0 = 1.25663706212e-6;

#ifndef EMPP_PAIR_BLOCK
#define EMPP_PAIR_BLOCK 512
#endif
constexpr int kBlock = EMPP_PAIR_BLOCK;  // threads per block of the mixed pair kernel and per-particle kernels
// Threads per block of the FP64 pair kernel: 1024 targets share each staged
// history tile (one block per CU at 128 registers per lane).
#ifndef EMPP_FP64_BLOCK
#define EMPP_FP64_BLOCK 1024
#endif
constexpr int kBlockFp64 = EMPP_FP64_BLOCK;

// Deepest supported history (slots): the pair kernel's LDS tile for it, one
// history of 32-byte records plus its light distances, fills a CU's 160 KiB.
constexpr int kMaxDepth = 4064;
constexpr int kMaxSplits = 1024;   // source chunks of one launch

// History layout in HBM (library-owned workspace):
//   ring_w[j * D + p] = {x, y, z, 0}     position of source j at physical slot p
//   vel: four planes of N D 16-byte records, record j * D + p of each
//     {vx, vy}, {vz, ax}, {ay, az}, {1/h, vz} velocity leaving that slot, the
//                                         acceleration (v_{p+1} - v_p)/h of the
//                                         segment that starts there and its
//                                         inverse length (0: newest)
//   T[p]                                  slot time
// Slot p holds logical slot "back" b (0 = newest) when p = (head - b) mod D.
// A source's positions are one contiguous 32*D-byte block, so a block
// of targets stages them into LDS with straight coalesced loads.

// The velocity ring in planes.  The pair kernels gather a lane's bracket
// record from L2 through the vector L1, which takes 37 cycles for a
// wavefront's 16-byte (or 8-byte) load from random places in 8 KiB, 25 in
// 2 KiB, 16.5 contiguous: three loads from dense planes instead of four from
// two 32-byte records (N = 65536, D = 512: 26.3 -> 25.7 ms, warm start 30.9 ->
// 28.3; mixed precision, which also takes the next slot's velocity and the
// inverse length, four loads as before).
struct VelRing {
    double2 *plane;  // plane k at plane + k n
    int64_t n;
    __device__ double3 v(int64_t q) const
    {
        const double2 a = plane[q];
        return make_double3(a.x, a.y, plane[n + q].x);
    }
    __device__ double inv_h(int64_t q) const { return plane[3 * n + q].x; }
    __device__ void set_v(int64_t q, double3 v, double ih) const
    {
        plane[q] = make_double2(v.x, v.y);
        plane[n + q].x = v.z;
        plane[3 * n + q] = make_double2(ih, v.z);
    }
    // acceleration of the segment at q that ends with velocity v2
    __device__ void set_a(int64_t q, double3 v1, double3 v2, double ih) const
    {
        plane[n + q].y = (v2.x - v1.x) * ih;
        plane[2 * n + q] = make_double2((v2.y - v1.y) * ih, (v2.z - v1.z) * ih);
    }
};

// Data of a source for the guessed bracket, in float: the slot
// b = d0.l + sqrt((d0.l)^2 + k |d0|^2), d0 = r - w_n the target's offset from
// the newest sample; {w_n - ref, k}, {l, -} with ref the sample of particle 0
// before the newest.  lines[2 j] from the chord, lines[2 (N + j)] from the
// newest velocity; made by the push for the next pass (and when a history is
// set): made in the pair kernel, one wavefront's work per tile, the pass took
// 23.9 ms instead of 23.6 at N = 65536, D = 512, and 29.1 instead of 28.4 at
// D = 1024.
struct GuessLine {
    float4 a, b;
};

// Along the chord from the newest to the oldest sample wo, Lo = c (t - T)
// there, the sign-test value is alpha b^2 - 2 alpha b (d0.l) - |d0|^2, exactly
// so on a straight path: alpha = (Lo^2 - |D|^2) / (D - 1)^2, l = D / ((D - 1)
// alpha), k = 1 / alpha.
__device__ inline GuessLine chord_line(double3 wn, double3 wo, double Lo, int depth, double3 ref)
{
    const double dx = wn.x - wo.x, dy = wn.y - wo.y, dz = wn.z - wo.z, n = (double)(depth - 1);
    const double ia = n * n / (Lo * Lo - (dx * dx + dy * dy + dz * dz));
    const double f = ia / n;
    return GuessLine{make_float4((float)(wn.x - ref.x), (float)(wn.y - ref.y), (float)(wn.z - ref.z), (float)ia),
                     make_float4((float)(dx * f), (float)(dy * f), (float)(dz * f), 0.0f)};
}

// Straight-line look-back: with beta the newest velocity / c, the positive
// root of (1 - beta^2) s^2 - 2 (R.beta) s - R^2 = 0, in steps of c dt.
__device__ inline GuessLine straight_line(double3 wn, double3 vn, double dt, double3 ref)
{
    const double ic = 1.0 / kC_LIGHT;
    const double bx = vn.x * ic, by = vn.y * ic, bz = vn.z * ic;
    const double ig2 = 1.0 / (1.0 - (bx * bx + by * by + bz * bz));
    const double is = 1.0 / (kC_LIGHT * dt), f = ig2 * is;
    return GuessLine{make_float4((float)(wn.x - ref.x), (float)(wn.y - ref.y), (float)(wn.z - ref.z), (float)(f * is)),
                     make_float4((float)(bx * f), (float)(by * f), (float)(bz * f), 0.0f)};
}

struct PairParams {
    const double4 *ring_w;
    VelRing vel;
    const float4 *line;  // guess data of the mode, [N][2]
    const double *T;
    int64_t n_src;      // sources N
    int32_t D;
    int32_t head;       // physical index of the newest slot
    double t;           // present time (== T[head]; the pair kernels read T[head])
    double kq;          // Coulomb constant times source charge
    // targets: external points x[k * x_stride + a] (x != nullptr) or the particles'
    // newest positions (x == nullptr, then target a is particle a and the
    // pair (a, a) is skipped).
    const double *x;
    int64_t x_stride;
    const int64_t *self_index;  // external mode only, may be null
    int64_t a_base;             // the launch's first target in its call (errors name the call's)
    const int32_t *order;       // step mode: target slot -> particle (spatial order), may be null
    int64_t m;
    int64_t src_per_split;
    int32_t nsplit;
    int32_t run_len;            // mixed precision: sources after which a plain partial is merged (as well)
    int32_t tile;               // sources staged per LDS tile
    int32_t sg_log2;            // log2 of the wavefronts that share a target's sources
    double *part;               // [nsplit][12][m] partial (sum, comp)
    int32_t *kstar;             // [m][N] or null
    unsigned long long *err;    // [2]: first failing pair, status bits
    unsigned long long *counters;  // [5] pairs, before, probes, rescues, fallbacks
    // surrogate / guided search
    int32_t guess;
    double dt;
    const float *G;             // surrogate guesses G[source * g_groups + (a >> g_shift)]
    int64_t g_groups;           // target groups of the launch
    int32_t g_shift;            // guess mode 1: log2 of the targets per guess; mode 3: 0 (one per pair)
    // guess modes: 0 bisection, 1 surrogate correction per target group,
    // 2 straight-line look-back, 3 surrogate delay per pair, 4/5 warm start
    // warm start (step mode): bracket of every (source j, target slot a)
    // from the previous step at kc[j * m + a]: back offset b* (1..D-1) or
    // kBracketBefore.  Read by the warm-start search (kc_cold = 0) and
    // written by it; on a cold step the bisection fills it.
    uint16_t *kc;
    int32_t kc_cold;
    // adaptive step (Sec. 2.4): min |eta| and max |v_i - v_j(t_r)|^2 over
    // the pairs with |eta| >= eta_allow, folded into ad[0] (atomicMin) and
    // ad[1] (atomicMax) as double bit patterns; null when the step is fixed
    unsigned long long *ad;
    double eta_allow;
    // reconstruction inside the bracket: 0 = local linear (Eq. linear, the
    // method), 1 = midpoint values (Eq. mid, accuracy ablation)
    int32_t recon;
};

constexpr uint16_t kBracketBefore = 0xFFFF;

struct PushParams {
    double4 *ring_w;
    VelRing vel;
    GuessLine *lines;   // [2][N]
    double dt_cfg;      // the configured step (straight-line guesses)
    double *T;
    double *u;          // [3][N]
    double *E;          // [3][N] self-field of the step (written by the merge)
    double *B;
    const double *part; // [nsplit][12][N], in the pair launch's target order
    const int32_t *order; // target order -> particle index
    int32_t nsplit;
    int64_t N;
    int32_t D;
    int32_t head;       // newest physical slot before the push
    double dt;
    double t_now;       // time of the newest slot before the push
    double t_next;      // time of the new slot
    double eps;         // q dt / (2 m)
    int32_t ext_field;
    double dip_k;       // b0 * re^3: (mu0/4pi) M0 for the centred dipole
    // adaptive step: ad = this step's {eta_min, v_max^2} slot (null: fixed
    // dt); the step is c_dt eta_min / v_max clamped to [dt_min, dt_max],
    // t_now is read from T[head], and ad_next/dt_out are reset/written
    unsigned long long *ad;
    unsigned long long *ad_next;
    double *dt_out;
    double c_dt, dt_min, dt_max;
    double q, m;
};

// Block of a pair-kernel launch -> (target block bx, source chunk split).
// The grid is one-dimensional, nbx * nsplit blocks.  Workgroups go to the 8
// XCDs round-robin by linear index.  A chunk's blocks go to one XCD, so that
// the target blocks that stage its histories run there together and share its
// L2: with a multiple of 8 chunks the XCDs take chunk after chunk in turn
// (N = 65536, D = 512, 128 chunks: 23.87 ms; an eighth of the range each
// 24.17), else each takes an eighth of the blocks in chunk order (N = 3000, 42
// chunks of 6 target blocks: 77 us; any order 96, as some XCDs got 36 blocks
// for their 32 CUs).
__device__ inline void pair_block_coords(int nbx, int nsplit, int &bx, int &split)
{
    const int L = blockIdx.x, xcd = L & 7;
    int k = L >> 3;
    if ((nsplit & 7) == 0) {
        const int round = k / nbx;
        split = xcd + 8 * round;
        bx = k - round * nbx;
    } else {
        const int total = nbx * nsplit;
        k += xcd * (total >> 3) + min(xcd, total & 7);
        split = k / nbx;
        bx = k - split * nbx;
    }
}

// Stage II (transport after the handoff): positions pos[i] = {x, y, z, 0},
// proper velocities u[3][N]; the step is
// dt = min(dt_max, gyro_k * min_i gamma_i / |B(y_i)|), the minimum being
// kept in three rotating slots of double bit patterns (positive doubles
// order like their unsigned bit patterns): step k reads slot k % 3, builds
// slot (k + 1) % 3 with atomicMin and clears slot (k + 2) % 3.
struct TransportParams {
    double4 *pos;
    double *u;
    int64_t N;
    double q_over_2m;
    double dip_k;
    int32_t ext_field;
    double dt_max;
    double gyro_k;
    unsigned long long *key;  // [3]
    double *t;                // [1] present time
    int64_t step;
    // several steps in one launch: the blocks' minima of even and odd steps
    // [2][kTransportBlocks], the steps that went through them before, and the
    // word that a wait that gave up sets
    unsigned long long *slots;
    int64_t nsteps, sync_step;
    unsigned long long *fail;
    unsigned polls;  // a wait gives up after
    int32_t queued;  // behind another launch of the call, which may have given up
};
constexpr int kTransportBlocks = 256;
// Polls after which a wait between the blocks of a cooperative launch gives up,
// some 15 s: a block may have to wait for another stream's pair pass to leave its CU.
constexpr unsigned kWaitPolls = 1u << 24;

constexpr unsigned long long kPosInfBits = 0x7FF0000000000000ull;

// Error word: err[0] = (target << 32 | source) of the lowest failing pair
// (atomicMin), err[1] = OR of status bits.
constexpr unsigned long long kErrCoincident = 1ull;
constexpr unsigned long long kErrDiscriminant = 2ull;

__device__ inline void report_error(unsigned long long *err, int64_t a, int64_t j,
                                    unsigned long long bit)
{
    unsigned long long key = ((unsigned long long)(uint32_t)a << 32) | (uint32_t)j;
    atomicMin(&err[0], key);
    atomicOr(&err[1], bit);
}

// Reciprocal of a positive normal double: hardware estimate plus one
// Newton-Raphson step, which squares the estimate's relative error (about
// 2^-26) to the last bits of the mantissa.
__device__ inline double rcp64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}

// Neumaier accumulation of x into (s, c).
__device__ inline void neumaier(double &s, double &c, double x)
{
    double t = s + x;
    double big = fabs(s) >= fabs(x) ? s : x;
    double small = fabs(s) >= fabs(x) ? x : s;
    c += (big - t) + small;
    s = t;
}

}  // namespace empp
