// pair_kernel.h -- the all-pairs Lienard-Wiechert pass shared by the FP64
// and the mixed-precision pair kernels (Secs. 2.1-2.2 of arXiv 2605.05543).
//
// One thread owns one target.  A block of kBlockFp64 (1024) threads walks its
// chunk of sources in staged tiles of up to 16 sources: the tile's
// positions, with the square of each slot's light distance, are staged once
// into LDS, double-buffered behind one barrier per tile, and
// every target of the block then searches them, so each history byte read
// from L2/HBM serves 1024 targets.  Source by source, a guessed bracket is
// confirmed by the two samples that define it, the two velocity records are
// fetched and the pair field evaluated.  Targets are visited in a spatial
// (Morton) order so that the lanes of a wavefront probe nearby history
// slots.  Sums are kept per
// target in registers: a plain partial merged into a compensated total
// (Neumaier in FP64 every 32 sources, Knuth's two-sum in FP32 every 8);
// source chunks write (sum, compensation) partials, in the launch's target
// order, that the merge kernel adds in a fixed order (and maps to particle
// indices), so results do not depend on scheduling.
//
// Every sign test is the FP64 test of the paper's bracket, in both
// precisions: the bracket index is bit-identical across paths and search
// modes.  MIX selects the mixed-precision field evaluation (root,
// reconstruction and LW terms in FP32 around FP64 coefficients).
//
// What bounds it: vector issue (132 instructions per wavefront and pair at
// N = 65536, D = 512, the VALU busy 67 % of the time), the vector L1 (three
// 16-byte gathers of a lane's segment and the tile's loads) and the latency
// of a pair's chain (LDS reads of the confirming samples, the gather from L2,
// about 70 dependent FP64 instructions) on four wavefronts per SIMD.
// The history is searched by guess and confirmation in every mode, the
// bisection's too: the unrolled bisection's ten probes of 32 bytes kept the
// LDS busy for nine tenths of the pass (33.1 ms; guessed along the chord to
// the oldest sample, with each segment's acceleration kept with the history
// and the root's square root reused as eta . v', 26.1 ms).  Positions are
// staged as they are and tested as L^2 - |r - w|^2, velocities gathered from
// planes and the guess's data made by the push: 23.7 ms (26.1 before), warm
// start 26.8 (30.8), mixed straight-line 25.9 (27.4), D = 1024 28.5 (31.0).  A
// curving history that bisects pays nine instructions a probe instead of six,
// which the leaner field algebra repays in FP64 and mixed precision does not have
// (a turn of 1.5 rad over the history, with the unrolled bisection and now: FP64,
// N = 16384 2.61 and 2.39 ms, N = 65536 34.9 and 34.1; mixed 2.57 and 2.41, 34.1 and
// 35.1).
#pragma once

#include "pair_common.h"

#include <algorithm>
#include <type_traits>

namespace empp {

// Records per half-array of a double-buffered LDS tile: 32 KiB of the
// records' first 16-byte halves, then 32 KiB of their second halves.
constexpr int kHalfRecs = 2048;
constexpr int kMaxTile = 16;  // sources per staged tile at most
constexpr int kWaves = kBlockFp64 / 64;

// Tiles are double-buffered (staging overlapped with the search) while a
// history fits in kHalfRecs records; deeper histories use one buffer sized
// to one history (kMaxDepth slots fill the CU's 160 KiB with the slot light
// distances and the per-source data).
constexpr bool pair_two_buffers(int D) { return D <= kHalfRecs; }

// Sources per staged LDS tile: as many as fill a buffer (one barrier per
// staged tile).
constexpr int pair_staged_tile(int D) { return D <= kHalfRecs ? std::min(kMaxTile, kHalfRecs / D) : 1; }

// The tile buffers, the light distance of every slot, with two buffers also
// the byte offsets of its ring row entry and of the next newer one, then
// per buffer and source the guess's data, and per buffer, wavefront and source
// the surrogate's correction.
constexpr size_t pair_lds_bytes(int D)
{
    const bool two = pair_two_buffers(D);
    const size_t ts = (size_t)pair_staged_tile(D);
    return (two ? 4 * (size_t)kHalfRecs : 2 * (size_t)D) * sizeof(double2) + (size_t)((D + 1) & ~1) * sizeof(double) +
           (two ? (size_t)((D + 3) & ~3) * sizeof(uint32_t) : 0) + 2 * ts * 2 * sizeof(float4) +
           2 * kWaves * ts * sizeof(float);
}

static_assert(pair_lds_bytes(kMaxDepth) <= 160 * 1024,
              "the deepest history's tile, light distances and per-source data fit a CU's LDS");
static_assert(pair_lds_bytes(kHalfRecs) <= 160 * 1024, "the deepest double-buffered tiles fit with the slot table");
// its 16-bit byte offsets of 16-byte ring entries
static_assert((kHalfRecs - 1) * 16 < 65536, "slot table offsets fit 16 bits");

namespace {

// sqrt of a positive normal double from the hardware reciprocal square
// root and one Newton correction of x y: the estimate's relative error
// (about 2^-26) is squared, to within a few units in the last place (no
// special-value handling, x > 0 here).  The root enters the pair's field
// through c (t_r - t_1), at most one step of light travel, against
// |eta| of millimetres, so this is far below the field tolerance.
__device__ inline double sqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double sq = x * y;
    const double r = __builtin_fma(-sq, sq, x);
    return __builtin_fma(r, 0.5 * y, sq);
}

// Retarded root, reconstruction and LW field of one pair (Eqs. dt,
// linear, linear2, LW_E, LW_B) without the factor kq, which the sums take at
// the end.  d = r - w_1, the target's offset from the bracket's older sample,
// C0 = L1^2 - |d|^2 (the sign test's value there), L1 = c (t - t_1); v1 the
// velocity and a the acceleration (zero out of history) of the bracket's
// segment.  E, and h = eta_hat / c for B = h x E.  Returns
// false on a numerical failure (negative discriminant, eta <= 0), which
// reaches the last test as a NaN.
// The root sq of the discriminant is eta . v' at v_1, C2 dt being
// -(C1h + sq): with v_r = v_1 + a dt, eta . v' = sq - dt (eta . a), one
// instruction and no difference of large terms (rounding of a pair's field
// at 5 MeV 1.6e-14 rms, against 7.5e-14 from c |eta| - eta . v_r).
// MID and mid: Eq. (mid) with the bracket's other velocity v2 and dw =
// w_2 - w_1 (the accuracy ablation).
template <bool MID>
__device__ __forceinline__ bool lw_pair(double3 d, double C0, double L1, double3 v1, double3 a, double3 &E, double3 &h,
                                        double &en, double3 &vr, bool mid, double3 v2, double3 dw)
{
    const double c = kC_LIGHT;
    const double c2 = c * c;
    // C2 dt^2 + 2 C1h dt + C0 = 0 (Eq. dt with C1 = 2 C1h); the physical
    // root -(C1h + sqrt(C1h^2 - C2 C0))/C2 in Vieta's form.
    const double C2 = __builtin_fma(-v1.x, v1.x, __builtin_fma(-v1.y, v1.y, __builtin_fma(-v1.z, v1.z, c2)));
    const double C1h = __builtin_fma(d.x, v1.x, __builtin_fma(d.y, v1.y, __builtin_fma(d.z, v1.z, -c * L1)));
    const double disc = __builtin_fma(C1h, C1h, -(C2 * C0));
    const double sq = sqrt_pos(disc);
    const double dtr = C0 * rcp64(sq - C1h);
    // reconstruction: v = v1 + a dt, eta = r - w1 - v1 dt, |eta| = c (t - t_r)
    vr.x = __builtin_fma(a.x, dtr, v1.x);
    vr.y = __builtin_fma(a.y, dtr, v1.y);
    vr.z = __builtin_fma(a.z, dtr, v1.z);
    double ex = __builtin_fma(-v1.x, dtr, d.x), ey = __builtin_fma(-v1.y, dtr, d.y), ez = __builtin_fma(-v1.z, dtr, d.z);
    en = __builtin_fma(-c, dtr, L1);
    if (MID && mid) {
        // Eq. (mid): the bracket ends' means, eta = r - (w_1 + w_2)/2
        ex = d.x - 0.5 * dw.x;
        ey = d.y - 0.5 * dw.y;
        ez = d.z - 0.5 * dw.z;
        en = sqrt(ex * ex + ey * ey + ez * ez);
        vr = make_double3(0.5 * (v1.x + v2.x), 0.5 * (v1.y + v2.y), 0.5 * (v1.z + v2.z));
    }
    const double ea = __builtin_fma(ex, a.x, __builtin_fma(ey, a.y, ez * a.z));
    double ev = __builtin_fma(-dtr, ea, sq);  // eta . v'
    if (MID && mid)
        ev = c * en - (ex * vr.x + ey * vr.y + ez * vr.z);
    const double inv = rcp64(en * ev);
    const double ien = ev * inv, iev = en * inv;
    const double icn = ien * (1.0 / c);
    h.x = ex * icn;
    h.y = ey * icn;
    h.z = ez * icn;  // eta_hat / c
    const double px = __builtin_fma(c2, h.x, -vr.x), py = __builtin_fma(c2, h.y, -vr.y),
                 pz = __builtin_fma(c2, h.z, -vr.z);  // v'
    // (c^2 - v^2) v' + eta x (v' x a), the cross product expanded as
    // v' (eta . a) - a (eta . v'), over (eta . v')^3 / |eta|
    const double S = __builtin_fma(-vr.x, vr.x, __builtin_fma(-vr.y, vr.y, __builtin_fma(-vr.z, vr.z, c2 + ea)));
    const double k2 = (en * iev) * iev;
    const double k1 = (k2 * iev) * S;
    E.x = __builtin_fma(k1, px, -(k2 * a.x));
    E.y = __builtin_fma(k1, py, -(k2 * a.y));
    E.z = __builtin_fma(k1, pz, -(k2 * a.z));
    return (en > 0.0) & (ev > 0.0);
}

// x, or a value below 1e-300 if z: one select of the high word.
__device__ __forceinline__ double zero_if(bool z, double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t hi = z ? 0u : (uint32_t)(u >> 32);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | (uint32_t)u));
}

// Knuth two-sum: s + e == a + b exactly.
__device__ inline void two_sum(float &s, float &e, float x)
{
    float t = s + x;
    float bb = t - s;
    float err = (s - (t - bb)) + (x - bb);
    s = t;
    e += err;
}

struct MixedPair {
    double3 d;           // r - w_1, the target's offset from the bracket's older sample
    double4 v1, v2;      // FP64 velocity records of the bracket ends
};

// Root, reconstruction and LW field from FP64 inputs.  The coefficients of
// the quadratic, the velocity at the root and u = eta - |eta| v/c (which
// carries the cancellation 1 - eta_hat.beta of nearly forward pairs) are
// formed in FP64; the root, the normalisations and the LW products in FP32.
// Since eta = d - v_1 dt and |eta| = L1 - c dt, u = d - (L1/c) v_r +
// dt (v_r - v_1): the FP64 offset d enters directly and no large terms
// cancel in FP32.  Writes E, B into f[0..5]; rescued = the FP32 root failed
// its residual test and was recomputed in FP64.  Returns false on a
// numerical failure.
// The FP64 re-solve is the same arithmetic in every search mode (refined
// hardware square root and reciprocal), so fields do not depend on the
// search.  BRANCH_RESCUE only decides how it is compiled: a branch around
// it (an empty volatile asm cannot be speculated), or left to the compiler,
// which may evaluate it for every pair and select (measured: a branch pays
// in the bisection pass, 43.2 -> 36.7 ms at N = 65536, D = 512; the guided
// passes are 1-2 % faster with the compiler's choice).
template <bool BRANCH_RESCUE>
__device__ __forceinline__ bool lw_pair_mixed(double L1d, MixedPair q, bool before,
                                              float kq, float f[6], bool &rescued)
{
    const double c = kC_LIGHT;
    const double ic = 1.0 / kC_LIGHT;
    const float cf = (float)kC_LIGHT;
    // FP64: offset to the bracket sample and the quadratic's coefficients
    double dxd = q.d.x, dyd = q.d.y, dzd = q.d.z;
    double C0d = L1d * L1d - (dxd * dxd + dyd * dyd + dzd * dzd);
    double C2d = c * c - (q.v1.x * q.v1.x + q.v1.y * q.v1.y + q.v1.z * q.v1.z);
    double C1hd = (dxd * q.v1.x + dyd * q.v1.y + dzd * q.v1.z) - c * L1d;
    double discd = C1hd * C1hd - C2d * C0d;
    bool ok = discd > 0.0;
    // FP32 root in the form without cancellation, checked by its residual
    float C0 = (float)C0d, C1h = (float)C1hd, C2 = (float)C2d;
    float sq = __builtin_amdgcn_sqrtf(ok ? (float)discd : 1.0f);
    float dtr = C1h <= 0.0f ? C0 * __builtin_amdgcn_rcpf(sq - C1h) : -(C1h + sq) * __builtin_amdgcn_rcpf(C2);
    float res = __builtin_fmaf(__builtin_fmaf(C2, dtr, 2.0f * C1h), dtr, C0);
    float tol = 8.0f * 5.9604645e-8f * (fabsf(C2) * dtr * dtr + 2.0f * fabsf(C1h * dtr) + fabsf(C0));
    rescued = !(fabsf(res) <= tol);
    if (rescued) {
        if constexpr (BRANCH_RESCUE)
            asm volatile("");
        // refined hardware estimates; both divisors are positive
        double sqd = sqrt_pos(ok ? discd : 1.0);
        double rd = C1hd <= 0.0 ? C0d * rcp64(sqd - C1hd) : -(C1hd + sqd) * rcp64(C2d);
        dtr = (float)rd;
    }
    // FP64: velocity at the root and u = d - (L1/c) v_r + dt (v_r - v_1)
    double inv_hd = before ? 0.0 : q.v1.w;
    double dtd = (double)dtr;
    double gxd = q.v2.x - q.v1.x, gyd = q.v2.y - q.v1.y, gzd = q.v2.z - q.v1.z;
    double dfd = dtd * inv_hd;
    double vrxd = q.v1.x + gxd * dfd, vryd = q.v1.y + gyd * dfd, vrzd = q.v1.z + gzd * dfd;
    double Lc = L1d * ic, tg = dtd * dfd;
    double uxd = dxd - Lc * vrxd + tg * gxd, uyd = dyd - Lc * vryd + tg * gyd, uzd = dzd - Lc * vrzd + tg * gzd;
    // FP32 from here
    float dx = (float)dxd, dy = (float)dyd, dz = (float)dzd;
    float vx = (float)q.v1.x, vy = (float)q.v1.y, vz = (float)q.v1.z;
    float inv_h = (float)inv_hd;
    float gx = (float)gxd, gy = (float)gyd, gz = (float)gzd;
    float ax = gx * inv_h, ay = gy * inv_h, az = gz * inv_h;  // zero out of history
    float df = (float)dfd;
    float ux = (float)uxd, uy = (float)uyd, uz = (float)uzd;
    float ex = dx - vx * dtr, ey = dy - vy * dtr, ez = dz - vz * dtr;  // eta
    float en = (float)L1d - cf * dtr;                                 // |eta| = c (t - t_r)
    ok = ok && en > 0.0f;
    float ien = __builtin_amdgcn_rcpf(en);
    float px = cf * ux * ien, py = cf * uy * ien, pz = cf * uz * ien;  // v' = c eta_hat - v_r
    float ev = ex * px + ey * py + ez * pz;                           // eta . v' = c |eta| kappa
    ok = ok && ev > 0.0f;
    float iev = __builtin_amdgcn_rcpf(ev);
    const float icn = ien * (float)ic;
    float hx = ex * icn, hy = ey * icn, hz = ez * icn;  // eta_hat / c
    // c^2 - |v_r|^2 from the FP64 value at v_1 plus the small correction
    float cv = C2 - df * (2.0f * (vx * gx + vy * gy + vz * gz) + df * (gx * gx + gy * gy + gz * gz));
    // eta x (v' x a) = v' (eta . a) - a (eta . v')
    float ea = ex * ax + ey * ay + ez * az;
    float pref = kq * en * (iev * iev * iev);
    float k1 = pref * (cv + ea), k2 = pref * ev;
    float Ex = k1 * px - k2 * ax;
    float Ey = k1 * py - k2 * ay;
    float Ez = k1 * pz - k2 * az;
    f[0] = Ex;
    f[1] = Ey;
    f[2] = Ez;
    // B = eta_hat x E / c
    f[3] = hy * Ez - hz * Ey;
    f[4] = hz * Ex - hx * Ez;
    f[5] = hx * Ey - hy * Ex;
    return ok;
}

}  // namespace

// True if pred holds in any active lane (a compare of the mask).
__device__ __forceinline__ bool any_lane(bool pred) { return __builtin_amdgcn_ballot_w64(pred) != 0; }

// A wavefront that misses its guess in kMissRun sources in a row bisects the
// next kBisectRun sources before it guesses again, and twice as many each time
// that guess misses too, up to kBisectMost (a curving history, N = 65536, D = 512,
// pair kernel: 35.6 ms with runs of 30, 35.0 so, 34.9 from 62 to 248; N = 16384 with
// one length, 30, 62 and 126: steps of 2.48, 2.46 and 2.45).  A warm start, whose
// guesses miss only now and then, keeps to the short run (36.0 ms, 36.5).
constexpr int kMissRun = 3, kBisectRun = 30, kBisectMost = 240;

// DB: double-buffered tiles (D <= kHalfRecs).
template <bool MIX, bool KSTAR, bool COUNT, int GUESS, bool ADAPT, bool MID, bool DB>
__device__ __forceinline__ void pair_body(const PairParams &p)
{
    static_assert(!MIX || (!ADAPT && !MID && GUESS <= 3), "mixed precision: fixed step, no warm start");
    extern __shared__ double4 lds[];
    typedef double dv2 __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(3))) dv2 *lds_dv2;
    // LDS address of the dynamic buffer (32-bit, for offset arithmetic)
    const uint32_t lds_base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)lds;
    const int D = p.D;
    const int tid = threadIdx.x, lane = tid & 63;
    // A block's wavefronts: 16 >> sg_log2 groups of 64 targets, each served
    // by 1 << sg_log2 wavefronts that take the tile's sources in turn.
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int SG = 1 << p.sg_log2, tw_log2 = 4 - p.sg_log2;
    const int sg = wave >> tw_log2, tw = wave & ((1 << tw_log2) - 1);
    const int targets = 64 << tw_log2;
    const int nbx = (int)((p.m + targets - 1) / targets);
    int bxi, split;
    pair_block_coords(nbx, p.nsplit, bxi, split);
    const int64_t a0 = (int64_t)bxi * targets + tw * 64;
    const int64_t a = a0 + lane;
    // The lanes beyond the last target go along with it and write nothing, so that
    // a wavefront takes its branches as one and its search's state stays scalar
    // (N = 65536, D = 512: 23.9 -> 23.7 ms; the adaptive kernels spilled 4 registers).
    const bool active = a < p.m, wave_on = a0 < p.m;
    const int64_t ac = active ? a : p.m - 1;
    // sources j0 .. j0 + nj - 1
    const int64_t j0 = (int64_t)split * p.src_per_split;
    const int nj = (int)max((int64_t)0, min(p.n_src - j0, p.src_per_split));

    double rx = 0, ry = 0, rz = 0;
    double3 vt = make_double3(0.0, 0.0, 0.0);  // target's present velocity (adaptive step)
    double eta_min = __longlong_as_double((long long)kPosInfBits), dv2_max = 0.0;
    int32_t self = -1;  // source left out (sources number at most 2^31)
    if (wave_on) {
        if (p.x) {
            rx = p.x[ac];
            ry = p.x[p.x_stride + ac];
            rz = p.x[2 * p.x_stride + ac];
            // (an index that names no source leaves none out)
            const int64_t out = p.self_index ? p.self_index[ac] : -1;
            self = out >= 0 && out < p.n_src ? (int32_t)out : -1;
        } else {
            const int64_t tgt = p.order ? (int64_t)p.order[ac] : ac;
            double4 w = p.ring_w[tgt * D + p.head];
            rx = w.x;
            ry = w.y;
            rz = w.z;
            self = (int32_t)tgt;
            if (ADAPT) {
                vt = p.vel.v(tgt * D + p.head);
            }
        }
    }
    // offset from the sample of particle 0 before the newest, in float, for
    // the guesses (GuessLine)
    const double4 ref = p.ring_w[p.head == 0 ? D - 1 : p.head - 1];
    const float rfx = (float)(rx - ref.x), rfy = (float)(ry - ref.y), rfz = (float)(rz - ref.z);
    // field sums: FP64 with Neumaier compensation, or FP32 with two-sum
    using Real = std::conditional_t<MIX, float, double>;
    Real sum[6] = {0, 0, 0, 0, 0, 0}, comp[6] = {0, 0, 0, 0, 0, 0};
    Real acc[6] = {0, 0, 0, 0, 0, 0};
    constexpr int kPlainRun = MIX ? 8 : 32;  // sources per plain partial
    // sources left in the plain partial, and after it to the end of the run
    int left = kPlainRun, run_left = 0;
    auto next_run = [&]() {
        left = kPlainRun;
        if constexpr (MIX) {
            run_left = run_left == 0 ? p.run_len : run_left;
            left = min(kPlainRun, run_left);
            run_left -= left;
        }
    };
    if constexpr (MIX)
        run_left = p.run_len - (int)(j0 % p.run_len);
    next_run();
    int probes = 0, nbefore = 0, npairs = 0, nfall = 0, nresc = 0;
    // first (lowest) source of a failing pair; sources number below 2^31
    int32_t fail_j = INT32_MAX;
    const float inv_cdt = (float)(1.0 / (kC_LIGHT * p.dt));
    const int64_t grp_index = ac >> p.g_shift;  // surrogate group of this target

    // LDS: the tile buffers, then the light distance L(b) = c (t - T_b) of
    // every logical slot (shared by all sources).  A buffer holds its TS * D
    // records {x, y, z, L^2} as two arrays of 16-byte halves, {x, y} then
    // {z, L^2}, hrec halves apart: lanes that probe different slots then
    // spread over twice as many LDS bank groups as with 32-byte records.
    // With two buffers the distance is the fixed kHalfRecs, so a probe's
    // reads share one address (the others at immediate offsets).
    constexpr int nbuf = DB ? 2 : 1;
    const int TS = DB ? p.tile : 1;
    const int hrec = DB ? kHalfRecs : D;
    const uint32_t hbytes = DB ? (uint32_t)(kHalfRecs * sizeof(double2)) : (uint32_t)D * (uint32_t)sizeof(double2);
    double2 *const halves = reinterpret_cast<double2 *>(lds);
    double *Ls = reinterpret_cast<double *>(halves + nbuf * 2 * hrec);
    // slot table (two buffers): for back offset b, the byte offset in a plane's
    // row of physical slot (head - b) mod D and, above 16 bits, of the next
    // newer slot's (the bracket's two velocity records)
    uint32_t *slot_off = reinterpret_cast<uint32_t *>(Ls + ((D + 1) & ~1));
    float4 *line = reinterpret_cast<float4 *>(slot_off + (DB ? ((D + 3) & ~3) : 0));  // [buffer][source][2]
    float *gcorr = reinterpret_cast<float *>(line + 2 * TS * 2);  // [buffer][wavefront][source]
    // The guess's data of a tile's sources and the surrogate's corrections
    // (guess mode 1, for groups of 64 or more targets: whole wavefronts), one
    // value a thread, are loaded ahead like its positions.
    constexpr bool kChord = GUESS == 0 || GUESS == 5;
    float line_pf = 0.0f;
    const int gc_w = tid / TS, gc_s = tid - gc_w * TS;
    const int64_t gc_a = (int64_t)bxi * targets + (gc_w & ((1 << tw_log2) - 1)) * 64;
    float gc_pf = 0.0f;
    auto load_line = [&](int64_t jt, int ns) {
        if (tid < 8 * ns)
            line_pf = reinterpret_cast<const float *>(p.line + 2 * jt)[tid];
        if (GUESS == 1 && tid < kWaves * TS && gc_s < ns && gc_a < p.m)
            gc_pf = p.G[(jt + gc_s) * p.g_groups + (gc_a >> p.g_shift)];
    };
    // the present time is the newest slot's (the clock lives in T)
    const double tnow = p.T[p.head];
    for (int b = tid; b < D; b += kBlockFp64) {
        int ph = p.head - b;
        ph += ph < 0 ? D : 0;
        Ls[b] = kC_LIGHT * (tnow - p.T[ph]);
        if constexpr (DB) {
            const int ph2 = ph + 1 == D ? 0 : ph + 1;  // back offset b - 1 (read for b >= 1)
            slot_off[b] = (uint32_t)ph * (uint32_t)sizeof(double2) | (uint32_t)ph2 * (uint32_t)sizeof(double2) << 16;
        }
    }
    // Record q of a tile: source q / D (q < TS D), slot q % D.  A thread's
    // records, q = tid + 1024 k, keep their source and slot in every tile: a
    // load is a uniform row base plus a fixed 32-bit offset.  Positions are
    // prefetched into registers one tile ahead (the first two of each thread:
    // a whole tile with two buffers), so the latency overlaps the previous
    // tile's work; deeper histories load the rest in place.  Records {-2 D,
    // L^2 - |D|^2} (D from the newest sample) save three instructions per
    // probe but are computed here: 25.7 ms instead of 23.9 at N = 65536,
    // D = 512, 30.4 instead of 29.1 at D = 1024.
    auto src_of = [&](int q) { return DB ? q / D : 0; };
    auto pos_off = [&](int q) {
        const int s = src_of(q);
        int ph = p.head - (q - s * D);
        ph += ph < 0 ? D : 0;
        return (uint32_t)(s * D + ph) * (uint32_t)sizeof(double4);
    };
    const int qa = min(tid, TS * D - 1), qb = min(tid + kBlockFp64, TS * D - 1);
    const uint32_t off_a = pos_off(qa), off_b = pos_off(qb);
    const int ba = qa - src_of(qa) * D, bb = qb - src_of(qb) * D;
    auto fetch = [&](int64_t jt, int nrec, int q, uint32_t off, double3 &w) {
        if (q < nrec)
            w = *reinterpret_cast<const double3 *>(reinterpret_cast<const char *>(p.ring_w + jt * D) + off);
    };
    auto put = [&](int bi, int nrec, int q, const double3 &w, int b) {
        if (q < nrec) {
            const double L = Ls[b];
            double2 *xy = halves + bi * 2 * hrec + q;
            xy[0] = make_double2(w.x, w.y);
            xy[hrec] = make_double2(w.z, L * L);
        }
    };
    // Tile jt of ns sources into buffer bi, from the prefetched positions.
    auto stage = [&](int bi, int64_t jt, int ns, const double3 &w0, const double3 &w1) {
        if (tid < 8 * ns)
            reinterpret_cast<float *>(line + bi * TS * 2)[tid] = line_pf;
        if (GUESS == 1 && tid < kWaves * TS && gc_s < ns)
            gcorr[(bi * kWaves + gc_w) * TS + gc_s] = gc_pf;
        const int nrec = ns * D;
        put(bi, nrec, tid, w0, ba);
        put(bi, nrec, tid + kBlockFp64, w1, bb);
        if constexpr (!DB)
            for (int q = tid + 2 * kBlockFp64; q < nrec; q += kBlockFp64) {
                double3 w;
                fetch(jt, nrec, q, pos_off(q), w);
                put(bi, nrec, q, w, q);
            }
    };
    auto tile_size = [&](int i) { return min(nj - i, TS); };
    double3 pf0, pf1;
    auto prefetch = [&](int i) {
        const int ns = tile_size(i);
        fetch(j0 + i, ns * D, tid, off_a, pf0);
        fetch(j0 + i, ns * D, tid + kBlockFp64, off_b, pf1);
        load_line(j0 + i, ns);
    };
    // Two buffers: tile i + 1 is written while tile i is searched, and one
    // barrier per tile both publishes tile i + 1 and retires tile i's
    // buffer for tile i + 2.  One buffer (deep histories): stage, then
    // search, with a barrier on either side.
    if (nj > 0) {
        prefetch(0);
        __syncthreads();  // light distances
        if (DB) {
            stage(0, j0, tile_size(0), pf0, pf1);
            if (TS < nj)
                prefetch(TS);
            __syncthreads();
        }
    }
    // previous-step bracket of this wavefront's next source (warm start)
    uint16_t knext = kBracketBefore;
    auto load_bracket = [&](int i) { knext = wave_on && i < nj ? p.kc[(j0 + i) * p.m + ac] : kBracketBefore; };
    if (GUESS == 4)
        load_bracket(sg);
    int miss_run = 0, bisect_left = 0, bisect_run = kBisectRun;
    int cb = 0;
    for (int i0 = 0; i0 < nj; i0 += TS) {
        if (DB) {
            if (i0 + TS < nj) {
                stage(cb ^ 1, j0 + i0 + TS, tile_size(i0 + TS), pf0, pf1);
                if (i0 + 2 * TS < nj)
                    prefetch(i0 + 2 * TS);
            }
        } else {
            __syncthreads();
            stage(0, j0 + i0, tile_size(i0), pf0, pf1);
            __syncthreads();
            if (i0 + TS < nj)
                prefetch(i0 + TS);
        }
        const int ns = tile_size(i0);
        for (int s = sg; s < ns; s += SG) {
            const int64_t jt = j0 + i0 + s;
            const int32_t j = (int32_t)jt;
            const uint16_t kcur = knext;
            if (GUESS == 4)
                load_bracket(s + SG < ns ? i0 + s + SG : i0 + TS + sg);
            if (wave_on) {
                if (KSTAR && active && j == self)
                    p.kstar[a * p.n_src + jt] = 0;
                // LDS byte address of the source's first record (its first half)
                const uint32_t src0 =
                    lds_base + (uint32_t)(cb * 2 * hrec + s * D) * (uint32_t)sizeof(double2);
                // the target's offset d = r - w_b from a sample and its
                // sign-test value L^2 - |d|^2
                auto value_at = [&](uint32_t o, double3 &d) {
                    const dv2 xy = *(lds_dv2)(uintptr_t)o, zl = *(lds_dv2)(uintptr_t)(o + hbytes);
                    d = make_double3(rx - xy.x, ry - xy.y, rz - zl.x);
                    return lightcone_value(d, zl.y);
                };
                auto addr = [&](int b) { return src0 + (uint32_t)b * (uint32_t)sizeof(double2); };
                auto test = [&](int b) {
                    double3 d;
                    return value_at(addr(b), d) > 0.0;
                };

                // the guessed slot
                float k_slot;  // 1 / curvature of the sign-test value in the slot
                auto guess_of = [&]() -> float {
                    const float4 l0 = line[(cb * TS + s) * 2], l1 = line[(cb * TS + s) * 2 + 1];
                    const float dx = rfx - l0.x, dy = rfy - l0.y, dz = rfz - l0.z;
                    const float r2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
                    k_slot = l0.w;
                    if constexpr (GUESS == 4) {
                        return kcur >= 1 && kcur < D ? (float)kcur : (float)(D - 1);
                    } else if constexpr (GUESS == 3) {
                        // surrogate per pair: predicted c (t - t_r) / |r - w_n| times the distance
                        return p.G[jt * p.g_groups + grp_index] * __builtin_amdgcn_sqrtf(r2) * inv_cdt;
                    } else {
                        const float b = __builtin_fmaf(dx, l1.x, __builtin_fmaf(dy, l1.y, dz * l1.z));
                        const float gf = b + __builtin_amdgcn_sqrtf(__builtin_fmaf(b, b, l0.w * r2));
                        // surrogate, one evaluation per group: the group's
                        // correction factor to straight-line motion
                        return GUESS == 1 ? gf * gcorr[(cb * kWaves + wave) * TS + s] : gf;
                    }
                };
                int g;           // the bracket's older end, D - 1 before the history
                double3 d1;      // the target's offset from it
                double q0, q1;   // sign-test values of its newer and older end
                bool before;     // the retarded time precedes the history
                auto bracket_at = [&](int at) {
                    double3 d;
                    g = at;
                    q0 = value_at(addr(g - 1), d);
                    q1 = value_at(addr(g - 1) + (uint32_t)sizeof(double2), d1);
                };
                const bool other = j != self;
                int n_tests = 0, n_fall = 0;  // of a plain search
                if constexpr (COUNT || (kChord && KSTAR)) {
                    // The mode's search in its plain form, whose sign tests
                    // are counted: the paper's bisection (the halvings of the
                    // whole history), or a guess confirmed by two samples and
                    // followed by a gallop.  k* of the bisection mode is this
                    // search's too, lane by lane (such calls are bound by the
                    // 4 N bytes of k* a target: 4096 targets of 8192 sources,
                    // D = 512, 699 us so and 778 by guess, 724 and 684 on a
                    // curving history).
                    int n = 0, b;
                    if constexpr (kChord) {
                        b = search_bisect(test, D, n);
                        n = b < 0 ? 1 : 1 + (D > 2 ? 32 - __clz(D - 2) : 0);
                    } else {
                        bool hit = false;
                        b = -1;
                        if (GUESS == 4) {
                            // the previous step's bracket still holds
                            const int k = kcur;
                            const bool was_before = kcur == kBracketBefore, in_range = k >= 1 && k < D;
                            hit = was_before ? !test(D - 1) : in_range && test(k) && !test(k - 1);
                            b = in_range ? k : -1;
                            n = was_before || k == 1 ? 1 : 2;
                        }
                        if (!hit && other)
                            b = search_guided(test, D, guess_of(), 6, n, n_fall);
                    }
                    n_tests = n;
                    before = b < 0;
                    bracket_at(before ? D - 1 : b);
                } else {
                    // A guessed bracket, confirmed by the two samples that
                    // define it, in every lane; lanes that miss get one more
                    // guess from the two values, and a wavefront with a lane
                    // that still misses bisects, all lanes in step.
                    bool miss = other;
                    if (bisect_left == 0) {
                        const float last = (float)(D - 1);
                        auto confirm = [&](float guess) {
                            bracket_at((int)__builtin_amdgcn_fmed3f(__builtin_ceilf(guess), 1.0f, last));
                            // hit: (in, out), or the oldest sample out
                            const bool in1 = q1 > 0.0;
                            miss = other & ((in1 & (q0 > 0.0)) | (!in1 & (g != D - 1)));
                        };
                        confirm(guess_of());
                        if (any_lane(miss)) {
                            // The sign-test value is close to a quadratic in
                            // the slot: its value and difference at the tested
                            // pair with the chord's curvature give the next
                            // guess.
                            if (miss) {
                                const float curv = __builtin_amdgcn_rcpf(k_slot);
                                const float F = (float)q1, S = (float)(q1 - q0) + curv;
                                confirm((float)g - 2.0f * F *
                                                       __builtin_amdgcn_rcpf(S + __builtin_amdgcn_sqrtf(__builtin_fmaf(
                                                                                     S, S, -4.0f * curv * F))));
                            }
                            if (any_lane(miss) && ++miss_run >= kMissRun) {
                                bisect_left = bisect_run;
                                if (GUESS != 4)
                                    bisect_run = min(2 * bisect_run, kBisectMost);
                            }
                        } else {
                            miss_run = 0;
                            bisect_run = kBisectRun;
                        }
                    } else {
                        --bisect_left;
                        // the search below gives every lane a bracket, also
                        // where all are left out (a single target's own source)
                        miss = true;
                    }
                    if (any_lane(miss)) {
                        // The paper's search: the halvings of the whole history,
                        // their widths uniform across lanes (extra halvings of a
                        // one-step bracket change nothing); out of history the
                        // bracket ends at the oldest sample, which is not in.  A
                        // wavefront whose first halvings all ran to the oldest end
                        // tests that sample and may be done.  Bound by LDS reads:
                        // steps on a curving history (N = 65536, D = 512) took 36.9
                        // ms with the oldest sample tested first, both of the
                        // bracket's samples read again and runs of 30, 34.2 now;
                        // D = 128 over a quarter of the time, half of the pairs
                        // before it, 28.9 and 25.9 (28.2 with whole batches of
                        // three halvings, 9 where 7 do).  A count of the sources
                        // out of history that puts the oldest sample first where
                        // they are many: 35.4 on the first, 26.5.  One loop for
                        // the first batch and the others keeps the kernel short:
                        // written out twice 34.5 and 26.1, and a step of 256
                        // particles, which fetches its code anew, 14.9 us for 14.6.
                        uint32_t xo = src0;  // f(xo) <= 0, the bracket lies in (xo, xo + n]
                        int n = D - 1;
                        auto halve = [&]() {
                            const int half = n >> 1;
                            const uint32_t mo = xo + (uint32_t)half * (uint32_t)sizeof(double2);
                            double3 d;
                            xo = value_at(mo, d) > 0.0 ? xo : mo;
                            n -= half;
                        };
                        for (bool first = true;; first = false) {
#pragma unroll
                            for (int k = 0; k < 3; ++k)
                                halve();
                            if (first && !any_lane(other & (xo != addr(D - 1 - n))) && !any_lane(other & test(D - 1))) {
                                xo = addr(D - 2);
                                n = 1;
                            }
                            if (n <= 4)
                                break;
                        }
                        while (n > 1)
                            halve();
                        g = (int)((xo - src0) / (uint32_t)sizeof(double2)) + 1;
                        q1 = value_at(addr(g), d1);
                        // the newer end's value matters at the newest sample alone
                        q0 = -1.0;
                        if (any_lane(g == 1)) {
                            double3 d;
                            q0 = value_at(src0, d);
                        }
                    }
                    before = !(q1 > 0.0);
                }
                // A target on the source's newest position (eta = 0) has the
                // value 0 there and the bracket next to it.
                bool valid = other;
                if (any_lane(q0 == 0.0))
                    valid = other & !((q0 == 0.0) & (g == 1));
                // the bracket's velocity records: uniform row base plus 32-bit
                // lane offsets
                uint32_t o1, o2;  // byte offsets of the two records in the source's row
                if constexpr (DB) {
                    const uint32_t w = slot_off[g];
                    o1 = w & 0xffffu;
                    o2 = w >> 16;
                } else {
                    int ph1 = p.head - g;
                    ph1 += ph1 < 0 ? D : 0;
                    const int ph2 = ph1 + 1 == D ? 0 : ph1 + 1;
                    o1 = (uint32_t)ph1 * (uint32_t)sizeof(double2);
                    o2 = (uint32_t)ph2 * (uint32_t)sizeof(double2);
                }
                const char *row = reinterpret_cast<const char *>(p.vel.plane + jt * D);
                const int64_t pl = p.vel.n * (int64_t)sizeof(double2);
                auto at = [&](int k, uint32_t o) { return *reinterpret_cast<const double2 *>(row + k * pl + o); };
                const double2 u0 = at(0, o1);
                bool ok;
                if constexpr (MIX) {
                    float f[6];
                    bool resc = false;
                    const double2 u3 = at(3, o1), w0 = at(0, o2), w3 = at(3, o2);  // plane 3: {1/h, v_z}
                    ok = lw_pair_mixed<GUESS == 0>(Ls[g], MixedPair{d1, make_double4(u0.x, u0.y, u3.y, u3.x),
                                                                   make_double4(w0.x, w0.y, w3.y, 0.0)},
                                                   before, (float)p.kq, f, resc);
                    if (COUNT && valid && active)
                        nresc += resc ? 1 : 0;
                    if (valid && ok) {
#pragma unroll
                        for (int k = 0; k < 6; ++k)
                            acc[k] += f[k];
                    }
                } else {
                    const double2 u1 = at(1, o1), u2 = at(2, o1);
                    const double3 v1 = make_double3(u0.x, u0.y, u1.x);
                    const double3 acc1 = make_double3(zero_if(before, u1.y), zero_if(before, u2.x), zero_if(before, u2.y));
                    double3 E, h, vr;
                    double en;
                    if constexpr (MID) {
                        // w_2 - w_1 from the offsets from both ends
                        double3 d2;
                        (void)value_at(addr(g - 1), d2);
                        const double3 dw = make_double3(d1.x - d2.x, d1.y - d2.y, d1.z - d2.z);
                        const double2 w0 = at(0, o2);
                        const double3 v2 = make_double3(w0.x, w0.y, at(3, o2).y);
                        ok = lw_pair<MID>(d1, q1, Ls[g], v1, acc1, E, h, en, vr, !before, v2, dw);
                    } else {
                        ok = lw_pair<MID>(d1, q1, Ls[g], v1, acc1, E, h, en, vr, false, v1, d1);
                    }
                    if (valid && ok) {
                        acc[0] += E.x;
                        acc[1] += E.y;
                        acc[2] += E.z;
                        // B = eta_hat x E / c
                        acc[3] = __builtin_fma(-h.z, E.y, __builtin_fma(h.y, E.z, acc[3]));
                        acc[4] = __builtin_fma(-h.x, E.z, __builtin_fma(h.z, E.x, acc[4]));
                        acc[5] = __builtin_fma(-h.y, E.x, __builtin_fma(h.x, E.y, acc[5]));
                        if constexpr (ADAPT) {
                            // selects, no branch (N = 65536: 30.6 ms, 31.7 with one)
                            const bool in = en >= p.eta_allow;
                            const double dx = vt.x - vr.x, dy = vt.y - vr.y, dz = vt.z - vr.z;
                            const double d2 = dx * dx + dy * dy + dz * dz;
                            eta_min = in & (en < eta_min) ? en : eta_min;
                            dv2_max = in & (d2 > dv2_max) ? d2 : dv2_max;
                        }
                    }
                }
                // a coincident pair that is not left out, or a failed root
                const bool failed = other & !(valid & ok);
                if (any_lane(failed) && failed)
                    fail_j = min(fail_j, j);
                // (kept out of the way of the loads: their wait is in order)
                if (GUESS >= 4 && valid && active) {
                    const uint16_t k = before ? kBracketBefore : (uint16_t)g;
                    if (GUESS == 5 || k != kcur)
                        p.kc[jt * p.m + a] = k;
                }
                if (KSTAR && valid && active)
                    p.kstar[a * p.n_src + jt] = before ? -1 : g;
                if (COUNT && valid && active) {
                    npairs += 1;
                    nbefore += before ? 1 : 0;
                    probes += n_tests;
                    nfall += n_fall;
                }
            }
            // plain partial sums over kPlainRun sources, then one compensated
            // merge (the same cadence for every search mode: results are
            // bit-identical)
            if (--left == 0) {
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    if constexpr (MIX)
                        two_sum(sum[k], comp[k], acc[k]);
                    else
                        neumaier(sum[k], comp[k], acc[k]);
                    acc[k] = 0;
                }
                next_run();
            }
        }
        if (DB) {
            cb ^= 1;
            __syncthreads();
        }
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        if constexpr (MIX)
            two_sum(sum[k], comp[k], acc[k]);
        else
            neumaier(sum[k], comp[k], acc[k]);
    }
    if constexpr (DB && !MIX) {
        // the sums of a target's other wavefronts, in order, through the tile
        // buffers (the last barrier has retired them)
        if (SG > 1) {
            double *red = reinterpret_cast<double *>(lds);
            const int t = tw * 64 + lane;
            if (sg > 0) {
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    red[((sg - 1) * 12 + k) * targets + t] = sum[k];
                    red[((sg - 1) * 12 + 6 + k) * targets + t] = comp[k];
                }
            }
            __syncthreads();
            if (sg == 0) {
                for (int g = 0; g + 1 < SG; ++g) {
#pragma unroll
                    for (int k = 0; k < 6; ++k) {
                        neumaier(sum[k], comp[k], red[(g * 12 + k) * targets + t]);
                        comp[k] += red[(g * 12 + 6 + k) * targets + t];
                    }
                }
            }
        }
    }
    if (active) {
        // partials in the launch's target order (consecutive threads write
        // consecutive entries); the merge maps them to particle indices
        double *out = p.part + (int64_t)split * 12 * p.m + a;
        const double scale = MIX ? 1.0 : p.kq;
        if (sg == 0) {
            for (int k = 0; k < 6; ++k) {
                out[k * p.m] = (double)sum[k] * scale;
                out[(6 + k) * p.m] = (double)comp[k] * scale;
            }
        }
        if (fail_j != INT32_MAX)
            report_error(p.err, !p.x && p.order ? (int64_t)p.order[a] : p.a_base + a, fail_j, kErrCoincident);
    }
    if (ADAPT) {
        // one atomic pair per wavefront
        for (int off = 32; off > 0; off >>= 1) {
            eta_min = fmin(eta_min, __shfl_xor(eta_min, off));
            dv2_max = fmax(dv2_max, __shfl_xor(dv2_max, off));
        }
        if (lane == 0) {
            atomicMin(&p.ad[0], (unsigned long long)__double_as_longlong(eta_min));
            atomicMax(&p.ad[1], (unsigned long long)__double_as_longlong(dv2_max));
        }
    }
    if (COUNT) {
        // one atomic per wavefront
        unsigned long long c0 = npairs, c1 = nbefore, c2 = probes, c3 = nfall, c4 = nresc;
        for (int off = 32; off > 0; off >>= 1) {
            c0 += __shfl_down(c0, off);
            c1 += __shfl_down(c1, off);
            c2 += __shfl_down(c2, off);
            c3 += __shfl_down(c3, off);
            c4 += __shfl_down(c4, off);
        }
        if (lane == 0) {
            atomicAdd(&p.counters[0], c0);
            atomicAdd(&p.counters[1], c1);
            atomicAdd(&p.counters[2], c2);
            atomicAdd(&p.counters[4], c3);
            if (MIX)
                atomicAdd(&p.counters[3], c4);
        }
    }
}

}  // namespace empp
