// pair_kernel.h -- the all-pairs Lienard-Wiechert pass shared by the FP64
// and the mixed-precision pair kernels (Secs. 2.1-2.2 of arXiv 2605.05543).
//
// One thread owns one target.  A block of kBlockFp64 (1024) threads walks its
// chunk of sources in staged tiles of up to 16 sources: the tile's
// histories, as the per-sample part of the split light-cone test (offsets
// from each source's newest sample and L^2 - |offset|^2, see pair_common.h),
// are staged once into LDS, double-buffered behind one barrier per tile, and
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
// What bounds it: the latency of a pair's chain (LDS reads of the confirming
// samples, a gather of two 32-byte records from L2, about 70 dependent FP64
// instructions) on four wavefronts per SIMD, then vector issue.  The history
// is searched by guess and confirmation in every mode, the bisection's too:
// the unrolled bisection's ten probes of 32 bytes kept the LDS busy for nine
// tenths of the pass at N = 65536, D = 512 (33.1 ms; with a guess from the
// oldest sample, the acceleration and c^2 - v^2 of each segment kept with the
// history, and the root's square root reused as eta . v', 26.1 ms: 141 vector
// instructions per wavefront and pair against 193).
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
// per buffer and source the guess's data, per buffer, wavefront and source
// the surrogate's correction, and the per-source data of three tiles.
constexpr size_t pair_lds_bytes(int D)
{
    const bool two = pair_two_buffers(D);
    const size_t ts = (size_t)pair_staged_tile(D);
    return (two ? 4 * (size_t)kHalfRecs : 2 * (size_t)D) * sizeof(double2) + (size_t)((D + 1) & ~1) * sizeof(double) +
           (two ? (size_t)((D + 3) & ~3) * sizeof(uint32_t) : 0) + 2 * ts * sizeof(float4) +
           2 * kWaves * ts * sizeof(float) + 3 * ts * 8 * sizeof(double);
}

static_assert(pair_lds_bytes(kMaxDepth) <= 160 * 1024,
              "the deepest history's tile, light distances and per-source data fit a CU's LDS");
static_assert(pair_lds_bytes(kHalfRecs) <= 160 * 1024, "the deepest double-buffered tiles fit with the slot table");
// its 16-bit byte offsets of 32-byte ring entries
static_assert((kHalfRecs - 1) * 32 < 65536, "slot table offsets fit 16 bits");

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
// velocity, a the acceleration (zero out of history) and C2 = c^2 - |v1|^2
// of the bracket's segment.  E, and h = eta_hat / c for B = h x E.  Returns
// false on a numerical failure (negative discriminant, eta <= 0), which
// reaches the last test as a NaN.
// The root sq of the discriminant is eta . v' at v_1, C2 dt being
// -(C1h + sq): with v_r = v_1 + a dt, eta . v' = sq - dt (eta . a), one
// instruction and no difference of large terms (rounding of a pair's field
// at 5 MeV 1.6e-14 rms, against 7.5e-14 from c |eta| - eta . v_r).
// MID and mid: Eq. (mid) with the bracket's other velocity v2 and dw =
// w_2 - w_1 (the accuracy ablation).
template <bool MID>
__device__ __forceinline__ bool lw_pair(double3 d, double C0, double L1, double4 v1, double3 a, double C2, double3 &E,
                                        double3 &h, double &en, double3 &vr, bool mid, double4 v2, double3 dw)
{
    const double c = kC_LIGHT;
    const double c2 = c * c;
    // C2 dt^2 + 2 C1h dt + C0 = 0 (Eq. dt with C1 = 2 C1h); the physical
    // root -(C1h + sqrt(C1h^2 - C2 C0))/C2 in Vieta's form.
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
// next kBisectRun sources before it guesses again.
constexpr int kMissRun = 3, kBisectRun = 30;

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
    const bool active = a < p.m;
    // sources j0 .. j0 + nj - 1
    const int64_t j0 = (int64_t)split * p.src_per_split;
    const int nj = (int)max((int64_t)0, min(p.n_src - j0, p.src_per_split));

    double rx = 0, ry = 0, rz = 0;
    double3 vt = make_double3(0.0, 0.0, 0.0);  // target's present velocity (adaptive step)
    double eta_min = __longlong_as_double((long long)kPosInfBits), dv2_max = 0.0;
    int64_t tgt = a;    // index the outputs are written at
    int32_t self = -1;  // source left out (sources number at most 2^31)
    if (active) {
        if (p.x) {
            rx = p.x[a];
            ry = p.x[p.m + a];
            rz = p.x[2 * p.m + a];
            self = p.self_index ? (int32_t)p.self_index[a] : -1;
        } else {
            tgt = p.order ? (int64_t)p.order[a] : a;
            double4 w = p.ring_w[tgt * D + p.head];
            rx = w.x;
            ry = w.y;
            rz = w.z;
            self = (int32_t)tgt;
            if (ADAPT) {
                double4 vn = p.ring_v[tgt * D + p.head];
                vt = make_double3(vn.x, vn.y, vn.z);
            }
        }
    }
    // field sums: FP64 with Neumaier compensation, or FP32 with two-sum
    using Real = std::conditional_t<MIX, float, double>;
    Real sum[6] = {0, 0, 0, 0, 0, 0}, comp[6] = {0, 0, 0, 0, 0, 0};
    Real acc[6] = {0, 0, 0, 0, 0, 0};
    constexpr int kPlainRun = MIX ? 8 : 32;  // sources per plain partial
    int in_acc = 0;
    int probes = 0, nbefore = 0, npairs = 0, nfall = 0, nresc = 0;
    // first (lowest) source of a failing pair; sources number below 2^31
    int32_t fail_j = INT32_MAX;
    const float inv_cdt = (float)(1.0 / (kC_LIGHT * p.dt));
    const int64_t grp_index = a >> p.g_shift;  // surrogate group of this target

    // LDS: the tile buffers, then the light distance of every logical slot
    // (shared by all sources).  A buffer holds its TS * D records
    // {-2 D, A} of the split sign test (lightcone_record) as two arrays of
    // 16-byte halves, {-2 D_x, -2 D_y} then {-2 D_z, A}, hrec halves apart:
    // lanes that probe different slots then spread over twice as many LDS
    // bank groups as with 32-byte records.  With two buffers the distance is
    // the fixed kHalfRecs, so a probe's reads share one address (the others
    // at immediate offsets).
    constexpr int nbuf = DB ? 2 : 1;
    const int TS = DB ? p.tile : 1;
    const int hrec = DB ? kHalfRecs : D;
    const uint32_t hbytes = DB ? (uint32_t)(kHalfRecs * sizeof(double2)) : (uint32_t)D * (uint32_t)sizeof(double2);
    double2 *const halves = reinterpret_cast<double2 *>(lds);
    double *Ls = reinterpret_cast<double *>(halves + nbuf * 2 * hrec);
    // slot table (two buffers): for back offset b, the byte offset in a ring
    // row of physical slot (head - b) mod D and, above 16 bits, of the next
    // newer slot's (the bracket's two velocity records)
    uint32_t *slot_off = reinterpret_cast<uint32_t *>(Ls + ((D + 1) & ~1));
    float4 *line = reinterpret_cast<float4 *>(slot_off + (DB ? ((D + 3) & ~3) : 0));  // [buffer][source]
    float *gcorr = reinterpret_cast<float *>(line + 2 * TS);  // [buffer][wavefront][source]
    // Per-source data of three consecutive staged tiles (tile i in slot
    // i % 3): the newest sample w_n and the vector the guess is made from
    // (the oldest sample of a bisection, else the newest velocity).  Eight
    // threads per source load a double each, two tiles ahead of the tile's
    // search, and write it a tile later, so that no wavefront waits for it.
    constexpr bool kChord = GUESS == 0 || GUESS == 5;
    constexpr bool kLine = GUESS <= 2 || GUESS == 5;
    double *aux = reinterpret_cast<double *>(gcorr + 2 * kWaves * TS);
    double aux_pf = 0.0;
    const char *const aux_src = [&]() {
        const int oldest = p.head + 1 == D ? 0 : p.head + 1;
        const double4 *v = kChord ? p.ring_w + oldest : p.ring_v + p.head;
        const double4 *at = ((tid & 4) ? v : p.ring_w + p.head) + (int64_t)(tid >> 3) * D;
        return reinterpret_cast<const char *>(at) + (tid & 3) * sizeof(double);
    }();
    auto load_aux = [&](int64_t jt, int ns) {
        if (tid < 8 * ns)
            aux_pf = *reinterpret_cast<const double *>(aux_src + jt * D * (int64_t)sizeof(double4));
    };
    auto put_aux = [&](int slot3, int ns) {
        if (tid < 8 * ns)
            aux[slot3 * TS * 8 + tid] = aux_pf;
    };
    auto next3 = [](int i) { return i == 2 ? 0 : i + 1; };
    // the present time is the newest slot's (the clock lives in T)
    const double tnow = p.T[p.head];
    for (int b = tid; b < D; b += kBlockFp64) {
        int ph = p.head - b;
        ph += ph < 0 ? D : 0;
        Ls[b] = kC_LIGHT * (tnow - p.T[ph]);
        if constexpr (DB) {
            const int ph2 = ph + 1 == D ? 0 : ph + 1;  // back offset b - 1 (read for b >= 1)
            slot_off[b] = (uint32_t)ph * (uint32_t)sizeof(double4) | (uint32_t)ph2 * (uint32_t)sizeof(double4) << 16;
        }
    }
    // Record q of a tile: source q / D (q < TS D), slot q % D, computed from
    // the position while staging.  A thread's records, q = tid + 1024 k, keep
    // their source and slot in every tile, so a load is a uniform row base plus
    // a fixed 32-bit offset.  Positions are prefetched into registers one tile
    // ahead (the first two of each thread: a whole tile with two buffers), so
    // the latency overlaps the previous tile's work; deeper histories load
    // the rest in place.
    auto src_of = [&](int q) { return DB ? q / D : 0; };
    auto pos_off = [&](int q) {
        const int s = src_of(q);
        int ph = p.head - (q - s * D);
        ph += ph < 0 ? D : 0;
        return (uint32_t)(s * D + ph) * (uint32_t)sizeof(double4);
    };
    const int qa = min(tid, TS * D - 1), qb = min(tid + kBlockFp64, TS * D - 1);
    const uint32_t off_a = pos_off(qa), off_b = pos_off(qb);
    const int sa = src_of(qa), sb = src_of(qb);
    auto fetch = [&](int64_t jt, int nrec, int q, uint32_t off, double4 &w) {
        if (q < nrec)
            w = *reinterpret_cast<const double4 *>(reinterpret_cast<const char *>(p.ring_w + jt * D) + off);
    };
    auto put = [&](int bi, int slot3, int nrec, int q, int s, int b, const double4 &w) {
        if (q < nrec) {
            const double *wn = aux + (slot3 * TS + s) * 8;
            const double4 r = lightcone_record(make_double4(wn[0], wn[1], wn[2], 0.0), w, Ls[b]);
            double2 *xy = halves + bi * 2 * hrec + q;
            xy[0] = make_double2(r.x, r.y);
            xy[hrec] = make_double2(r.z, r.w);
        }
    };
    // Tile jt of ns sources into buffer bi, from the prefetched positions.
    auto stage = [&](int bi, int slot3, int64_t jt, int ns, const double4 &w0, const double4 &w1) {
        if (kLine && tid < ns) {
            // the guessed slot b = d0.l + sqrt((d0.l)^2 + k |d0|^2) in float
            const double *ax = aux + (slot3 * TS + tid) * 8;
            if constexpr (kChord) {
                // along the chord from the newest to the oldest sample the
                // sign-test value is alpha b^2 - 2 alpha b (d0.l) - |d0|^2,
                // exactly so on a straight path: alpha = (L^2 - |D|^2) /
                // (D - 1)^2 of the oldest sample, l = D / ((D - 1) alpha)
                const double dx = ax[0] - ax[4], dy = ax[1] - ax[5], dz = ax[2] - ax[6];
                const double Lo = Ls[D - 1], n = (double)(D - 1);
                const double ia = n * n / (Lo * Lo - (dx * dx + dy * dy + dz * dz));
                const double f = ia / n;
                line[bi * TS + tid] = make_float4((float)(dx * f), (float)(dy * f), (float)(dz * f), (float)ia);
            } else {
                // straight-line look-back: with beta the source's newest
                // velocity / c, the positive root of
                // (1 - beta^2) s^2 - 2 (R.beta) s - R^2 = 0, in steps of c dt
                const double ic = 1.0 / kC_LIGHT;
                const double bx = ax[4] * ic, by = ax[5] * ic, bz = ax[6] * ic;
                const double ig2 = 1.0 / (1.0 - (bx * bx + by * by + bz * bz));
                const double is = 1.0 / (kC_LIGHT * p.dt), f = ig2 * is;
                line[bi * TS + tid] = make_float4((float)(bx * f), (float)(by * f), (float)(bz * f), (float)(f * is));
            }
        }
        if (GUESS == 1 && tid < kWaves * TS) {
            // guess mode 1: the surrogate's correction for groups of 64 or
            // more targets (whole wavefronts) is staged with the tile
            const int w = tid / TS, sj = tid - w * TS;
            const int64_t aw = (int64_t)bxi * targets + (w & ((1 << tw_log2) - 1)) * 64;
            if (sj < ns && aw < p.m)
                gcorr[(bi * kWaves + w) * TS + sj] = p.G[(jt + sj) * p.g_groups + (aw >> p.g_shift)];
        }
        const int nrec = ns * D;
        put(bi, slot3, nrec, tid, sa, qa - sa * D, w0);
        put(bi, slot3, nrec, tid + kBlockFp64, sb, qb - sb * D, w1);
        if constexpr (!DB)
            for (int q = tid + 2 * kBlockFp64; q < nrec; q += kBlockFp64) {
                double4 w;
                fetch(jt, nrec, q, pos_off(q), w);
                put(bi, slot3, nrec, q, 0, q, w);
            }
    };
    auto tile_size = [&](int i) { return min(nj - i, TS); };
    double4 pf0, pf1;
    auto prefetch = [&](int i) {
        fetch(j0 + i, tile_size(i) * D, tid, off_a, pf0);
        fetch(j0 + i, tile_size(i) * D, tid + kBlockFp64, off_b, pf1);
    };
    // Two buffers: tile i + 1 is written while tile i is searched, and one
    // barrier per tile both publishes tile i + 1 and retires tile i's
    // buffer for tile i + 2.  One buffer (deep histories): stage, then
    // search, with a barrier on either side.
    int cur3 = 0;  // the searched tile's slot of the per-source data
    if (nj > 0) {
        prefetch(0);
        load_aux(j0, tile_size(0));
        put_aux(0, tile_size(0));
        if (TS < nj) {
            load_aux(j0 + TS, tile_size(TS));
            put_aux(1, tile_size(TS));
        }
        if (2 * TS < nj)
            load_aux(j0 + 2 * TS, tile_size(2 * TS));
        if (DB) {
            __syncthreads();
            stage(0, 0, j0, tile_size(0), pf0, pf1);
            if (TS < nj)
                prefetch(TS);
            __syncthreads();
        }
    }
    // previous-step bracket of this wavefront's next source (warm start)
    uint16_t knext = kBracketBefore;
    auto load_bracket = [&](int i) { knext = active && i < nj ? p.kc[(j0 + i) * p.m + a] : kBracketBefore; };
    if (GUESS == 4)
        load_bracket(sg);
    int miss_run = 0, bisect_left = 0;
    int cb = 0;
    for (int i0 = 0; i0 < nj; i0 += TS) {
        if (DB) {
            if (i0 + TS < nj) {
                stage(cb ^ 1, next3(cur3), j0 + i0 + TS, tile_size(i0 + TS), pf0, pf1);
                if (i0 + 2 * TS < nj) {
                    prefetch(i0 + 2 * TS);
                    put_aux(next3(next3(cur3)), tile_size(i0 + 2 * TS));
                    if (i0 + 3 * TS < nj)
                        load_aux(j0 + i0 + 3 * TS, tile_size(i0 + 3 * TS));
                }
            }
        } else {
            __syncthreads();
            stage(0, cur3, j0 + i0, tile_size(i0), pf0, pf1);
            __syncthreads();
            if (i0 + TS < nj)
                prefetch(i0 + TS);
            if (i0 + 2 * TS < nj) {
                put_aux(next3(next3(cur3)), tile_size(i0 + 2 * TS));
                if (i0 + 3 * TS < nj)
                    load_aux(j0 + i0 + 3 * TS, tile_size(i0 + 3 * TS));
            }
        }
        const int ns = tile_size(i0);
        for (int s = sg; s < ns; s += SG) {
            const int64_t jt = j0 + i0 + s;
            const int32_t j = (int32_t)jt;
            const uint16_t kcur = knext;
            if (GUESS == 4)
                load_bracket(s + SG < ns ? i0 + s + SG : i0 + TS + sg);
            if (active) {
                // the target's offset d0 = r - w_n from the source's newest
                // sample, and |d0|^2 (the pair's part of the sign test)
                const double *wn = aux + (cur3 * TS + s) * 8;
                const double d0x = rx - wn[0], d0y = ry - wn[1], d0z = rz - wn[2];
                const double R0 = offset_sq(d0x, d0y, d0z);
                // a target on the source's present position has eta = 0 (one
                // compare: |d0|^2 is 0 only when d0 is, for offsets above
                // 1e-154 m)
                const bool valid = (R0 != 0.0) & (j != self);
                if (KSTAR && j == self)
                    p.kstar[a * p.n_src + jt] = 0;
                // LDS byte address of the source's first record (its first half)
                const uint32_t src0 =
                    lds_base + (uint32_t)(cb * 2 * hrec + s * D) * (uint32_t)sizeof(double2);
                auto rec_at = [&](uint32_t o) {
                    const dv2 va = *(lds_dv2)(uintptr_t)o, vb = *(lds_dv2)(uintptr_t)(o + hbytes);
                    return make_double4(va.x, va.y, vb.x, vb.y);
                };
                auto rec = [&](int b) { return rec_at(src0 + (uint32_t)b * (uint32_t)sizeof(double2)); };
                auto value = [&](double4 r) { return lightcone_value(r, d0x, d0y, d0z); };
                auto test = [&](int b) { return value(rec(b)) > R0; };

                int g;        // the bracket's older end, D - 1 before the history
                double4 r1;   // its record
                double q1;    // and sign-test value
                bool before;  // the retarded time precedes the history
                // the guessed slot of a guided search
                auto guess_of = [&]() -> float {
                    if constexpr (kLine) {
                        const float4 l = line[cb * TS + s];
                        const float b = __builtin_fmaf((float)d0x, l.x, __builtin_fmaf((float)d0y, l.y, (float)d0z * l.z));
                        const float gf = b + __builtin_amdgcn_sqrtf(__builtin_fmaf(b, b, l.w * (float)R0));
                        // surrogate, one evaluation per group: the group's
                        // correction factor to straight-line motion
                        return GUESS == 1 ? gf * gcorr[(cb * kWaves + wave) * TS + s] : gf;
                    } else if constexpr (GUESS == 4) {
                        return kcur >= 1 && kcur < D ? (float)kcur : (float)(D - 1);
                    } else {
                        // surrogate per pair: predicted c (t - t_r) / |r - w_n| times the distance
                        return p.G[jt * p.g_groups + grp_index] * __builtin_amdgcn_sqrtf((float)R0) * inv_cdt;
                    }
                };
                if constexpr (COUNT || (kChord && KSTAR)) {
                    // The mode's search in its plain form, whose sign tests
                    // are counted: the paper's bisection (the halvings of the
                    // whole history), or a guess confirmed by two samples and
                    // followed by a gallop.
                    int n = 0, fb = 0, b;
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
                        if (!hit && valid)
                            b = search_guided(test, D, guess_of(), 6, n, fb);
                    }
                    if (COUNT && valid) {
                        probes += n;
                        nfall += fb;
                    }
                    before = b < 0;
                    g = before ? D - 1 : b;
                    r1 = rec(g);
                    q1 = value(r1);
                } else {
                    // A guessed bracket, confirmed by the two samples that
                    // define it, in every lane; lanes that miss get one more
                    // guess from the two values, and a wavefront with a lane
                    // that still misses bisects, all lanes in step.
                    bool in1, miss = true;
                    if (bisect_left == 0) {
                        const float last = (float)(D - 1);
                        double q0;
                        auto confirm = [&](float guess) {
                            g = (int)__builtin_amdgcn_fmed3f(__builtin_ceilf(guess), 1.0f, last);
                            const uint32_t o = src0 + (uint32_t)(g - 1) * (uint32_t)sizeof(double2);
                            q0 = value(rec_at(o));
                            r1 = rec_at(o + (uint32_t)sizeof(double2));
                            q1 = value(r1);
                            in1 = q1 > R0;
                            // hit: (in, out), or the oldest sample out
                            miss = valid & ((in1 & (q0 > R0)) | (!in1 & (g != D - 1)));
                        };
                        confirm(guess_of());
                        if (any_lane(miss)) {
                            // The sign-test value is close to a quadratic in
                            // the slot: its value and difference at the tested
                            // pair with the chord's curvature give the next
                            // guess.
                            if (miss) {
                                const float curv = (float)rec(D - 1).w * __builtin_amdgcn_rcpf(last * last);
                                const float F = (float)(q1 - R0), S = (float)(q1 - q0) + curv;
                                confirm((float)g - 2.0f * F *
                                                       __builtin_amdgcn_rcpf(S + __builtin_amdgcn_sqrtf(__builtin_fmaf(
                                                                                     S, S, -4.0f * curv * F))));
                            }
                            if (any_lane(miss) && ++miss_run >= kMissRun)
                                bisect_left = kBisectRun;
                        } else {
                            miss_run = 0;
                        }
                    } else {
                        --bisect_left;
                        miss = valid;
                    }
                    if (any_lane(miss)) {
                        // The paper's search: the oldest sample, then the
                        // halvings of the whole history, their widths uniform
                        // across lanes (extra halvings of a one-step bracket
                        // change nothing).
                        in1 = test(D - 1);
                        uint32_t xo = src0;  // f(xo) <= 0, the bracket lies in (xo, xo + n]
                        if (any_lane(in1 & valid)) {
                            int n = D - 1;
                            do {
#pragma unroll
                                for (int k = 0; k < 3; ++k) {
                                    const int half = n >> 1;
                                    const uint32_t mo = xo + (uint32_t)half * (uint32_t)sizeof(double2);
                                    xo = value(rec_at(mo)) > R0 ? xo : mo;
                                    n -= half;
                                }
                            } while (n > 1);
                        }
                        g = in1 ? (int)((xo - src0) / (uint32_t)sizeof(double2)) + 1 : D - 1;
                        r1 = rec(g);
                        q1 = value(r1);
                    }
                    before = !in1;
                }
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
                    o1 = (uint32_t)ph1 * (uint32_t)sizeof(double4);
                    o2 = (uint32_t)ph2 * (uint32_t)sizeof(double4);
                }
                const int64_t row = jt * D * (int64_t)sizeof(double4);
                auto at = [&](const double4 *ring, uint32_t o) {
                    return *reinterpret_cast<const double4 *>(reinterpret_cast<const char *>(ring) + row + o);
                };
                const double4 v1 = at(p.ring_v, o1);
                // r - w_1 = d0 + D from the staged -2 D
                const double3 d1 = make_double3(__builtin_fma(-0.5, r1.x, d0x), __builtin_fma(-0.5, r1.y, d0y),
                                                __builtin_fma(-0.5, r1.z, d0z));
                bool ok;
                if constexpr (MIX) {
                    float f[6];
                    bool resc = false;
                    ok = lw_pair_mixed<GUESS == 0>(Ls[g], MixedPair{d1, v1, at(p.ring_v, o2)}, before, (float)p.kq, f, resc);
                    if (COUNT && valid)
                        nresc += resc ? 1 : 0;
                    if (valid && ok) {
#pragma unroll
                        for (int k = 0; k < 6; ++k)
                            acc[k] += f[k];
                    }
                } else {
                    const double4 sg1 = at(p.seg, o1);
                    const double3 acc1 = make_double3(zero_if(before, sg1.x), zero_if(before, sg1.y), zero_if(before, sg1.z));
                    double3 E, h, vr;
                    double en;
                    if constexpr (MID) {
                        // w_2 - w_1 = D_1 - D_2 from the staged -2 D of both ends
                        const double4 r2 = rec(g - 1), v2 = at(p.ring_v, o2);
                        const double3 dw = make_double3(-0.5 * (r1.x - r2.x), -0.5 * (r1.y - r2.y), -0.5 * (r1.z - r2.z));
                        ok = lw_pair<MID>(d1, q1 - R0, Ls[g], v1, acc1, sg1.w, E, h, en, vr, !before, v2, dw);
                    } else {
                        ok = lw_pair<MID>(d1, q1 - R0, Ls[g], v1, acc1, sg1.w, E, h, en, vr, false, v1, d1);
                    }
                    if (valid && ok) {
                        acc[0] += E.x;
                        acc[1] += E.y;
                        acc[2] += E.z;
                        // B = eta_hat x E / c
                        acc[3] = __builtin_fma(-h.z, E.y, __builtin_fma(h.y, E.z, acc[3]));
                        acc[4] = __builtin_fma(-h.x, E.z, __builtin_fma(h.z, E.x, acc[4]));
                        acc[5] = __builtin_fma(-h.y, E.x, __builtin_fma(h.x, E.y, acc[5]));
                        if (ADAPT && en >= p.eta_allow) {
                            const double dx = vt.x - vr.x, dy = vt.y - vr.y, dz = vt.z - vr.z;
                            eta_min = fmin(eta_min, en);
                            dv2_max = fmax(dv2_max, dx * dx + dy * dy + dz * dz);
                        }
                    }
                }
                // a coincident pair that is not left out, or a failed root
                const bool failed = (j != self) & !(valid & ok);
                if (any_lane(failed) && failed)
                    fail_j = min(fail_j, j);
                // (kept out of the way of the loads: their wait is in order)
                if (GUESS >= 4 && valid) {
                    const uint16_t k = before ? kBracketBefore : (uint16_t)g;
                    if (GUESS == 5 || k != kcur)
                        p.kc[jt * p.m + a] = k;
                }
                if (KSTAR && valid)
                    p.kstar[a * p.n_src + jt] = before ? -1 : g;
                if (COUNT && valid) {
                    npairs += 1;
                    nbefore += before ? 1 : 0;
                }
            }
            // plain partial sums over kPlainRun sources, then one compensated
            // merge (the same cadence for every search mode: results are
            // bit-identical)
            if (++in_acc == kPlainRun) {
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    if constexpr (MIX)
                        two_sum(sum[k], comp[k], acc[k]);
                    else
                        neumaier(sum[k], comp[k], acc[k]);
                    acc[k] = 0;
                }
                in_acc = 0;
            }
        }
        cur3 = next3(cur3);
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
            report_error(p.err, tgt, fail_j, kErrCoincident);
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
