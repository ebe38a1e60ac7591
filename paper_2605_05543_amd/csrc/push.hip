// push.hip -- per-particle kernels: merge of the pair partials, centred
// dipole, Higuera-Cary push, drift and history update (Secs. 2.3, 2.6 of
// arXiv 2605.05543), the straight-line prior history, layout conversions
// and bunch diagnostics (Secs. 2.5, 2.7).
#include "empp_dev.h"
#include "pair_common.h"

namespace empp {

// Velocity records {v, 1/h} as checkpoints hold them: records q0 .. q0 + n - 1
// of the ring to or from rec.
__global__ void vel_pack_kernel(VelRing vel, int64_t q0, int64_t n, double4 *rec)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n)
        return;
    const double3 v = vel.v(q0 + k);
    rec[k] = make_double4(v.x, v.y, v.z, vel.inv_h(q0 + k));
}

__global__ void vel_unpack_kernel(const double4 *rec, int64_t q0, int64_t n, VelRing vel)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n)
        return;
    const double4 r = rec[k];
    vel.set_v(q0 + k, make_double3(r.x, r.y, r.z), r.w);
}

// Accelerations of every (source, slot) from the velocities (a ring read
// from a checkpoint; the newest slot has no segment).
__global__ void vel_accel_kernel(VelRing vel, int64_t N, int D)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N * (int64_t)D)
        return;
    const int64_t j = q / D;
    const int ph = (int)(q - j * D);
    vel.set_a(q, vel.v(q), vel.v(j * D + (ph + 1 == D ? 0 : ph + 1)), vel.inv_h(q));
}

// Guess data of every source of a history that was set.
__global__ void guess_lines_kernel(const double4 *ring_w, VelRing vel, const double *T, int64_t N, int D, int head,
                                   double dt, GuessLine *lines)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    const int oldest = head + 1 == D ? 0 : head + 1, before = head == 0 ? D - 1 : head - 1;
    const double4 w = ring_w[i * D + head], wo = ring_w[i * D + oldest], ref = ring_w[before];
    const double3 wn = make_double3(w.x, w.y, w.z), r0 = make_double3(ref.x, ref.y, ref.z);
    lines[i] = chord_line(wn, make_double3(wo.x, wo.y, wo.z), kC_LIGHT * (T[head] - T[oldest]), D, r0);
    lines[N + i] = straight_line(wn, vel.v(i * D + head), dt, r0);
}

static dim3 blocks_of(int64_t n) { return dim3((unsigned)((n + 255) / 256)); }

hipError_t launch_vel_pack(VelRing vel, int64_t q0, int64_t n, double4 *rec, hipStream_t s)
{
    hipLaunchKernelGGL(vel_pack_kernel, blocks_of(n), dim3(256), 0, s, vel, q0, n, rec);
    return hipGetLastError();
}

hipError_t launch_vel_unpack(const double4 *rec, int64_t q0, int64_t n, VelRing vel, hipStream_t s)
{
    hipLaunchKernelGGL(vel_unpack_kernel, blocks_of(n), dim3(256), 0, s, rec, q0, n, vel);
    return hipGetLastError();
}

hipError_t launch_vel_accel(VelRing vel, int64_t N, int D, hipStream_t s)
{
    hipLaunchKernelGGL(vel_accel_kernel, blocks_of(N * (int64_t)D), dim3(256), 0, s, vel, N, D);
    return hipGetLastError();
}

hipError_t launch_guess_lines(const double4 *ring_w, VelRing vel, const double *T, int64_t N, int D, int head, double dt,
                              GuessLine *lines, hipStream_t s)
{
    hipLaunchKernelGGL(guess_lines_kernel, blocks_of(N), dim3(256), 0, s, ring_w, vel, T, N, D, head, dt, lines);
    return hipGetLastError();
}

// Merge of the pair partials part[nsplit][12][m].  Bound by HBM where m is
// large, by the few CUs that a block of targets each puts to work where it is
// small: a chain of compensated additions per component and target, over
// nsplit x 2 loads.  A block takes TG consecutive targets and SL slices of the
// chunks, slice w the chunks w, w + SL, ...; the SL sums are then added in
// order: a fixed order, whatever the scheduling.  Up to kMergeSmall targets it
// is 16 targets (rows of 128 bytes, one line) and 32 slices, or in a step 8
// slices of each of the six components (a step of N = 1024, 256 chunks: 48 us
// with blocks of 64 targets and 16 slices, 30 with 16 and 32; the components
// side by side and not in turn: N = 256 16.1 -> 13.5 us, N = 1024 with 64 chunks
// 26.5 -> 22.9), beyond it 64 and four.
template <int TG, int SL>
__device__ inline void merge_slice(double2 (*red)[TG], const double *part, int nsplit, int64_t m, int k, int64_t a)
{
    const int w = threadIdx.x / TG % SL;
    double s = 0.0, c = 0.0;
    if (a < m) {
        const double *at = part + k * m + a;
#pragma unroll 4
        for (int sp = w; sp < nsplit; sp += SL) {
            const double *base = at + (int64_t)sp * 12 * m;
            neumaier(s, c, base[0]);
            neumaier(s, c, base[6 * m]);
        }
    }
    red[w][threadIdx.x % TG] = make_double2(s, c);
}

// The SL slices' sums of target t, in order.
template <int TG, int SL>
__device__ inline double merge_slices(const double2 (*red)[TG], int t)
{
    double s = 0.0, c = 0.0;
#pragma unroll
    for (int w = 0; w < SL; ++w) {
        const double2 x = red[w][t];
        neumaier(s, c, x.x);
        c += x.y;
    }
    return s + c;
}

// Fields of external targets: component blockIdx.y of TG targets per block,
// written to rows `stride` apart.
template <int TG, int SL>
__global__ __launch_bounds__(TG * SL) void merge_fields_kernel(const double *part, int nsplit, int64_t m, double *E,
                                                               double *B, int64_t stride)
{
    __shared__ double2 red[SL][TG];
    const int t = threadIdx.x % TG, k = blockIdx.y;
    const int64_t a = (int64_t)blockIdx.x * TG + t;
    merge_slice<TG, SL>(red, part, nsplit, m, k, a);
    __syncthreads();
    if (threadIdx.x < TG && a < m)
        (k < 3 ? E + k * stride : B + (k - 3) * stride)[a] = merge_slices<TG, SL>(red, t);
}

// Sec. 2.6: B = (mu0/4pi)(3 (M.rhat) rhat - M)/r^3 with M = M0 e_z, written
// with dip_k = (mu0/4pi) M0 = b0 re^3.
__device__ inline void dipole_field(double x, double y, double z, double dip_k, double &bx, double &by,
                                    double &bz)
{
    double r2 = x * x + y * y + z * z;
    double ir = 1.0 / sqrt(r2);
    double ir3 = ir * ir * ir;
    double mr = z * ir;  // M_hat . r_hat
    double f = dip_k * ir3;
    bx = f * (3.0 * mr * x * ir);
    by = f * (3.0 * mr * y * ir);
    bz = f * (3.0 * mr * z * ir - 1.0);
}

// Sec. 2.3, Higuera-Cary: half electric kick, magnetic rotation with the
// time-centred Lorentz factor gamma+, second half kick (the rotation's
// last term uses u+).
__device__ inline void higuera_cary(double &ux, double &uy, double &uz, double Ex, double Ey, double Ez,
                                    double Bx, double By, double Bz, double eps)
{
    const double c = kC_LIGHT;
    const double ic2 = 1.0 / (c * c);
    double umx = ux + eps * Ex, umy = uy + eps * Ey, umz = uz + eps * Ez;
    double tx = eps * Bx, ty = eps * By, tz = eps * Bz;
    double gm2 = 1.0 + (umx * umx + umy * umy + umz * umz) * ic2;
    double ustar = (umx * tx + umy * ty + umz * tz) / c;
    double tau2 = tx * tx + ty * ty + tz * tz;
    double sig = gm2 - tau2;
    double gp = sqrt(0.5 * (sig + sqrt(sig * sig + 4.0 * (tau2 + ustar * ustar))));
    double igp = 1.0 / gp;
    tx *= igp;
    ty *= igp;
    tz *= igp;
    double s = 1.0 / (1.0 + tx * tx + ty * ty + tz * tz);
    double ut = umx * tx + umy * ty + umz * tz;
    double upx = s * (umx + ut * tx + (umy * tz - umz * ty));
    double upy = s * (umy + ut * ty + (umz * tx - umx * tz));
    double upz = s * (umz + ut * tz + (umx * ty - umy * tx));
    ux = upx + eps * Ex + (upy * tz - upz * ty);
    uy = upy + eps * Ey + (upz * tx - upx * tz);
    uz = upz + eps * Ez + (upx * ty - upy * tx);
}

// One push per particle: add the dipole to the merged self-field,
// Higuera-Cary, finalise the newest slot's velocity, drift, and write the
// new newest slot at physical index head+1.
__device__ inline void push_particle(const PushParams &p, int64_t i, double Ex, double Ey, double Ez, double Bx,
                                     double By, double Bz)
{
    const int D = p.D;
    double4 y = p.ring_w[i * D + p.head];
    if (p.ext_field == 1) {
        double gx, gy, gz;
        dipole_field(y.x, y.y, y.z, p.dip_k, gx, gy, gz);
        Bx += gx;
        By += gy;
        Bz += gz;
    }
    double ux = p.u[i], uy = p.u[p.N + i], uz = p.u[2 * p.N + i];
    higuera_cary(ux, uy, uz, Ex, Ey, Ez, Bx, By, Bz, p.eps);
    p.u[i] = ux;
    p.u[p.N + i] = uy;
    p.u[2 * p.N + i] = uz;
    const double c = kC_LIGHT;
    double g = sqrt(1.0 + (ux * ux + uy * uy + uz * uz) / (c * c));
    double ig = 1.0 / g;
    // velocity records carry 1/(T_{k+1} - T_k) of their segment (0 for the
    // newest slot, which has no segment yet)
    const double3 vn = make_double3(ux * ig, uy * ig, uz * ig);
    const double ih = 1.0 / (p.t_next - p.t_now);
    p.vel.set_v(i * D + p.head, vn, ih);
    p.vel.set_a(i * D + p.head, vn, vn, ih);
    int nh = p.head + 1 == D ? 0 : p.head + 1;
    // the segment that ends at this slot has its final velocity; the one
    // that starts here has no acceleration before the next push
    const int ph = p.head == 0 ? D - 1 : p.head - 1;
    if (ph != nh)
        p.vel.set_a(i * D + ph, p.vel.v(i * D + ph), vn, p.vel.inv_h(i * D + ph));
    const double3 wn = make_double3(y.x + vn.x * p.dt, y.y + vn.y * p.dt, y.z + vn.z * p.dt);
    p.ring_w[i * D + nh] = make_double4(wn.x, wn.y, wn.z, 0.0);
    // guess data of the next pass
    const int oldest = nh + 1 == D ? 0 : nh + 1;
    const double4 wo = p.ring_w[i * D + oldest], ref = p.ring_w[p.head];
    const double3 r0 = make_double3(ref.x, ref.y, ref.z);
    p.lines[i] = chord_line(wn, make_double3(wo.x, wo.y, wo.z), c * (p.t_next - p.T[oldest]), D, r0);
    p.lines[p.N + i] = straight_line(wn, vn, p.dt_cfg, r0);
    p.vel.set_v(i * D + nh, vn, 0.0);
    p.vel.set_a(i * D + nh, vn, vn, 0.0);
}

// A step's merge and push in one launch: a block merges the six components
// of TG targets of the pair launch's order, NK at a time side by side, and
// pushes those particles, a thread each.
template <int TG, int SL, int NK>
__global__ __launch_bounds__(TG * SL * NK) void merge_push_kernel(PushParams p)
{
    __shared__ double2 red[6][SL][TG];
    const int t = threadIdx.x % TG;
    const int64_t a = (int64_t)blockIdx.x * TG + t;
    const bool first = blockIdx.x == 0 && threadIdx.x == 0;
    if (p.ad) {
        // Sec. 2.4: this step's dt from the pair kernel's reductions (the
        // same value in every thread); the clock lives in T[head]
        const double eta_min = __longlong_as_double((long long)p.ad[0]);
        const double v_max = sqrt(__longlong_as_double((long long)p.ad[1]));
        double dt = p.dt_max;
        if (v_max > 0.0 && eta_min < __longlong_as_double((long long)kPosInfBits))
            dt = fmin(p.dt_max, fmax(p.dt_min, p.c_dt * eta_min / v_max));
        p.dt = dt;
        p.eps = p.q * dt / (2.0 * p.m);
        p.t_now = p.T[p.head];
        p.t_next = p.t_now + dt;
        if (first) {
            p.ad_next[0] = kPosInfBits;
            p.ad_next[1] = 0ull;
            p.dt_out[0] = dt;
        }
    }
    for (int k = threadIdx.x / (TG * SL); k < 6; k += NK)
        merge_slice<TG, SL>(red[k], p.part, p.nsplit, p.N, k, a);
    __syncthreads();
    if (first)
        p.T[p.head + 1 == p.D ? 0 : p.head + 1] = p.t_next;
    for (int k = threadIdx.x / TG; k < 6; k += SL * NK)
        red[k][0][t].x = merge_slices<TG, SL>(red[k], t);
    __syncthreads();
    if (threadIdx.x >= TG || a >= p.N)
        return;
    double f[6];
#pragma unroll
    for (int k = 0; k < 6; ++k)
        f[k] = red[k][0][t].x;
    const int64_t i = p.order[a];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        p.E[k * p.N + i] = f[k];
        p.B[k * p.N + i] = f[3 + k];
    }
    push_particle(p, i, f[0], f[1], f[2], f[3], f[4], f[5]);
}

// Straight-line prior history: logical slot k = -(D-1)..0 (physical
// index k + D - 1) at T_k = t0 + k dt, w_k = r + v0 (k dt), v_k = v0.
__global__ void init_straight_kernel(double4 *ring_w, VelRing vel, double *T, const double *r,
                                     const double *u, int64_t N, int D, double t0, double dt)
{
    // Rounded exactly as a plain IEEE evaluation (no fused multiply-add),
    // so that the stored history is reproducible bit for bit on any host.
#pragma clang fp contract(off)
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= N * D)
        return;
    int64_t i = idx / D;
    int s = (int)(idx - i * D);
    const double c = kC_LIGHT;
    double ux = u[i], uy = u[N + i], uz = u[2 * N + i];
    double g = sqrt(1.0 + ((ux * ux + uy * uy) + uz * uz) / (c * c));
    double vx = ux / g, vy = uy / g, vz = uz / g;
    int64_t k = (int64_t)s - (D - 1);
    double kdt = (double)k * dt;
    ring_w[idx] = make_double4(r[i] + vx * kdt, r[N + i] + vy * kdt, r[2 * N + i] + vz * kdt, 0.0);
    double inv_h = s + 1 < D ? 1.0 / ((t0 + (double)(k + 1) * dt) - (t0 + kdt)) : 0.0;
    const double3 v = make_double3(vx, vy, vz);
    vel.set_v(idx, v, inv_h);
    vel.set_a(idx, v, v, inv_h);
    if (i == 0)
        T[s] = t0 + kdt;
}

// [ns][3][N] component-major history (oldest first) -> ring layout with
// logical slot s at physical slot s (head = D - 1).
__global__ void history_to_ring_kernel(const double *w, const double *v, const double *T, double4 *ring_w,
                                       VelRing vel, int64_t N, int D)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= N * D)
        return;
    int64_t i = idx / D;
    int64_t s = idx - i * D;
    const double *ws = w + s * 3 * N;
    const double *vs = v + s * 3 * N;
    ring_w[idx] = make_double4(ws[i], ws[N + i], ws[2 * N + i], 0.0);
    double inv_h = s + 1 < D ? 1.0 / (T[s + 1] - T[s]) : 0.0;
    const double3 v1 = make_double3(vs[i], vs[N + i], vs[2 * N + i]);
    const double *v2 = s + 1 < D ? vs + 3 * N : vs;
    vel.set_v(idx, v1, inv_h);
    vel.set_a(idx, v1, make_double3(v2[i], v2[N + i], v2[2 * N + i]), inv_h);
}

// Ring -> [D][3][N] oldest first (logical order).
__global__ void ring_to_history_kernel(const double4 *ring_w, VelRing vel, double *w, double *v,
                                       int64_t N, int D, int head)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= N * D)
        return;
    int64_t i = idx / D;
    int s = (int)(idx - i * D);          // logical slot, 0 = oldest
    int ph = head - (D - 1 - s);
    ph += ph < 0 ? D : 0;
    double4 a = ring_w[i * D + ph];
    double3 b = vel.v(i * D + ph);
    double *ws = w + (int64_t)s * 3 * N;
    double *vs = v + (int64_t)s * 3 * N;
    ws[i] = a.x;
    ws[N + i] = a.y;
    ws[2 * N + i] = a.z;
    vs[i] = b.x;
    vs[N + i] = b.y;
    vs[2 * N + i] = b.z;
}

__global__ void newest_positions_kernel(const double4 *ring_w, double *r, int64_t N, int D, int head)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N)
        return;
    double4 a = ring_w[i * D + head];
    r[i] = a.x;
    r[N + i] = a.y;
    r[2 * N + i] = a.z;
}

// Diagnostics partial sums per block: positions relative to particle 0's
// (so that offsets of Earth radii do not swamp millimetre spreads), their
// squares, and gamma - 1.  out[block][7] = {sx, sy, sz, sxx, syy, szz, sg}.
__global__ void diag_kernel(const double4 *ring_w, const double *u, int64_t N, int D, int head, double *out)
{
    __shared__ double red[7][kBlock];
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    double4 ref = ring_w[head];
    if (i < N) {
        double4 y = ring_w[i * D + head];
        double dx = y.x - ref.x, dy = y.y - ref.y, dz = y.z - ref.z;
        v[0] = dx;
        v[1] = dy;
        v[2] = dz;
        v[3] = dx * dx;
        v[4] = dy * dy;
        v[5] = dz * dz;
        const double c = kC_LIGHT;
        double u2 = (u[i] * u[i] + u[N + i] * u[N + i] + u[2 * N + i] * u[2 * N + i]) / (c * c);
        v[6] = u2 / (sqrt(1.0 + u2) + 1.0);  // gamma - 1 without cancellation
    }
    for (int k = 0; k < 7; ++k)
        red[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off)
            for (int k = 0; k < 7; ++k)
                red[k][threadIdx.x] += red[k][threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int k = 0; k < 7; ++k)
            out[blockIdx.x * 7 + k] = red[k][0];
}

// ---- Stage II: prescribed field only (Sec. 2.7) ---------------------------

// gamma / |B| of one particle, +inf where it sees no field.
__device__ inline double gyro_key(double4 y, double ux, double uy, double uz, double dip_k, int ext_field)
{
    if (ext_field != 1)
        return __longlong_as_double((long long)kPosInfBits);
    double bx, by, bz;
    dipole_field(y.x, y.y, y.z, dip_k, bx, by, bz);
    const double c = kC_LIGHT;
    double g = sqrt(1.0 + (ux * ux + uy * uy + uz * uz) / (c * c));
    double bm = sqrt(bx * bx + by * by + bz * bz);
    return bm > 0.0 ? g / bm : __longlong_as_double((long long)kPosInfBits);
}

// Block minimum of a positive double, folded into *slot with one atomic.
__device__ inline void block_min_to(double v, unsigned long long *slot)
{
    __shared__ double wmin[16];
    for (int off = 32; off > 0; off >>= 1)
        v = fmin(v, __shfl_xor(v, off));
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        wmin[w] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = wmin[0];
        for (int k = 1; k < (int)(blockDim.x >> 6); ++k)
            m = fmin(m, wmin[k]);
        atomicMin(slot, (unsigned long long)__double_as_longlong(m));
    }
}

// Positions of the newest slot -> compact Stage-II array; clears the three
// step slots and sets the clock.
__global__ void handoff_kernel(const double4 *ring_w, int D, int head, double4 *pos, int64_t N,
                               unsigned long long *key, double *t, double t_now)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) {
        double4 y = ring_w[i * D + head];
        pos[i] = make_double4(y.x, y.y, y.z, 0.0);
    }
    if (i == 0) {
        key[0] = key[1] = key[2] = kPosInfBits;
        t[0] = t_now;
    }
}

// The first step's minimum (slot 0) from the handed-off state.
__global__ void transport_key_kernel(const double4 *pos, const double *u, int64_t N, double dip_k, int ext_field,
                                     unsigned long long *key)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double k = __longlong_as_double((long long)kPosInfBits);
    if (i < N)
        k = gyro_key(pos[i], u[i], u[N + i], u[2 * N + i], dip_k, ext_field);
    block_min_to(k, key);
}

// One Stage-II step: E = 0, B = B_geo, Higuera-Cary, drift with the new
// velocity; then the next step's gamma / |B| at the new state.
__global__ void transport_kernel(TransportParams p)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int s0 = (int)(p.step % 3);
    const int s1 = s0 == 2 ? 0 : s0 + 1;
    const int s2 = s1 == 2 ? 0 : s1 + 1;
    const double kmin = __longlong_as_double((long long)p.key[s0]);
    double dt = p.dt_max;
    const double d = p.gyro_k * kmin;
    if (d < dt)
        dt = d;
    double knext = __longlong_as_double((long long)kPosInfBits);
    if (i < p.N) {
        double4 y = p.pos[i];
        double bx = 0.0, by = 0.0, bz = 0.0;
        if (p.ext_field == 1)
            dipole_field(y.x, y.y, y.z, p.dip_k, bx, by, bz);
        double ux = p.u[i], uy = p.u[p.N + i], uz = p.u[2 * p.N + i];
        higuera_cary(ux, uy, uz, 0.0, 0.0, 0.0, bx, by, bz, p.q_over_2m * dt);
        const double c = kC_LIGHT;
        double ig = 1.0 / sqrt(1.0 + (ux * ux + uy * uy + uz * uz) / (c * c));
        y = make_double4(y.x + ux * ig * dt, y.y + uy * ig * dt, y.z + uz * ig * dt, 0.0);
        p.pos[i] = y;
        p.u[i] = ux;
        p.u[p.N + i] = uy;
        p.u[2 * p.N + i] = uz;
        knext = gyro_key(y, ux, uy, uz, p.dip_k, p.ext_field);
    }
    block_min_to(knext, p.key + s1);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        p.key[s2] = kPosInfBits;
        p.t[0] += dt;
    }
}

// Step minima of a transport_steps_kernel launch: thread b < gridDim.x waits for
// block b's minimum of the step that `tag` (the sign bit, else clear in these
// positive doubles) and `slots` (even or odd steps) name; returns the smallest
// to every thread.  The wait is bounded: a thread that has polled `polls` times, or
// sees that another gave up, sets *fail, and the block gets a negative value.
__device__ inline double wait_for_minima(const unsigned long long *slots, unsigned long long tag,
                                         unsigned long long *fail, unsigned polls, double (*wmin)[4])
{
    double v = __longlong_as_double((long long)kPosInfBits);
    if (threadIdx.x < gridDim.x) {
        unsigned long long x;
        unsigned spins = 0, look = min(polls, 255u);  // a look beyond the slot every 256 polls
        while (((x = __hip_atomic_load(&slots[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 63) != tag) {
            if (__builtin_expect(++spins > look, 0)) {
                if (spins > polls || __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
                    atomicOr(fail, 1ull);
                    look = 0;
                    break;
                }
                look += 256;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        v = spins > look ? -1.0 : __longlong_as_double((long long)(x & ~(1ull << 63)));
    }
    const int w = threadIdx.x >> 6;
    if (w < kTransportBlocks / 64) {
        for (int off = 32; off > 0; off >>= 1)
            v = fmin(v, __shfl_xor(v, off));
        if ((threadIdx.x & 63) == 0)
            (*wmin)[w] = v;
    }
    __syncthreads();
    const int nw = min(kTransportBlocks, (int)blockDim.x) >> 6;
    v = (*wmin)[0];
    for (int k = 1; k < nw; ++k)
        v = fmin(v, (*wmin)[k]);
    return v;
}

// p.nsteps steps in one launch, one particle a thread, its state and its field
// (which the step's minimum and the next step's push share) in registers.  A step
// of transport_kernel is a launch's gap, the loads and a chain of about ten
// divisions and roots: 7 us at N = 65536, 17 at 262144.  Here a step's only
// exchange is its minimum: every block stores its own into its slot, with the
// step's parity in the sign, and reads all of them, one hop and no counter;
// slots are used by alternate steps, so a block that is a step ahead (it has
// read every block's previous minimum) overwrites none that is still read.
// 4.3 us a step at N = 65536, 6.2 at 262144 (of which about 2.4 are the chain; polls
// without a pause between them 0.5 more).  The launch is cooperative, so every
// block is resident.  A block whose wait gives up ends and writes nothing, and so
// does every block of a launch queued behind; the bunch then has no valid state.
__global__ __launch_bounds__(1024) void transport_steps_kernel(TransportParams p)
{
    __shared__ double wblock[2][16], wall[2][4];
    if (p.queued && __syncthreads_or(__hip_atomic_load(p.fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0))
        return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = i < p.N, first = i == 0;
    const double inf = __longlong_as_double((long long)kPosInfBits);
    const double c = kC_LIGHT;
    double4 y = make_double4(0.0, 0.0, 0.0, 0.0);
    double ux = 0.0, uy = 0.0, uz = 0.0, bx = 0.0, by = 0.0, bz = 0.0;
    if (live) {
        y = p.pos[i];
        ux = p.u[i];
        uy = p.u[p.N + i];
        uz = p.u[2 * p.N + i];
        if (p.ext_field == 1)
            dipole_field(y.x, y.y, y.z, p.dip_k, bx, by, bz);
    }
    double kmin = __longlong_as_double((long long)p.key[p.step % 3]), kold = kmin;
    double t = first ? p.t[0] : 0.0;
    for (int64_t k = 0; k < p.nsteps; ++k) {
        double dt = p.dt_max;
        const double d = p.gyro_k * kmin;
        if (d < dt)
            dt = d;
        t += dt;
        double v = inf;
        if (live) {
            higuera_cary(ux, uy, uz, 0.0, 0.0, 0.0, bx, by, bz, p.q_over_2m * dt);
            double ig = 1.0 / sqrt(1.0 + (ux * ux + uy * uy + uz * uz) / (c * c));
            y = make_double4(y.x + ux * ig * dt, y.y + uy * ig * dt, y.z + uz * ig * dt, 0.0);
            if (p.ext_field == 1) {
                dipole_field(y.x, y.y, y.z, p.dip_k, bx, by, bz);
                double g = sqrt(1.0 + (ux * ux + uy * uy + uz * uz) / (c * c));
                double bm = sqrt(bx * bx + by * by + bz * bz);
                v = bm > 0.0 ? g / bm : inf;
            }
        }
        for (int off = 32; off > 0; off >>= 1)
            v = fmin(v, __shfl_xor(v, off));
        const int par = (int)(k & 1);
        if ((threadIdx.x & 63) == 0)
            wblock[par][threadIdx.x >> 6] = v;
        __syncthreads();
        const int64_t s = p.sync_step + k;
        unsigned long long *slots = p.slots + (s & 1) * kTransportBlocks;
        const unsigned long long tag = (unsigned long long)(s >> 1 & 1);
        if (threadIdx.x == 0) {
            double m = fmin(inf, wblock[par][0]);
            for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
                m = fmin(m, wblock[par][w]);
            __hip_atomic_store(&slots[blockIdx.x], (unsigned long long)__double_as_longlong(m) | tag << 63,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        kold = kmin;
        kmin = wait_for_minima(slots, tag, p.fail, p.polls, &wall[par]);
        if (kmin < 0.0)
            return;
    }
    if (live) {
        p.pos[i] = y;
        p.u[i] = ux;
        p.u[p.N + i] = uy;
        p.u[2 * p.N + i] = uz;
    }
    if (first) {
        // as transport_kernel leaves them
        const int64_t last = p.step + p.nsteps - 1;
        p.key[last % 3] = (unsigned long long)__double_as_longlong(kold);
        p.key[(last + 1) % 3] = (unsigned long long)__double_as_longlong(kmin);
        p.key[(last + 2) % 3] = kPosInfBits;
        p.t[0] = t;
    }
}

// No step has gone through the slots yet: all carry the tag of the third step.
__global__ void transport_slots_kernel(unsigned long long *slots, unsigned long long *fail)
{
    slots[threadIdx.x] = kPosInfBits | 1ull << 63;
    if (threadIdx.x == 0)
        *fail = 0;
}

hipError_t launch_handoff(const double4 *ring_w, int D, int head, double4 *pos, const double *u, int64_t N,
                          double dip_k, int ext_field, unsigned long long *key, double *t, double t_now,
                          hipStream_t s)
{
    const unsigned nb = (unsigned)((N + 255) / 256);
    hipLaunchKernelGGL(handoff_kernel, dim3(nb), dim3(256), 0, s, ring_w, D, head, pos, N, key, t, t_now);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(transport_key_kernel, dim3(nb), dim3(256), 0, s, (const double4 *)pos, u, N, dip_k,
                       ext_field, key);
    return hipGetLastError();
}

hipError_t launch_transport_slots(const TransportParams &p, hipStream_t s)
{
    hipLaunchKernelGGL(transport_slots_kernel, dim3(1), dim3(2 * kTransportBlocks), 0, s, p.slots, p.fail);
    return hipGetLastError();
}

// p.nsteps steps on blocks of `threads` (at most kTransportBlocks of them, all
// resident).
hipError_t launch_transport_steps(const TransportParams &p, int threads, hipStream_t s)
{
    TransportParams arg = p;
    void *args[] = {&arg};
    return hipLaunchCooperativeKernel((const void *)transport_steps_kernel,
                                      dim3((unsigned)((p.N + threads - 1) / threads)), dim3((unsigned)threads), args, 0,
                                      s);
}

hipError_t launch_transport(const TransportParams &p, hipStream_t s)
{
    hipLaunchKernelGGL(transport_kernel, dim3((unsigned)((p.N + 255) / 256)), dim3(256), 0, s, p);
    return hipGetLastError();
}

// Targets of a merge up to which its blocks take 16 each.  Merge and push of a
// step, D = 64, us, 16 and 64 targets a block: N = 4096 9.6 and 15.5, 8192 11.9 and
// 15.5, 12288 21.5 and 22.2, 16384 19.6 and 17.8, 20480 32.0 and 28.4, 32768 36.5 and
// 32.3, 65536 75 and 55: equal within 2 us from 12288 to 16384.
constexpr int64_t kMergeSmall = 16384;

hipError_t launch_merge_fields(const double *part, int nsplit, int64_t m, double *E, double *B, int64_t stride,
                               hipStream_t s)
{
    if (m <= kMergeSmall)
        hipLaunchKernelGGL((merge_fields_kernel<16, 32>), dim3((unsigned)((m + 15) / 16), 6), dim3(512), 0, s, part,
                           nsplit, m, E, B, stride);
    else
        hipLaunchKernelGGL((merge_fields_kernel<64, 4>), dim3((unsigned)((m + 63) / 64), 6), dim3(256), 0, s, part,
                           nsplit, m, E, B, stride);
    return hipGetLastError();
}

// Merge of the self-field partials into E, B, and the push.
hipError_t launch_push(const PushParams &p, hipStream_t s)
{
    if (p.N <= kMergeSmall)
        hipLaunchKernelGGL((merge_push_kernel<16, 8, 6>), dim3((unsigned)((p.N + 15) / 16)), dim3(768), 0, s, p);
    else
        hipLaunchKernelGGL((merge_push_kernel<64, 4, 1>), dim3((unsigned)((p.N + 63) / 64)), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_init_straight(double4 *rw, VelRing vel, double *T, const double *r, const double *u, int64_t N,
                                int D, double t0, double dt, hipStream_t s)
{
    int64_t tot = N * D;
    hipLaunchKernelGGL(init_straight_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, rw, vel, T, r, u,
                       N, D, t0, dt);
    return hipGetLastError();
}

hipError_t launch_history_to_ring(const double *w, const double *v, const double *T, double4 *rw, VelRing vel,
                                  int64_t N, int D, hipStream_t s)
{
    int64_t tot = N * D;
    hipLaunchKernelGGL(history_to_ring_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, w, v, T, rw,
                       vel, N, D);
    return hipGetLastError();
}

hipError_t launch_ring_to_history(const double4 *rw, VelRing vel, double *w, double *v, int64_t N, int D,
                                  int head, hipStream_t s)
{
    int64_t tot = N * D;
    hipLaunchKernelGGL(ring_to_history_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, rw, vel, w, v,
                       N, D, head);
    return hipGetLastError();
}

hipError_t launch_newest_positions(const double4 *rw, double *r, int64_t N, int D, int head, hipStream_t s)
{
    hipLaunchKernelGGL(newest_positions_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, rw, r, N, D,
                       head);
    return hipGetLastError();
}

hipError_t launch_diag(const double4 *rw, const double *u, int64_t N, int D, int head, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(diag_kernel, dim3((unsigned)((N + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, rw, u, N, D,
                       head, out);
    return hipGetLastError();
}

}  // namespace empp
