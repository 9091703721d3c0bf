// HIP kernels (gfx950) of one DBaS-Log-MPPI iteration apart from the rollout
// (whose kernels are compiled per model, in mppi_rollout_<model>.hip, from
// the templates of mppi_device.hpp):
//   update kernel   -- one workgroup per four control rows (t, c).  Every
//                      workgroup merges the tile minima and normalisers
//                      itself (eq. control_update: rho = min S, eta), then
//                      one wave per row forms U*[t][c] = U[t][c] +
//                      sum_b f_b N_b[t][c] / eta, coalesced over tiles, and
//                      writes U* and the shifted warm start (Alg. 1 closing
//                      loop) into the other half of a double buffer, and u0*.
//   explore kernel  -- the noise-free rollout of U* and its barrier cost
//                      (Sec. IV-B eq. scaling factor), the next S_e.
//   the weights and Philox-word inspection kernels, and the host launchers.
#include "mppi_device.hpp"

#include <algorithm>

namespace dbas {
namespace {

// ---------------------------------------------------------------------------
// Update of control rows [row0, row0 + 4) of one controller, one wave per row.
// Every workgroup first merges the tile minima and normalisers itself
// (eq. control_update: rho = min_b rho_b, f_b = exp(-(rho_b - rho)/lambda),
// eta = sum_b f_b eta_b), then U*[t][c] = U[t][c] + sum_b f_b N_b[t][c] / eta,
// coalesced over tiles; it writes U*, the shifted warm start (Alg. 1 closing
// loop) into the other half of the double buffer and u0*; the workgroup of
// row 0 also records the iteration in the controller's state.
// host: what goes to the pinned host result block -- kHostNone: nothing;
// kHostPlain: u0, status and counter, seen by the host after the launch
// completes; kHostMark: the same, then the completion mark behind one
// system-scope fence, for a host thread that spins on the mark.
// plan, with the mark: every row also goes to the host, one 8-byte store of the
// value and the iteration (seq), which the host checks row by row -- so no
// workgroup waits for another and no fence is needed.  (One workgroup of 1024
// threads for all rows, publishing them before its mark, took 10.6 against
// 4.6 us at K=4096, T=50 and 16.4 against 5.1 at K=16384, T=100.)
// ---------------------------------------------------------------------------
enum HostOut { kHostNone = 0, kHostPlain = 1, kHostMark = 2 };

__device__ void update_rows(const DevParams& p, int row0, uint32_t parity, float* u0_dev, int32_t* status_dev,
                            int host, double* sf, double* slots, uint64_t* plan = nullptr, uint32_t seq = 0)
{
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid >> 6;
    const int T = p.T, nt = p.tiles;
    CtrlState* st = p.st;
    const float* Uin = p.U + (size_t)(parity & 1u) * T * kM;
    float* Uout = p.Unext ? p.Unext : p.U + (size_t)((parity + 1u) & 1u) * T * kM;
    const bool first = row0 == 0;

    // Every load that does not depend on the merge is issued first: this
    // wave's row of partN (its first kPre elements per lane), U_r, and, with
    // at most one tile per thread, the tile's scalars.
    constexpr int kPre = 8;
    const int r = row0 + wave;
    const bool has_row = r < 2 * T;
    const double* row = p.partN + (size_t)(has_row ? r : 0) * nt;
    double pre[kPre];
#pragma unroll
    for (int i = 0; i < kPre; ++i) pre[i] = (has_row && lane + i * kWave < nt) ? row[lane + i * kWave] : 0.0;
    const float u_in = has_row ? Uin[r] : 0.0f;
    // the state words the first workgroup updates at the end (the rollout
    // does not write them)
    uint64_t ctr = 0;
    uint32_t it0 = 0;
    if (first && tid == 0) {
        ctr = st->counter;
        it0 = st->iter;
    }
    HostResult* res = host != kHostNone ? p.res : nullptr;
    const bool one = nt <= kUpdBlock;
    double rb1 = INFINITY, eb1 = 0.0, fl1 = 0.0;
    if (one && tid < nt) {
        rb1 = p.rho_b[tid];
        eb1 = p.eta_b[tid];
        fl1 = (double)p.flag_b[tid];
    }

    double m = rb1;
    if (!one)
        for (int b = tid; b < nt; b += kUpdBlock) m = fmin(m, p.rho_b[b]);
    const double rho = block_min_d<kUpdWaves>(m, slots);
    double es = 0.0, n64 = 0.0;
    if (one) {
        if (tid < nt) {
            const double f = (isfinite(rho) && isfinite(rb1)) ? exp(-(rb1 - rho) / (double)p.lambda) : 0.0;
            sf[tid] = f;
            if (first) p.f_b[tid] = f;
            es = f * eb1;
            n64 = fl1;
        }
    } else {
        for (int b = tid; b < nt; b += kUpdBlock) {
            const double rb = p.rho_b[b];
            const double f = (isfinite(rho) && isfinite(rb)) ? exp(-(rb - rho) / (double)p.lambda) : 0.0;
            sf[b] = f;
            if (first) p.f_b[b] = f;
            es += f * p.eta_b[b];
            n64 += (double)p.flag_b[b];
        }
    }
    const double2 sums = block_sum_d2<kUpdWaves>(es, n64, slots);     // also publishes sf to the block
    const double eta = sums.x, n64s = sums.y;
    const bool ok = isfinite(rho) && isfinite(eta) && eta > 0.0;

    if (has_row) {
        float us;
        if (ok) {
            double a = 0.0;
#pragma unroll
            for (int i = 0; i < kPre; ++i)
                if (lane + i * kWave < nt) a += sf[lane + i * kWave] * pre[i];
            for (int b = lane + kPre * kWave; b < nt; b += kWave) a += sf[b] * row[b];
            a = wave_sum_d(a);
            us = (float)((double)u_in + a / eta);
        } else {
            us = u_in;
        }
        if (lane == 0) {
            p.Ustar[r] = us;
            if (plan)
                __hip_atomic_store(&plan[r], (uint64_t)seq << 32 | __float_as_uint(us), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            const int t = r >> 1;
            if (ok) {
                if (t >= 1) Uout[r - 2] = us;
                if (t == T - 1) Uout[r] = p.init_mode == MPPI_INIT_ZERO ? 0.0f : us;
            } else {
                Uout[r] = us;
            }
            if (t == 0) {
                if (u0_dev) u0_dev[r] = us;
                if (first) reinterpret_cast<float*>(slots)[2 * kUpdWaves * 2 + r] = us;   // for thread 0
            }
        }
    }
    if (first) {
        __syncthreads();                        // rows 0 and 1 (u0) are in LDS
        if (tid == 0) {
            const int status = ok ? MPPI_OK : MPPI_E_NUMERIC;
            st->last_counter = ctr;
            if (ok) st->counter = ctr + 1u;
            st->rho = rho;
            st->eta = eta;
            st->status = status;
            st->fp64_tiles = (int32_t)n64s;
            if (status_dev) *status_dev = status;
            const uint32_t it = it0 + 1u;
            st->iter = it;
            if (res) {
                const float* u0l = reinterpret_cast<const float*>(slots) + 2 * kUpdWaves * 2;
                res->u0[0] = u0l[0];
                res->u0[1] = u0l[1];
                res->status = status;
                res->counter = ctr;
                if (host == kHostMark) {
                    // u0, status and counter are this thread's own stores: one
                    // fence orders them before the mark
                    __threadfence_system();
                    res->seq = it;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Adaptive exploration (Sec. IV-B eq. scaling factor; closing loop of
// Algorithm 1), one workgroup per controller: U* is rolled out once without
// noise from x0 (one lane; inputs saturated inside f), the fused barrier of
// every pose is summed by one wave per pose, then one lane runs
// eq. barrier_update from beta_0 in FP64, forms C_B = sum_{t=1..T} R_B beta_t
// and sets the next iteration's S_e = mu ln(e + max(C_B, 0)).
// ---------------------------------------------------------------------------
constexpr int kExpBlock = 256;

template <int MODEL>
__device__ void explore_poses(const DevParams& p, const X0& xs, float4* pose)
{
    float th = xs.v[2], hw = Model<MODEL>::W ? xs.v[Model<MODEL>::W] : 0.0f;
    float q[2] = {0.0f, 0.0f}, v[2] = {xs.v[3], MODEL == MPPI_CAR ? xs.v[3] : xs.v[4]};
    float sth, cth;
    heading_sincos(th, sth, cth);
    pose[0] = make_float4(0.0f, 0.0f, cth, sth);
    for (int t = 0; t < p.T; ++t) {
        const float s0 = fminf(fmaxf(p.Ustar[2 * t], p.u_min[0]), p.u_max[0]);
        const float s1 = fminf(fmaxf(p.Ustar[2 * t + 1], p.u_min[1]), p.u_max[1]);
        float f0, f1;
        Model<MODEL>::inputs(p, s0, s1, f0, f1);
        const float y = Model<MODEL>::heading(p.dt, th, hw, f0, f1);
        Model<MODEL>::position(p, 0, q[0], v[0], f0, y, sth, cth);
        Model<MODEL>::position(p, 1, q[1], v[1], f0, y, sth, cth);
        heading_sincos(th, sth, cth);
        pose[t + 1] = make_float4(q[0], q[1], cth, sth);
    }
}

__device__ void explore_ctrl(const DevParams& p, const X0& xs, unsigned char* smem)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int T = p.T, J = p.J, P = p.P;
    float4* obs = reinterpret_cast<float4*>(smem);
    float4* pose = reinterpret_cast<float4*>(smem + (size_t)obstacle_slots(J) * 16);
    float* bv = reinterpret_cast<float*>(smem + (size_t)obstacle_slots(J) * 16 + (size_t)(T + 1) * 16);
    // the rollout's local frame, centred on the start position
    const double ox = (double)xs.v[0], oy = (double)xs.v[1];
    for (int j = tid; j < J; j += kExpBlock) {
        const double cx = (double)p.obs[3 * j], cy = (double)p.obs[3 * j + 1], r = (double)p.obs[3 * j + 2];
        obs[j] = make_float4((float)(cx - ox), (float)(cy - oy), (float)(-(r * r)), 0.0f);
    }
    float inv_res = 0.0f, offx = 0.0f, offy = 0.0f;
    const bool has_map = p.sdf != nullptr;
    if (has_map) {
        inv_res = (float)(1.0 / (double)p.map_res);
        offx = (float)((ox - (double)p.map_x0) / (double)p.map_res - 0.5);
        offy = (float)((oy - (double)p.map_y0) / (double)p.map_res - 0.5);
    }
    if (tid == 0) {
        switch (p.model) {
        case MPPI_QUAD6: explore_poses<MPPI_QUAD6>(p, xs, pose); break;
        case MPPI_QUAD5: explore_poses<MPPI_QUAD5>(p, xs, pose); break;
        default: explore_poses<MPPI_CAR>(p, xs, pose); break;
        }
    }
    __syncthreads();
    for (int t = wave; t <= T; t += kExpBlock / kWave) {
        const float4 q = pose[t];
        float acc = 0.0f;
        for (int idx = lane; idx < P * J; idx += kWave) {
            const int i = idx / J, j = idx - i * J;
            const float px = fmaf(p.shape[i][0], q.z, fmaf(-p.shape[i][1], q.w, q.x));
            const float py = fmaf(p.shape[i][0], q.w, fmaf(p.shape[i][1], q.z, q.y));
            const float4 o = obs[j];
            const float dx = px - o.x, dy = py - o.y;
            acc += barrier_rcp(fmaf(dx, dx, fmaf(dy, dy, o.z)), p.h_eps);
        }
        if (has_map && lane < P) {
            const float px = fmaf(p.shape[lane][0], q.z, fmaf(-p.shape[lane][1], q.w, q.x));
            const float py = fmaf(p.shape[lane][0], q.w, fmaf(p.shape[lane][1], q.z, q.y));
            acc += barrier_rcp(sdf_sample(p, fmaf(px, inv_res, offx), fmaf(py, inv_res, offy)),
                               p.h_eps);
        }
        acc = wave_sum_f(acc);
        if (lane == 0) bv[t] = acc;
    }
    __syncthreads();
    if (tid == 0) {
        CtrlState* st = p.st;
        const double g = (double)p.gamma_b, bd = (double)st->beta_d;
        double beta = (double)bv[0], cb = 0.0;
        for (int t = 1; t <= T; ++t) {
            beta = (double)bv[t] - g * (bd - beta);
            cb += (double)p.r_b * beta;
        }
        st->cost_b = (float)cb;
        st->S_e = (float)((double)p.explore_mu * log(2.718281828459045 + fmax(cb, 0.0)));
    }
}

__global__ __launch_bounds__(kUpdBlock) void k_update(DevParams p, StepArgs a)
{
    __shared__ double sf[kMaxTiles];
    __shared__ double slots[2 * kUpdWaves + 1];       // + u0 of rows 0 and 1
    update_rows(p, blockIdx.x * kUpdWaves, a.parity, a.u0_dev, a.status_dev, a.mark ? kHostMark : kHostNone, sf,
                slots, a.mark ? p.plan : nullptr, a.seq);
}

// One workgroup per (controller, four control rows) of the batch.
__global__ __launch_bounds__(kUpdBlock) void k_batch_update(const DevParams* __restrict__ ps,
                                                            const RowUnit* __restrict__ units,
                                                            const BatchIn* __restrict__ in, float* u0s)
{
    __shared__ double sf[kMaxTiles];
    __shared__ double slots[2 * kUpdWaves + 1];       // + u0 of rows 0 and 1
    const RowUnit ru = units[blockIdx.x];
    update_rows(ps[ru.ctrl], ru.row0, in[ru.ctrl].parity, u0s ? u0s + (size_t)ru.ctrl * kM : nullptr, nullptr,
                kHostPlain, sf, slots);
}

__global__ __launch_bounds__(kExpBlock) void k_explore(DevParams p, StepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    X0 xs;
#pragma unroll
    for (int i = 0; i < MPPI_NMAX + 2; ++i) xs.v[i] = a.x0_ptr ? (i < p.n ? a.x0_ptr[i] : 0.0f) : a.x0[i];
    xs.parity = a.parity;
    explore_ctrl(p, xs, smem);
}

// One workgroup per listed controller of a batch.
__global__ __launch_bounds__(kExpBlock) void k_batch_explore(const DevParams* __restrict__ ps,
                                                             const int32_t* __restrict__ ids,
                                                             const BatchIn* __restrict__ in)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int c = ids[blockIdx.x];
    X0 xs;
#pragma unroll
    for (int i = 0; i < MPPI_NMAX + 2; ++i) xs.v[i] = in[c].x0[i];
    xs.parity = in[c].parity;
    explore_ctrl(ps[c], xs, smem);
}

// The four-texel records of a costmap: record (i, j), 0 <= i < W-1,
// 0 <= j < H-1, holds the values at cell centres (i, j), (i+1, j), (i, j+1),
// (i+1, j+1).
__global__ __launch_bounds__(256) void k_sdf_cells(const float* __restrict__ sdf, int W, int H, float4* out)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= (W - 1) * (H - 1)) return;
    const int j = idx / (W - 1), i = idx - j * (W - 1);
    const float* r0 = sdf + (size_t)j * W + i;
    out[idx] = make_float4(r0[0], r0[1], r0[W], r0[W + 1]);
}

// Words from pinned host memory to the device, in stream order.
__global__ __launch_bounds__(256) void k_upload(uint32_t* __restrict__ dst, const uint32_t* __restrict__ src, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// w_k = e_k f_b(k) / eta: the weights the update used.
__global__ __launch_bounds__(256) void k_weights(DevParams p, double* w)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= p.K) return;
    const CtrlState* st = p.st;
    w[k] = st->status == MPPI_OK ? (double)p.e[k] * p.f_b[k / p.spt] / st->eta : 0.0;
}

__global__ __launch_bounds__(256) void k_philox_words(DevParams p, uint64_t counter, uint32_t* out)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= p.K * p.T) return;
    const int k = idx / p.T, t = idx - k * p.T;
    const uint4 r = philox4x32_10(make_uint4((uint32_t)k, (uint32_t)t, (uint32_t)counter, (uint32_t)(counter >> 32)),
                                  p.seed_lo, p.seed_hi);
    uint4* o = reinterpret_cast<uint4*>(out) + idx;
    *o = r;
}
}  // namespace

// ---------------------------------------------------------------------------
// The obstacles' far field (mppi_field.hpp).
// ---------------------------------------------------------------------------
namespace {

// Interpolation at the Padua points of degree n = 8 (Caliari, De Marchi and
// Vianello, "Bivariate polynomial interpolation on the square at new nodal
// sets", 2005; the explicit formula of Bos et al., 2006): the 45 points
// (cos(j pi/n), cos(k pi/(n+1))), j + k even, determine a polynomial of total
// degree n, whose Chebyshev coefficients are weighted sums of the values.
// fit[p][q]: what the value at point p adds to the monomial coefficient q;
// coefficient q = (8-l)(9-l)/2 + 8-l-k belongs to u^k v^l (rows of falling
// powers of v, each in falling powers of u: the order Horner's rule takes).
struct Padua {
    double x[kFieldCoefs], y[kFieldCoefs];
    double fit[kFieldCoefs][kFieldCoefs];
};

constexpr double cosine(double a)       // Taylor series, 0 <= a <= pi
{
    double t = 1.0, s = 1.0;
    for (int i = 1; i <= 16; ++i) {
        t *= -a * a / (double)((2 * i - 1) * (2 * i));
        s += t;
    }
    return s;
}

constexpr Padua make_padua()
{
    constexpr int n = kFieldDeg;
    constexpr double pi = 3.14159265358979323846;
    Padua r{};
    double mono[n + 1][n + 1] = {};     // T_i = sum_k mono[i][k] x^k
    mono[0][0] = 1.0;
    mono[1][1] = 1.0;
    for (int i = 2; i <= n; ++i)
        for (int k = 0; k <= i; ++k) mono[i][k] = (k > 0 ? 2.0 * mono[i - 1][k - 1] : 0.0) - mono[i - 2][k];
    int p = 0;
    for (int j = 0; j <= n; ++j)
        for (int k = 0; k <= n + 1; ++k) {
            if ((j + k) & 1) continue;
            const double x = cosine(j * pi / n), y = cosine(k * pi / (n + 1));
            const bool ex = j == 0 || j == n, ey = k == 0 || k == n + 1;
            const double w = (ex && ey ? 0.5 : ex || ey ? 1.0 : 2.0) / (double)(n * (n + 1));
            double tx[n + 1] = {1.0, x}, ty[n + 1] = {1.0, y};
            for (int i = 2; i <= n; ++i) {
                tx[i] = 2.0 * x * tx[i - 1] - tx[i - 2];
                ty[i] = 2.0 * y * ty[i - 1] - ty[i - 2];
            }
            r.x[p] = x;
            r.y[p] = y;
            for (int a = 0; a <= n; ++a)
                for (int b = 0; a + b <= n; ++b) {
                    const double g = w * (a ? 2.0 : 1.0) * (b ? 2.0 : 1.0) * (a == n ? 0.5 : 1.0) * tx[a] * ty[b];
                    for (int kk = a & 1; kk <= a; kk += 2)
                        for (int l = b & 1; l <= b; l += 2)
                            r.fit[p][(n - l) * (n - l + 1) / 2 + n - l - kk] += g * mono[a][kk] * mono[b][l];
                }
            ++p;
        }
    return r;
}

__device__ const Padua kPadua = make_padua();

// A polynomial at (u, v), FP64: rows of falling powers of v, nine slots a row
// in falling powers of u (the unused ones in front, zero).
constexpr int kFieldRow = kFieldDeg + 1;

__device__ __forceinline__ double field_eval_d(const double* c, double u, double v)
{
    double acc = 0.0;
#pragma unroll 1
    for (int i = 0; i < kFieldRow; ++i, c += kFieldRow) {
        double r = c[0];
#pragma unroll
        for (int k = 1; k < kFieldRow; ++k) r = fma(r, u, c[k]);
        acc = fma(acc, v, r);
    }
    return acc;
}

constexpr int kFieldBlock = 512;
constexpr int kFieldWaves = kFieldBlock / kWave;
// The thresholds a cell tries, and the one it takes when none holds.
constexpr int kKappas = 3;
__device__ constexpr float kKappa[kKappas + 1] = {3.25f, 4.0f, 4.75f, 6.0f};
constexpr float kFieldTol = 1.5e-7f;        // of the macro cell's and of the cell's far sums, each

// The relative error that an obstacle kappa half-widths off leaves.
__device__ __forceinline__ float field_error(float kappa) { return 8.0f * exp2f(-9.25f * log2f(kappa + 1.0f)); }

// Grid l of an obstacle set from its bounding box.
__device__ FieldLevel field_level(int l, double cx, double cy, double w, double hh, int J, float margin)
{
    // cells of 0.3 obstacle spacings: about five obstacles near a cell, and
    // no finer than the body they carry; twice and four times that outside
    const double want = fmax(0.3 * sqrt(w * hh / J), (double)margin);
    const int cap = l == 0 ? kFieldMacros0 : l == 1 ? kFieldMacros1 : kFieldMacros2;
    const int base = l == 0 ? 0 : l == 1 ? kFieldMacros0 : kFieldMacros0 + kFieldMacros1;
    // the box itself, and half and one and a half boxes around it
    const double pad = l == 0 ? want : (l == 1 ? 0.5 : 1.5) * fmax(w, hh);
    const double W = w + 2.0 * pad, H = hh + 2.0 * pad;
    double c = fmax(sqrt(W * H / (cap * kMacro * kMacro)), want * (1 << l));
    int mx = 1, my = 1;
    for (int i = 0; i < 200; ++i) {
        const double qx = ceil(W / (kMacro * c)), qy = ceil(H / (kMacro * c));
        if (qx * qy <= (double)cap) {
            mx = (int)qx;
            my = (int)qy;
            break;
        }
        c *= 1.04;
    }
    return FieldLevel{cx - 0.5 * mx * kMacro * c, cy - 0.5 * my * kMacro * c, c, mx * kMacro, my * kMacro,
                      base * kMacro * kMacro, 0};
}

// Terms of an obstacle at (x, y) from a cell's centre, for the choice of
// kappa: its edge's distance beyond the cell in half-widths (below every
// threshold where the cell's smallest h is below h_eps), and its term at the
// centre.
__device__ __forceinline__ float field_kappa(float x, float y, float r, float W, float h_eps, float& f)
{
    const float dx = fmaxf(fabsf(x) - W, 0.0f), dy = fmaxf(fabsf(y) - W, 0.0f);
    const float d2 = fmaf(dx, dx, dy * dy);
    f = __builtin_amdgcn_rcpf(fmaf(x, x, fmaf(y, y, -r * r)));
    return fmaf(-r, r, d2) >= h_eps ? (sqrtf(d2) - r) * __builtin_amdgcn_rcpf(W) : -1.0f;
}

// One workgroup per macro cell of 4 x 4 cells.  The obstacles far from the
// macro cell (at its own, four times larger, scale) enter one polynomial of
// it, which each of its cells takes over by its values at the cell's nodes, so
// a cell itself sums only the obstacles around its macro cell: about 40 of 400
// where every cell summing them all took eight times the work.
__global__ __launch_bounds__(kFieldBlock, 4) void k_field(const float* __restrict__ obs, int J, float margin, float h_eps,
                                                       FieldHeader* hdr, float* __restrict__ cells)
{
    // per obstacle: the macro-far ones, macro-centred (near ones: at infinity),
    // then in their place the macro-near ones (with r); the obstacles; the
    // macro-near list
    extern __shared__ __align__(16) unsigned char dyn[];
    float4* so = reinterpret_cast<float4*>(dyn);
    float4* sn = so;
    float3* sobs = reinterpret_cast<float3*>(dyn + (size_t)J * 16);
    uint16_t* snear = reinterpret_cast<uint16_t*>(dyn + (size_t)J * 28);
    __shared__ double sfit[kFieldCoefs * kFieldCoefs];
    __shared__ double sf[kFieldWaves][kFieldCoefs];     // node values
    __shared__ double sc[kFieldRow * kFieldRow];        // the macro cell's polynomial, in rows
    __shared__ float sred[kFieldWaves][8];
    __shared__ FieldHeader sh;
    __shared__ int snn;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // (the fit from LDS: read from memory where it is used, each of a cell's
    // 45 terms waited on it)
    for (int i = tid; i < kFieldCoefs * kFieldCoefs; i += kFieldBlock) sfit[i] = (&kPadua.fit[0][0])[i];
    const bool node = lane < kFieldCoefs;
    const int nq = node ? lane : 0;
    const double nx = kPadua.x[nq], ny = kPadua.y[nq];
    // the coefficient of lane q from the node values f
    auto coefficient = [&](const double* f) {
        double c = 0.0;
#pragma unroll 9
        for (int p = 0; p < kFieldCoefs; ++p) c = fma(sfit[p * kFieldCoefs + nq], f[p], c);
        return c;
    };
    // ---- the grids (every workgroup forms them alike) ----
    float b[4] = {INFINITY, INFINITY, INFINITY, INFINITY};      // min x, -max x, min y, -max y
    bool bad = false;
    for (int j = tid; j < J; j += kFieldBlock) {
        // (the walk squares r: a negative radius in device memory, which the
        // host cannot check, is its magnitude here too)
        const float x = obs[3 * j], y = obs[3 * j + 1], r = fabsf(obs[3 * j + 2]);
        sobs[j] = make_float3(x, y, r);
        bad |= !(fabsf(x) < 1e8f && fabsf(y) < 1e8f && r < 1e8f);
        b[0] = fminf(b[0], x);
        b[1] = fminf(b[1], -x);
        b[2] = fminf(b[2], y);
        b[3] = fminf(b[3], -y);
    }
    const bool wave_bad = __ballot(bad) != 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        for (int m = 32; m >= 1; m >>= 1) b[i] = fminf(b[i], __shfl_xor(b[i], m));
        if (lane == 0) sred[wave][i] = b[i];
    }
    if (lane == 0) sred[wave][4] = wave_bad ? 1.0f : 0.0f;
    __syncthreads();
    if (tid < kFieldLevels) {
        bool any = false;
        for (int w = 0; w < kFieldWaves; ++w) {
            for (int i = 0; i < 4; ++i) b[i] = fminf(b[i], sred[w][i]);
            any |= sred[w][4] != 0.0f;
        }
        const double w = fmax(-(double)b[1] - b[0], 1.0), hh = fmax(-(double)b[3] - b[2], 1.0);
        const bool valid = !any && fmax(w, hh) < 1e6;
        const double cx = valid ? 0.5 * ((double)b[0] - b[1]) : 0.0, cy = valid ? 0.5 * ((double)b[2] - b[3]) : 0.0;
        sh.level[tid] = field_level(tid, cx, cy, valid ? w : 1.0, valid ? hh : 1.0, J, margin);
        if (tid == 0) {
            sh.margin = margin;
            sh.J = valid ? J : 0;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && tid == 0) *hdr = sh;
    if (sh.J == 0) return;
    int l = 0, mi = blockIdx.x;
    if (mi >= kFieldMacros0) { mi -= kFieldMacros0; l = 1; }
    if (l == 1 && mi >= kFieldMacros1) { mi -= kFieldMacros1; l = 2; }
    const FieldLevel lv = sh.level[l];
    const int mxn = lv.nx / kMacro, myn = lv.ny / kMacro;
    if (mi >= mxn * myn) return;
    const int mx = mi % mxn, my = mi / mxn;
    const double mside = kMacro * lv.side;
    const double mcx = lv.x0 + (mx + 0.5) * mside, mcy = lv.y0 + (my + 0.5) * mside;
    if (l > 0) {
        // inside the finer grid no query comes here
        const FieldLevel f = sh.level[l - 1];
        const double e = 0.5 * mside + f.side;
        if (mcx - e > f.x0 && mcx + e < f.x0 + f.nx * f.side && mcy - e > f.y0 && mcy + e < f.y0 + f.ny * f.side) return;
    }
    const float MW = (float)(0.5 * mside) + margin;
    // the smallest kappa at which the far obstacles' errors stay below the
    // tolerance, from the sums over the thresholds and the far sum
    auto choose = [&](const float* err, const float* far) {
        float k = kKappa[kKappas];
        for (int i = kKappas - 1; i >= 0; --i)
            if (err[i] <= kFieldTol * far[i]) k = kKappa[i];
        return k;
    };
    auto add_errors = [&](float k, float f, float (&err)[kKappas], float (&far)[kKappas]) {
        const float fe = f * field_error(k);
#pragma unroll
        for (int i = 0; i < kKappas; ++i) {
            err[i] += k >= kKappa[i] ? fe : 0.0f;
            far[i] += k >= kKappa[i] ? f : 0.0f;
        }
    };
    // ---- macro cell: choose kappa, split the obstacles ----
    float err[kKappas] = {}, far[kKappas] = {};
    for (int j = tid; j < J; j += kFieldBlock) {
        const float3 o = sobs[j];
        const float x = (float)((double)o.x - mcx), y = (float)((double)o.y - mcy);
        float f;
        const float k = field_kappa(x, y, o.z, MW, h_eps, f);
        add_errors(k, f, err, far);
    }
    __shared__ float skap[kFieldWaves][2 * kKappas];
#pragma unroll
    for (int i = 0; i < kKappas; ++i) {
        err[i] = wave_sum_f(err[i]);
        far[i] = wave_sum_f(far[i]);
        if (lane == 0) {
            skap[wave][i] = err[i];
            skap[wave][kKappas + i] = far[i];
        }
    }
    __syncthreads();
    for (int i = 0; i < kKappas; ++i) {
        err[i] = far[i] = 0.0f;
        for (int w = 0; w < kFieldWaves; ++w) {
            err[i] += skap[w][i];
            far[i] += skap[w][kKappas + i];
        }
    }
    const float mk = choose(err, far);
    const float4 away = make_float4(1e18f, 0.0f, 0.0f, 0.0f);       // 1/h = 1e-36
    for (int j = tid; j < J; j += kFieldBlock) {
        const float3 o = sobs[j];
        const float x = (float)((double)o.x - mcx), y = (float)((double)o.y - mcy), r = o.z;
        float f;
        so[j] = field_kappa(x, y, r, MW, h_eps, f) >= mk ? make_float4(x, y, -r * r, 0.0f) : away;
    }
    __syncthreads();
    if (wave == 0) {
        int n = 0;
        for (int j0 = 0; j0 < J; j0 += kWave) {
            const int j = j0 + lane;
            const bool near = j < J && so[j].x == 1e18f;
            const uint64_t m = __ballot(near);
            if (near) snear[n + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)j;
            n += __popcll(m);
        }
        if (lane == 0) snn = n;
    }
    // ---- macro polynomial: a node per lane, the obstacles shared out to the waves ----
    // the sum of 1/h over n obstacles at (x, y): FP32 terms, added up in FP64
    // by eights
    auto node_sum = [&](const float4* o, int n, float x, float y) {
        double s = 0.0;
        int j = 0;
        for (; j + 8 <= n; j += 8) {
            float a = 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float4 c = o[j + i];
                const float ex = x - c.x, ey = y - c.y;
                a += __builtin_amdgcn_rcpf(fmaf(ex, ex, fmaf(ey, ey, c.z)));
            }
            s += (double)a;
        }
        for (; j < n; ++j) {
            const float4 c = o[j];
            const float ex = x - c.x, ey = y - c.y;
            s += (double)__builtin_amdgcn_rcpf(fmaf(ex, ex, fmaf(ey, ey, c.z)));
        }
        return s;
    };
    {
        const int q = (J + kFieldWaves - 1) / kFieldWaves, j0 = min(wave * q, J);
        const double s = node_sum(so + j0, min(q, J - j0), (float)nx * MW, (float)ny * MW);
        if (node) sf[wave][lane] = s;
    }
    __syncthreads();
    if (tid < kFieldCoefs) {
        double v = sf[0][tid];
        for (int w = 1; w < kFieldWaves; ++w) v += sf[w][tid];
        sf[0][tid] = v;
    }
    if (wave == 0) {
        wave_fence();
        // coefficient q of row i lies (i+1)(i+2)/2 - 1 - q before the row's end
        int i = 0;
        while ((i + 1) * (i + 2) / 2 <= nq) ++i;
        for (int k = lane; k < kFieldRow * kFieldRow; k += kWave) sc[k] = 0.0;
        wave_fence();
        if (node) sc[i * kFieldRow + kFieldDeg + nq - ((i + 1) * (i + 2) / 2 - 1)] = coefficient(sf[0]);
    }
    const int nn = snn;
    for (int i = tid; i < nn; i += kFieldBlock) {
        const float3 o = sobs[snear[i]];
        sn[i] = make_float4((float)((double)o.x - mcx), (float)((double)o.y - mcy), -o.z * o.z, o.z);
    }
    __syncthreads();
    // ---- the macro cell's 16 cells, two per wave at once (one LDS read of an
    // obstacle serves both: the reads bound the sums) ----
    constexpr int C = kMacro * kMacro / kFieldWaves;
    const float W = (float)(0.5 * lv.side) + margin, iMW = 1.0f / MW;
    float cx[C], cy[C], ck[C];          // centres from the macro cell's; the chosen kappas
    double v[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int ci = wave * C + c;
        cx[c] = (float)((ci % kMacro - 0.5 * (kMacro - 1)) * lv.side);
        cy[c] = (float)((ci / kMacro - 0.5 * (kMacro - 1)) * lv.side);
        v[c] = field_eval_d(sc, (double)(fmaf((float)nx, W, cx[c]) * iMW), (double)(fmaf((float)ny, W, cy[c]) * iMW));
        ck[c] = kKappa[kKappas];
    }
    // (around a large set the outer grids' cells take the widest kappa: the
    // choice would cost as much as the sum)
    if (nn <= 4 * kWave) {
        float e[C][kKappas] = {}, fr[C][kKappas] = {};
        for (int i0 = lane; i0 < nn; i0 += kWave) {
            const float4 o = sn[i0];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                float f;
                const float k = field_kappa(o.x - cx[c], o.y - cy[c], o.w, W, h_eps, f);
                add_errors(k, f, e[c], fr[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            // (the macro-far part: its value at the first node will do)
            const float macro = fmaxf(__shfl((float)v[c], 0), 0.0f);
#pragma unroll
            for (int i = 0; i < kKappas; ++i) {
                e[c][i] = wave_sum_f(e[c][i]);
                fr[c][i] = wave_sum_f(fr[c][i]) + macro;
            }
            ck[c] = choose(e[c], fr[c]);
        }
    }
    float px[C], py[C];                 // this lane's node of either cell
    int cnt[C];
    float* rec[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int ci = wave * C + c, ix = mx * kMacro + ci % kMacro, iy = my * kMacro + ci / kMacro;
        rec[c] = cells + (size_t)(lv.base + iy * lv.nx + ix) * kFieldWords;
        px[c] = fmaf((float)nx, W, cx[c]);
        py[c] = fmaf((float)ny, W, cy[c]);
        cnt[c] = 0;
    }
    for (int i0 = 0; i0 < nn; i0 += kWave) {
        const int n = min(kWave, nn - i0);
        uint64_t far_of[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            bool near = false;
            if (lane < n) {
                const float4 o = sn[i0 + lane];
                float f;
                near = !(field_kappa(o.x - cx[c], o.y - cy[c], o.w, W, h_eps, f) >= ck[c]);
            }
            const uint64_t m = __ballot(near);
            const int at = cnt[c] + __popcll(m & ((1ull << lane) - 1ull));
            if (near && at < kFieldNear) reinterpret_cast<uint16_t*>(rec[c] + kFieldCoefs + 1)[at] = snear[i0 + lane];
            cnt[c] += __popcll(m);
            far_of[c] = ~m;
        }
        // FP32 terms, added up in FP64 by eights
        for (int j = 0; j < n; j += 8) {
            float a[C] = {};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (j + i < n) {
                    const float4 o = sn[i0 + j + i];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const float ex = px[c] - o.x, ey = py[c] - o.y;
                        const float f = __builtin_amdgcn_rcpf(fmaf(ex, ex, fmaf(ey, ey, o.z)));
                        a[c] += (far_of[c] >> (j + i)) & 1 ? f : 0.0f;
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < C; ++c) v[c] += (double)a[c];
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (node) sf[wave][lane] = v[c];
        wave_fence();
        if (node) rec[c][lane] = (float)coefficient(sf[wave]);
        if (lane == 0) rec[c][kFieldCoefs] = __int_as_float(cnt[c] <= kFieldNear ? cnt[c] : kFieldFull);
        wave_fence();
    }
}

}  // namespace

hipError_t launch_field(const float* d_obs, int J, float margin, float h_eps, void* d_field, hipStream_t s)
{
    if (J < 1 || J > MPPI_JMAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_field, dim3(kFieldMacros), dim3(kFieldBlock), ((size_t)J * 30 + 15) & ~(size_t)15, s, d_obs, J, margin,
                       h_eps, static_cast<FieldHeader*>(d_field),
                       reinterpret_cast<float*>(static_cast<char*>(d_field) + 256));
    return hipGetLastError();
}

bool tile_samples_supported(int S) { return S >= 16 && S <= kMaxTile && (S & (S - 1)) == 0; }

hipError_t launch_rollout(const DevParams& p0, const StepArgs& a, hipStream_t s)
{
    DevParams p = p0;
    if (!tile_samples_supported(p.spt)) return hipErrorInvalidValue;
    set_splits(p);
    const size_t lds = tile_lds_bytes(p.J, p.T, p.n, p.spt);
    switch (p.model) {
    case MPPI_QUAD6: return launch_rollout_quad6(p, a, lds, s);
    case MPPI_QUAD5: return launch_rollout_quad5(p, a, lds, s);
    case MPPI_CAR: return launch_rollout_car(p, a, lds, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_update(const DevParams& p, const StepArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(k_update, dim3((2 * p.T + kUpdWaves - 1) / kUpdWaves), dim3(kUpdBlock), 0, s, p, a);
    return hipGetLastError();
}

namespace {

BatchRolloutKernel batch_rollout_kernel(int group)
{
    const int key = group % kBatchKeys;
    switch (group / kBatchKeys) {
    case MPPI_QUAD6: return batch_rollout_kernel_quad6(key);
    case MPPI_QUAD5: return batch_rollout_kernel_quad5(key);
    default: return batch_rollout_kernel_car(key);
    }
}

}  // namespace

UnitGroups group_units(std::vector<BatchWork>& work, BatchUnit* out)
{
    std::stable_sort(work.begin(), work.end(), [](const BatchWork& a, const BatchWork& b) {
        return a.group != b.group ? a.group < b.group : a.cost > b.cost;
    });
    UnitGroups g{};
    for (int m = 0; m < kBatchGroups; ++m) g.begin[m] = -1;
    for (size_t i = 0; i < work.size(); ++i) {
        const int m = work[i].group;
        if (g.begin[m] < 0) g.begin[m] = (int)i;
        ++g.count[m];
        g.work[m] += work[i].cost;
        if (work[i].lds > g.lds[m]) g.lds[m] = work[i].lds;
        out[i] = work[i].unit;
    }
    for (int m = 0; m < kBatchGroups; ++m)
        if (g.begin[m] < 0) g.begin[m] = 0;
    return g;
}

hipError_t launch_batch_rollouts(const DevParams* d_params, const BatchUnit* d_units, const UnitGroups& g,
                                 const BatchIn* d_in, uint32_t* d_queue, int cus, hipStream_t s)
{
    int order[kBatchGroups];
    for (int i = 0; i < kBatchGroups; ++i) order[i] = i;
    std::stable_sort(order, order + kBatchGroups, [&](int a, int b) { return g.work[a] > g.work[b]; });
    for (int i = 0; i < kBatchGroups; ++i) {
        const int m = order[i];
        if (g.count[m] == 0) continue;
        const int grid = std::max(1, std::min(g.count[m], cus * batch_rollout_blocks_per_cu(m, g.lds[m])));
        hipLaunchKernelGGL(batch_rollout_kernel(m), dim3(grid), dim3(kRollBlock), g.lds[m], s, d_params,
                           d_units + g.begin[m], g.count[m], d_in, d_queue + 2 * m);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_batch_update(const DevParams* d_params, const RowUnit* d_units, int nunits, const BatchIn* d_in,
                               float* d_u0s, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_update, dim3(nunits), dim3(kUpdBlock), 0, s, d_params, d_units, d_in, d_u0s);
    return hipGetLastError();
}

hipError_t launch_explore(const DevParams& p, const StepArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(k_explore, dim3(1), dim3(kExpBlock), explore_lds_bytes(p.J, p.T), s, p, a);
    return hipGetLastError();
}

hipError_t launch_batch_explore(const DevParams* d_params, const int32_t* d_ids, int n, const BatchIn* d_in,
                                size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_explore, dim3(n), dim3(kExpBlock), lds, s, d_params, d_ids, d_in);
    return hipGetLastError();
}

hipError_t launch_upload(void* dst, const void* src, size_t words, hipStream_t s)
{
    hipLaunchKernelGGL(k_upload, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, static_cast<uint32_t*>(dst),
                       static_cast<const uint32_t*>(src), (int)words);
    return hipGetLastError();
}

hipError_t launch_weights(const DevParams& p, double* d_w, hipStream_t s)
{
    hipLaunchKernelGGL(k_weights, dim3((p.K + 255) / 256), dim3(256), 0, s, p, d_w);
    return hipGetLastError();
}

hipError_t launch_sdf_cells(const float* sdf, int W, int H, float4* out, hipStream_t s)
{
    const int n = (W - 1) * (H - 1);
    hipLaunchKernelGGL(k_sdf_cells, dim3((n + 255) / 256), dim3(256), 0, s, sdf, W, H, out);
    return hipGetLastError();
}

hipError_t launch_philox_words(const DevParams& p, uint64_t counter, uint32_t* d_words, hipStream_t s)
{
    const int n = p.K * p.T;
    hipLaunchKernelGGL(k_philox_words, dim3((n + 255) / 256), dim3(256), 0, s, p, counter, d_words);
    return hipGetLastError();
}

int batch_group(const DevParams& p) { return p.model * kBatchKeys + tile_key(p); }

int batch_rollout_blocks_per_cu(int group, size_t lds)
{
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, batch_rollout_kernel(group), kRollBlock, lds) !=
        hipSuccess)
        return 1;
    return blocks > 0 ? blocks : 1;
}

}  // namespace dbas
