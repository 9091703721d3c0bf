// Device code of the DBaS-Log-MPPI rollout (gfx950), shared by the kernel
// translation units: helpers, the models, the rollout tile and the rollout
// kernel templates (standalone and batched).  Everything has internal
// linkage; each unit instantiates what it launches.
//
//   rollout kernel  -- one workgroup per tile of S samples.  The horizon is
//                      cut into as few chunks as LDS allows (mostly one); per
//                      chunk the workgroup runs these phases:
//                       - inputs: Philox4x32-10 normal x log-normal noise
//                         (Sec. IV-C) for every (step, sample), turned into the
//                         state-independent terms (saturated inputs, their
//                         model terms) in LDS; the control cost of Alg. 1;
//                       - headings: one lane per sample integrates the heading
//                         (and what drives it), the first half of eq. veh_dyn;
//                       - their sines and cosines, every item in parallel;
//                       - positions: one lane per sample and axis integrates
//                         velocity and position;
//                       - the tracking cost, every item in parallel;
//                       - poses: every (step, sample) is split over lanes that
//                         each take a range of obstacles (LDS), and the costmap
//                         -- the bulk of the work, no dependence between items;
//                       - barrier state: one lane per sample runs the
//                         recursion of eq. barrier_update (Alg. 1, eq.
//                         cost-to-go_bas).
//                      Only what depends on the step before is sequential: the
//                      recurrences are a few operations a step, and everything
//                      else (sines, costs, barriers) runs on all lanes.
//                      The tile then forms its own min-shifted exponentials
//                      and the tile sums eta_b = sum e_k and N_b[t][c] =
//                      sum e_k du_k.  Tiles never wait for one another.
// Positions are handled in a frame centred on the iteration's start position
// (obstacles, reference and costmap offset are translated once in FP64), so
// FP32 rounding is relative to the rollout's extent, not the world's.
#pragma once

#include "mppi_field.hpp"
#include "mppi_internal.hpp"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace dbas {
namespace {

// ---------------------------------------------------------------------------
// Counter-based generator: Philox4x32-10 (Salmon et al., SC'11).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
        const uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
        c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// 23 high bits centred in their cell: ((r >> 9) + 1/2) 2^-23, exact in FP32.
__device__ __forceinline__ float word_to_uniform(uint32_t r)
{
    return fmaf((float)(r >> 9), 0x1p-23f, 0x1p-24f);
}

// Normal x log-normal pair for inputs (0, 1) from one Philox block: Box-Muller
// normals n from words (0, 1), z from words (2, 3);
// du_c = sqrt(S_e) sigma_c n_c exp(mu_ln + sigma_ln z_c), or with `normal`
// (Vanilla MPPI's law) the normal part sqrt(S_e) sigma_c n_c alone.
__device__ __forceinline__ float2 nln_pair(uint4 r, float scale0, float scale1, float mu_ln, float sigma_ln,
                                           bool normal)
{
    const float u0 = word_to_uniform(r.x), u1 = word_to_uniform(r.y);
    const float rn = sqrtf(-2.0f * logf(u0));
    float sn, cn;
    sincospif(2.0f * u1, &sn, &cn);
    float2 o;
    o.x = scale0 * (rn * cn);
    o.y = scale1 * (rn * sn);
    if (!normal) {
        const float u2 = word_to_uniform(r.z), u3 = word_to_uniform(r.w);
        const float rz = sqrtf(-2.0f * logf(u2));
        float sz, cz;
        sincospif(2.0f * u3, &sz, &cz);
        o.x *= expf(fmaf(sigma_ln, rz * cz, mu_ln));
        o.y *= expf(fmaf(sigma_ln, rz * sz, mu_ln));
    }
    return o;
}

// sin and cos of an angle (a heading, a steering angle).  Cody-Waite
// reduction by pi/2 (three-part split of pi/2, each product exact inside an
// FMA) to |r| <= pi/4, then the Taylor series of sin to r^9 and of cos to
// r^10 (truncation < 3e-9 on |r| <= pi/4, below half an FP32 ulp), and the
// quadrant's swap and signs.  Angles beyond 4096 quarter turns fall back to
// the library routine.
__device__ __forceinline__ void heading_sincos(float x, float& s, float& c)
{
    const float k = rintf(x * 0.63661975f);
    if (fabsf(k) > 4096.0f) {
        sincosf(x, &s, &c);
        return;
    }
    float r = fmaf(-k, 1.5707963705062866f, x);
    r = fmaf(-k, -4.371138828673793e-08f, r);
    r = fmaf(-k, -1.7151245100058819e-15f, r);
    const float r2 = r * r;
    const float ps = r2 * fmaf(r2, fmaf(r2, fmaf(r2, 2.7557319e-06f, -1.9841270e-04f), 8.3333333e-03f),
                               -1.6666667e-01f);
    const float sr = fmaf(r, ps, r);
    const float pc = fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, -2.7557319e-07f, 2.4801587e-05f), -1.3888889e-03f),
                                             4.1666667e-02f), -0.5f), 1.0f);
    const int q = (int)k & 3;
    const float a = (q & 1) ? pc : sr;
    const float b = (q & 1) ? sr : pc;
    s = (q & 2) ? -a : a;
    c = ((q + 1) & 2) ? -b : b;
}

// ---------------------------------------------------------------------------
// Reductions.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum_f(float v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    return v;
}

__device__ __forceinline__ double wave_sum_d(double v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    return v;
}

__device__ __forceinline__ double wave_min_d(double v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmin(v, __shfl_xor(v, m));
    return v;
}

// Block reductions over NW waves; every thread gets the result.  slots
// holds at least NW doubles.
template <int NW>
__device__ __forceinline__ double block_min_d(double v, double* slots)
{
    v = wave_min_d(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) slots[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = slots[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) r = fmin(r, slots[i]);
    return r;
}

template <int NW>
__device__ __forceinline__ double block_sum_d(double v, double* slots)
{
    v = wave_sum_d(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) slots[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = slots[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) r += slots[i];
    return r;
}

// two sums with one pair of barriers; slots holds at least 2 NW doubles
template <int NW>
__device__ __forceinline__ double2 block_sum_d2(double a, double b, double* slots)
{
    a = wave_sum_d(a);
    b = wave_sum_d(b);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        slots[threadIdx.x >> 6] = a;
        slots[NW + (threadIdx.x >> 6)] = b;
    }
    __syncthreads();
    double ra = slots[0], rb = slots[NW];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
        ra += slots[i];
        rb += slots[NW + i];
    }
    return make_double2(ra, rb);
}

template <int NW>
__device__ __forceinline__ float block_sum_f(float v, double* slots)
{
    v = wave_sum_f(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) slots[threadIdx.x >> 6] = (double)v;
    __syncthreads();
    float r = (float)slots[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) r += (float)slots[i];
    return r;
}

// A value that is the same on every lane, moved to a scalar register.
__device__ __forceinline__ float uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Workgroup barrier that orders LDS accesses only: global stores issued
// before it may still be in flight after it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------
// Barrier terms.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float barrier_rcp(float h, float eps)
{
    return __builtin_amdgcn_rcpf(fmaxf(h, eps));
}

// h clamped to [eps, kHMax]: the lower end is the barrier's own cap
// B = 1/max(h, eps); the upper end (h = 1e9 m^2, 31 km) keeps the products of
// four clamped values below the FP32 range while changing B by < 1e-9.
constexpr float kHMax = 1e9f;

__device__ __forceinline__ float clamp_h(float h, float eps)
{
    return __builtin_amdgcn_fmed3f(h, eps, kHMax);
}

// sum_i 1/h_i for N clamped values, taken four at a time as one fraction
// ((a+b)cd + (c+d)ab) / (abcd) -- exact up to rounding, all terms positive,
// one reciprocal per four -- alternating between two accumulators.
template <int N>
__device__ __forceinline__ void reciprocal_sum(const float* h, float& acc, float& acc2)
{
    int k = 0;
#pragma unroll
    for (int i = 0; i + 4 <= N; i += 4, ++k) {
        const float ab = h[i] * h[i + 1], cd = h[i + 2] * h[i + 3];
        const float num = fmaf(h[i] + h[i + 1], cd, (h[i + 2] + h[i + 3]) * ab);
        float& a = (k & 1) ? acc2 : acc;
        a = fmaf(num, __builtin_amdgcn_rcpf(ab * cd), a);
    }
    constexpr int r = N % 4;
    constexpr int i = N - r;
    float& a = (k & 1) ? acc2 : acc;
    if constexpr (r == 3) {
        const float ab = h[i] * h[i + 1];
        a = fmaf(fmaf(h[i] + h[i + 1], h[i + 2], ab), __builtin_amdgcn_rcpf(ab * h[i + 2]), a);
    } else if constexpr (r == 2) {
        a = fmaf(h[i] + h[i + 1], __builtin_amdgcn_rcpf(h[i] * h[i + 1]), a);
    } else if constexpr (r == 1) {
        a += __builtin_amdgcn_rcpf(h[i]);
    }
}

// The same of the first n >= 1 of four (the rest are not read): as one fraction
// with the absent values 1 and their numerators 0.
__device__ __forceinline__ float reciprocal_head(const float (&h)[4], int n)
{
    const float h1 = n > 1 ? h[1] : 1.0f, h2 = n > 2 ? h[2] : 1.0f, h3 = n > 3 ? h[3] : 1.0f;
    const float ab = h[0] * h1, cd = h2 * h3;
    const float na = n > 1 ? h[0] + h1 : 1.0f, nc = n > 3 ? h2 + h3 : n > 2 ? 1.0f : 0.0f;
    return fmaf(na, cd, nc * ab) * __builtin_amdgcn_rcpf(ab * cd);
}

// sum_i 1/h_i of N clamped values as a value (the clamped form of the layout
// bodies' obstacles that leave the pair-fraction form).
template <int N>
__device__ __forceinline__ float reciprocal_total(const float* h)
{
    float a = 0.0f, b = 0.0f;
    reciprocal_sum<N>(h, a, b);
    return a + b;
}

// Bilinear costmap sample between cell centres, clamped to the edge cells.
// (gx, gy) are continuous cell coordinates; any float input stays in bounds.
// With the four-texel layout (sdf4: for every square between four cell
// centres, its four values in one 16-byte record) a sample is one load
// instead of four scattered ones; the arithmetic, and so the result, is the
// same.
__device__ __forceinline__ float sdf_sample(const DevParams& p, float gx, float gy)
{
    const int W = p.map_w, H = p.map_h;
    gx = fminf(fmaxf(gx, 0.0f), (float)(W - 1));
    gy = fminf(fmaxf(gy, 0.0f), (float)(H - 1));
    const int i0 = min((int)floorf(gx), W - 2);
    const int j0 = min((int)floorf(gy), H - 2);
    const float fx = gx - (float)i0, fy = gy - (float)j0;
    float s00, s01, s10, s11;
    if (p.sdf4) {
        const float4 c = p.sdf4[(size_t)j0 * (W - 1) + i0];
        s00 = c.x;
        s01 = c.y;
        s10 = c.z;
        s11 = c.w;
    } else {
        const float* r0 = p.sdf + (size_t)j0 * W + i0;
        const float* r1 = r0 + W;
        s00 = r0[0];
        s01 = r0[1];
        s10 = r1[0];
        s11 = r1[1];
    }
    const float top = fmaf(fx, s01 - s00, s00);
    const float bot = fmaf(fx, s11 - s10, s10);
    return fmaf(fy, bot - top, top);
}

// ---------------------------------------------------------------------------
// Models (explicit Euler, inputs saturated inside f).  inputs() turns the
// saturated controls into the model's state-independent terms (f0, f1).  A
// step splits into the heading, which follows only from the inputs (and, for
// the vehicle, the speed they drive), and the position along each axis, which
// needs the sine and cosine of the *old* heading:
//   heading(th, w, f0, f1): the new heading th and its companion w (QUAD6:
//     the turn rate; CAR: the speed; QUAD5: none); returns the word kept
//     beside f0 for the position (CAR: the new speed, QUAD5: f1);
//   position(axis, q, v, f0, y, sn, cs): the new position q and velocity v
//     along axis 0 or 1 (CAR: v is the speed on both).
// ---------------------------------------------------------------------------
template <int MODEL> struct Model;

template <> struct Model<MPPI_QUAD6> {
    static constexpr int NS = 6;
    static constexpr int W = 5;      // state index of the heading's companion (0: none)
    // state (x, z, theta, vx, vz, omega); inputs: rotor thrust deviations from
    // hover.  f0 = (F1 + F2)/m, f1 = (F2 - F1) arm / I.
    __device__ static __forceinline__ void inputs(const DevParams& p, float s0, float s1, float& f0, float& f1)
    {
        const float hover = 0.5f * p.mass * p.gravity;
        const float F1 = hover + s0, F2 = hover + s1;
        f0 = (F1 + F2) / p.mass;
        f1 = (F2 - F1) * (p.arm / p.inertia);
    }
    __device__ static __forceinline__ float heading(float dt, float& th, float& w, float, float f1)
    {
        th = fmaf(w, dt, th);
        w = fmaf(f1, dt, w);
        return w;
    }
    __device__ static __forceinline__ void position(const DevParams& p, int axis, float& q, float& v, float f0, float,
                                                    float sn, float cs)
    {
        const float a = axis == 0 ? -(f0 * sn) : fmaf(f0, cs, -p.gravity);
        q = fmaf(v, p.dt, q);
        v = fmaf(a, p.dt, v);
    }
};

template <> struct Model<MPPI_QUAD5> {
    static constexpr int NS = 5;
    static constexpr int W = 0;
    // Sec. V-A: state (x, z, theta, vx, vz); inputs (pitch rate, throttle).
    // f0 = pitch rate, f1 = (m g + u_t)/m.
    __device__ static __forceinline__ void inputs(const DevParams& p, float s0, float s1, float& f0, float& f1)
    {
        f0 = s0;
        f1 = (p.mass * p.gravity + s1) / p.mass;
    }
    __device__ static __forceinline__ float heading(float dt, float& th, float&, float f0, float f1)
    {
        th = fmaf(f0, dt, th);
        return f1;
    }
    __device__ static __forceinline__ void position(const DevParams& p, int axis, float& q, float& v, float, float f1,
                                                    float sn, float cs)
    {
        Model<MPPI_QUAD6>::position(p, axis, q, v, f1, 0.0f, sn, cs);
    }
};

template <> struct Model<MPPI_CAR> {
    static constexpr int NS = 4;
    static constexpr int W = 3;
    // Sec. V-B Ackermann model: state (x, y, theta, v); inputs (steer, accel).
    // f0 = tan(phi)/L = sin(phi) / (cos(phi) L), f1 = a.
    __device__ static __forceinline__ void inputs(const DevParams& p, float s0, float s1, float& f0, float& f1)
    {
        float sp, cp;
        heading_sincos(s0, sp, cp);
        f0 = sp / (cp * p.wheelbase);
        f1 = s1;
    }
    __device__ static __forceinline__ float heading(float dt, float& th, float& v, float f0, float f1)
    {
        th = fmaf(v * f0, dt, th);
        v = fmaf(f1, dt, v);
        return v;
    }
    __device__ static __forceinline__ void position(const DevParams& p, int axis, float& q, float& v, float, float vn,
                                                    float sn, float cs)
    {
        q = fmaf(v * (axis == 0 ? cs : sn), p.dt, q);
        v = vn;
    }
};

// A grid of the far field seen from the start position: the cell of a local
// position (x, y) is (ix + floor(gx), iy + floor(gy)) with gx = x inv + fx
// (the start's own cell and its place in it, split in FP64, so that a query
// rounds at the rollout's extent, not the world's).
struct FieldGrid {
    int32_t ix, iy, nx, ny, base;
    float fx, fy, inv;
    float half;         // cell side / W: grid units to the polynomial's coordinates
    float iw;           // 1 / W: metres to the polynomial's coordinates
    float pad[2];
};
static_assert(sizeof(FieldGrid) * kFieldLevels <= 192, "LDS of the grids");

// LDS carve-up of one rollout tile (sizes: tile_fixed_lds, slot_area, noise).
struct TileLds {
    float4* obs;      // [J] (ox, oy, -r^2 + d, -r^2), local frame; d = |s_0|^2 on the
                      // vehicle's layout-form and the quadrotor's mirrored-axis tiles, else 0
    float2* U;        // [T]
    float* ref;       // [(T+1) n], local frame
    double* e;        // [kMaxTile] tile exponentials
    double* red;      // [kRollBlock] partial costs, [group][sample]
    double* slots;    // [16] block-reduction slots
    int* omax;        // the bits of the largest |o|^2 over the obstacles
    int* next;        // [2] the next unit of a chunk, by chunk parity
    FieldGrid* grid;  // [kFieldLevels] the far field's grids (no cells: no field)
    float2* shape;    // [MPPI_PMAX] shape points (for lanes that differ in theirs: the kernel
                      // arguments lie in host memory, and only scalar reads of them are cached)
    // slots of one chunk, per (step, sample), and kXSlots more:
    float4* a;        // (f0, f1, -, control cost), (f0, y, theta, control cost), then (f0, y, sin, cos)
    float* px;        // position, local frame
    float* py;
    float* vx;        // velocity (quadrotors)
    float* vy;
    float* b;         // theta, then the fused barrier (indicator: smallest h)
    float* mp;        // the control cost, then the costmap terms: sum B(sdf) or, with the indicator, the smallest sdf
    float2* nz;       // [T][S] the tile's noise, when it fits (else null)
};

__device__ __forceinline__ TileLds carve(unsigned char* smem, int J, int T, int n, int S, int tc, bool keep_noise)
{
    TileLds L;
    size_t off = 0;
    L.obs = reinterpret_cast<float4*>(smem + off);
    off += (size_t)obstacle_slots(J) * 16;
    L.U = reinterpret_cast<float2*>(smem + off);
    off += (size_t)T * 8;
    L.ref = reinterpret_cast<float*>(smem + off);
    off += (size_t)(T + 1) * n * 4;
    off = (off + 15) & ~(size_t)15;
    L.e = reinterpret_cast<double*>(smem + off);
    off += (size_t)kMaxTile * 8;
    L.red = reinterpret_cast<double*>(smem + off);
    off += (size_t)kRollBlock * 8;
    L.slots = reinterpret_cast<double*>(smem + off);
    off += 16 * 8;
    L.omax = reinterpret_cast<int*>(smem + off);
    L.next = L.omax + 1;
    off += 64;
    L.grid = reinterpret_cast<FieldGrid*>(smem + off);
    off += 192;
    L.shape = reinterpret_cast<float2*>(smem + off);
    off += MPPI_PMAX * 8;
    const int items = tc * (S + kRowPad) + kXSlots;
    L.a = reinterpret_cast<float4*>(smem + off);
    L.px = reinterpret_cast<float*>(L.a + items);
    L.py = L.px + items;
    L.b = L.py + items;
    L.mp = L.b + items;
    L.vx = L.mp + items;      // (only carved for n > 4)
    L.vy = L.vx + items;
    off += slot_area(T, n, S, tc);
    L.nz = keep_noise ? reinterpret_cast<float2*>(smem + off) : nullptr;
    return L;
}

struct X0 {
    float v[MPPI_NMAX + 2];
    uint32_t parity;     // which half of the warm-start double buffer holds U
    float S_e;           // exploration rate
    uint64_t counter;    // Philox step counter
};

constexpr int kRollWaves = kRollBlock / kWave;
// Most lanes (2^kFieldLgMax) that share an item whose barrier comes from the
// far field.
constexpr int kFieldLgMax = 2;
// Steps a recurrence reads from LDS ahead of their use: one at a time, each
// step waits for its read (about 120 cycles a step, against the few of its
// arithmetic).
constexpr int kAhead = 8;
constexpr int kUpdWaves = kUpdBlock / kWave;

// The quadrotor's mirrored axis with its middle point at the centre, against
// one obstacle (see fused_barrier_pose): fast() gives half the sum of 1/h over
// the seven points as one fraction, exact where m > 0 and f <= fcap; slow()
// the clamped per-point form.  The shape constants are uniform.
struct AxisBody {
    float px, py, csw, snw;             // position; 2 a_0 times the heading
    float D1, D2, DM, R1, R2, nK1, nK2, fcap, eps;

    __device__ __forceinline__ AxisBody(const float* sa2, const float* ss, float4 pose, float eps_)
    {
        const float A0 = sa2[0];
        px = pose.x;
        py = pose.y;
        csw = A0 * pose.z;
        snw = A0 * pose.w;
        D1 = uniform(ss[1] - ss[0]);
        D2 = uniform(ss[2] - ss[0]);
        DM = uniform(-ss[0]);
        // The heading projection enters scaled by A0 = 2 a_0: w = A0 e.u,
        // so pair 0's q is b0^2 - w^2 with no coefficient, and pair i's
        // is b_i^2 - (A_i / A0)^2 w^2.  (A0 = 0 only for a body whose
        // points all sit at its centre: then every A_i is 0.)
        R1 = uniform(A0 != 0.0f ? sa2[1] / A0 : 0.0f);
        R2 = uniform(A0 != 0.0f ? sa2[2] / A0 : 0.0f);
        nK1 = uniform(-(R1 * R1));
        nK2 = uniform(-(R2 * R2));
        fcap = uniform(0.5f / fmaxf(eps_, 1e-4f));
        eps = eps_;
    }
    // The guard reads the fraction itself: h_m = b0 - a_0^2 is the
    // smallest c_i, so h_m > 0 and q_i = (c_i - d_i)(c_i + d_i) > 0 put
    // every h above 0; then f = (1/2) sum 1/h <= 1/(2 gmin) puts every
    // h at or above gmin.  (A NaN f fails the comparison.)
    // (the middle point enters as hd = 2 h_m, so that pair 2 and the
    // middle point meet as b2/q2 + 1/hd = (b2 hd + q2)/(q2 hd))
    __device__ __forceinline__ float fast(const float4 o, float& m) const
    {
        const float ex = px - o.x, ey = py - o.y;
        const float b0 = fmaf(ex, ex, fmaf(ey, ey, o.z));
        const float w = fmaf(ex, csw, ey * snw);
        const float b1 = b0 + D1, b2 = b0 + D2;
        const float hd = fmaf(2.0f, b0, 2.0f * DM);
        const float w2 = w * w;
        const float q0 = fmaf(b0, b0, -w2), q1 = fmaf(b1, b1, nK1 * w2);
        const float q2 = fmaf(b2, b2, nK2 * w2);
        const float n01 = fmaf(b0, q1, b1 * q0), d01 = q0 * q1;
        const float n2m = fmaf(b2, hd, q2), d2m = q2 * hd;
        m = fminf(fminf(q0, q1), fminf(q2, hd));
        return fmaf(n01, d2m, n2m * d01) * __builtin_amdgcn_rcpf(d01 * d2m);
    }
    __device__ __forceinline__ float slow(const float4 o) const
    {
        const float ex = px - o.x, ey = py - o.y;
        const float b0 = fmaf(ex, ex, fmaf(ey, ey, o.z));
        const float w = fmaf(ex, csw, ey * snw);
        const float b1 = b0 + D1, b2 = b0 + D2, hm = b0 + DM;
        float h[7] = {b0 + w, fmaf(R1, w, b1), fmaf(R2, w, b2), hm, fmaf(-R2, w, b2), fmaf(-R1, w, b1), b0 - w};
#pragma unroll
        for (int i = 0; i < 7; ++i) h[i] = clamp_h(h[i], eps);
        return 0.5f * reciprocal_total<7>(h);
    }
    // Four obstacles' terms behind one wave-uniform test (a wave takes the
    // clamped form of an obstacle only when a lane needs it).
    __device__ __forceinline__ float4 four(const float4 o0, const float4 o1, const float4 o2, const float4 o3) const
    {
        float m0, m1, m2, m3;
        float f0 = fast(o0, m0), f1 = fast(o1, m1), f2 = fast(o2, m2), f3 = fast(o3, m3);
        const bool low = fminf(fminf(m0, m1), fminf(m2, m3)) > 0.0f;
        const bool ok = low && fmaxf(fmaxf(f0, f1), fmaxf(f2, f3)) <= fcap;
        if (__builtin_expect(__ballot(!ok) != 0, 0)) {
            const bool k0 = m0 > 0.0f && f0 <= fcap, k1 = m1 > 0.0f && f1 <= fcap;
            const bool k2 = m2 > 0.0f && f2 <= fcap, k3 = m3 > 0.0f && f3 <= fcap;
            if (__ballot(!k0)) { const float s = slow(o0); f0 = k0 ? f0 : s; }
            if (__ballot(!k1)) { const float s = slow(o1); f1 = k1 ? f1 : s; }
            if (__ballot(!k2)) { const float s = slow(o2); f2 = k2 ? f2 : s; }
            if (__ballot(!k3)) { const float s = slow(o3); f3 = k3 ? f3 : s; }
        }
        return make_float4(f0, f1, f2, f3);
    }
    __device__ __forceinline__ float one(const float4 o) const
    {
        float m;
        float f = fast(o, m);
        const bool ok = m > 0.0f && f <= fcap;
        if (__builtin_expect(__ballot(!ok) != 0, 0)) {
            const float s = slow(o);
            f = ok ? f : s;
        }
        return f;
    }
};

// Part of the fused barrier of one pose, lane sp of a group of 2^lg lanes:
// every shape point against the obstacles (read from LDS) of this lane's runs.
// Run r of the pose's js = 2^rlg takes obstacles r, r + js, r + 2 js, ... below
// J and adds them up in that order; the lane's 2^(rlg - lg) <= 4 runs are
// neighbours, and their sums meet in pairs, as those of the lanes do.  The
// costmap terms are formed apart (map_terms).
//
// With e = pose - o, the heading u = (cos, sin) and its normal v, a shape
// point with body offset (a, b) gives
//   h = |e + a u + b v|^2 - r^2 = (|e|^2 - r^2) + (a^2 + 2a e.u) + (b^2 + 2b e.v).
// The fixed-P tiles use the layout of the paper's bodies (the host checks it):
// * vehicle, the corners and side midpoints of a rectangle: the two terms
//   take only the values for a = +-alpha, 0 and b = +-beta, 0, so one
//   obstacle costs 20 operations for its 8 pairs;
// * quadrotors, every point on the body axis (b = 0): h = |e|^2 - r^2 +
//   fma(2a, e.u, a^2), two operations a pair; when the points mirror about
//   the centre (the paper's frame), a mirrored pair takes three operations.
// Any other shape takes the general form: h = (|e|^2 - r^2) + 2 e.d_i + |d_i|^2
// with d_i the rotated offset, an add and two FMAs a pair.
// (sa2, sb2) = 2 (a_i, b_i), ss = a_i^2 + b_i^2.
// In a far field's tile (FIELD) a run is a whole lane's, up to 2048 obstacles,
// and is added up in FP64: its FP32 sum rounded to 5.2e-6 of a cost in contact
// where the shorter runs round to 3.7e-6.
template <int MODEL, int PT, bool FIELD, class Sum = std::conditional_t<FIELD, double, float>>
__device__ __forceinline__ Sum fused_barrier_pose(const DevParams& p, const TileLds& L, const float* sa2,
                                                  const float* sb2, const float* ss, float4 pose, int sp, int lg,
                                                  int rlg, float omax2)
{
    constexpr int PM = PT ? PT : MPPI_PMAX;
    const float eps = p.h_eps;
    const float cs = pose.z, sn = pose.w;
    const int J = p.J, js = 1 << rlg;
    // A run has q obstacles, and one more when r < rem.  The loop count q is
    // the same on every lane, so the loop is counted in scalar registers; both
    // reads of a pair are issued before either obstacle is used.
    const int q = J >> rlg, rem = J & (js - 1);
    auto run = [&](int r, auto&& body) __attribute__((always_inline)) {
        const float4* ob = L.obs + r;
        for (int i = 0; i + 2 <= q; i += 2) {
            const float4 o0 = ob[0], o1 = ob[js];
            ob += 2 * js;
            body(o0);
            body(o1);
        }
        if (q & 1) {
            body(ob[0]);
            ob += js;
        }
        if (r < rem) body(ob[0]);
    };
    // The sum over this lane's runs of sum(r).
    auto over_runs = [&](auto&& sum) __attribute__((always_inline)) {
        const int n = 1 << (rlg - lg);
        if constexpr (FIELD) return sum(sp);
        Sum all = 0, pair = 0;
#pragma unroll 1
        for (int g = 0; g < n; ++g) {
            const Sum w = sum(sp * n + g);
            pair = (g & 1) ? pair + w : w;
            if (g < 2) all = pair;
            else if (g == 3) all += pair;
        }
        return all;
    };
    // Pair fractions (the layout forms' fast path).  Two points whose h are
    // c + d and c - d give 1/(c+d) + 1/(c-d) = 2c/(c^2 - d^2); the bodies of
    // Sec. V split into such pairs (the vehicle's four, the quadrotor's three
    // mirrored ones plus its middle point), and their fractions meet in one:
    // one reciprocal per obstacle, no clamp.  It holds when every h of the
    // obstacle is at least gmin = max(h_eps, 1e-4) -- then B(h) = 1/h, and
    // every h lies in [gmin, 2c] -- and c is at most the form's cap, so the
    // products of all the h stay inside the FP32 range.  Any other obstacle
    // takes the clamped per-point form.  The sums are of c/q, half of each
    // fraction.
    const float gmin = fmaxf(eps, 1e-4f);
    if constexpr (PT == 0) {
        // 2 d_i of every point, in registers; the rest of a pair is an add, two
        // FMAs, the clamp and the reciprocal
        float tx[PM], ty[PM], d2[PM];
        const int P = p.P;
        if (J == 0) return (Sum)0;
#pragma unroll
        for (int i = 0; i < PM; ++i) {
            tx[i] = ty[i] = d2[i] = 0.0f;
            if (i < P) {
                const float a = p.shape[i][0], b = p.shape[i][1];
                tx[i] = fmaf(2.0f * a, cs, -(2.0f * b) * sn);
                ty[i] = fmaf(2.0f * a, sn, (2.0f * b) * cs);
                d2[i] = uniform(fmaf(a, a, b * b));
                asm volatile("" : "+v"(tx[i]));
            }
        }
        return over_runs([&](int r) __attribute__((always_inline)) {
            Sum acc = 0;
            run(r, [&](const float4 o) __attribute__((always_inline)) {
                const float ex = pose.x - o.x, ey = pose.y - o.y;
                const float ee = fmaf(ex, ex, fmaf(ey, ey, o.w));
                // two points behind one branch (the empty asm keeps it one: as
                // selects, all 16 points were formed whatever P)
#pragma unroll
                for (int i = 0; i < PM; i += 2) {
                    if (i < P) {
                        const float h0 = clamp_h(fmaf(ex, tx[i], fmaf(ey, ty[i], ee + d2[i])), eps);
                        const float h1 = clamp_h(fmaf(ex, tx[i + 1], fmaf(ey, ty[i + 1], ee + d2[i + 1])), eps);
                        acc += __builtin_amdgcn_rcpf(h0);
                        const float f1 = __builtin_amdgcn_rcpf(h1);
                        acc += i + 1 < P ? f1 : 0.0f;
                        asm volatile("" : "+v"(acc));
                    }
                }
            });
            return acc;
        });
    } else if constexpr (MODEL == MPPI_CAR) {
        static_assert(PT == 8, "vehicle layout: 8 points");
        // point 0 is (a, b); o.z = -r^2 + a^2 + b^2, so C = |e|^2 - r^2 + a^2 +
        // b^2 takes two operations, and with P = 2a e.u, Q = 2b e.v the
        // corners are (C +- P) +- Q, the side midpoints C +- P - b^2 and
        // C - a^2 +- Q.  Pairs: (C+P) +- Q, (C-P) +- Q, (C-b^2) +- P and
        // (C-a^2) +- Q; the smallest h is C - |P| - |Q| (a corner),
        // C - b^2 - |P| or C - a^2 - |Q|, the largest at most 2C.
        // Cap: C <= 2e4, so 8 values of h <= 4e4 multiply below 7e36.
        constexpr float kCap = 2.0e4f;
        const float AA = ss[4], BB = ss[6];
        const float cu = sa2[0] * cs, su = sa2[0] * sn, cv = sb2[0] * cs, sv = sb2[0] * sn;
        // NOCAP: C <= |pose - o|^2 + a^2 + b^2 <= 2 |pose|^2 + 2 max_j |o_j|^2 +
        // a^2 + b^2 is below the cap on every lane of the unit, so no obstacle
        // needs the cap term in the guard
        auto body = [&](auto nocap_tag) __attribute__((always_inline)) {
            constexpr bool NOCAP = decltype(nocap_tag)::value;
            return over_runs([&](int r) __attribute__((always_inline)) {
                Sum half = 0;
                run(r, [&](const float4 o) __attribute__((always_inline)) {
                    const float ex = pose.x - o.x, ey = pose.y - o.y;
                    const float C = fmaf(ex, ex, fmaf(ey, ey, o.z));
                    const float Pu = fmaf(ex, cu, ey * su), Qv = fmaf(ey, cv, -ex * sv);
                    const float X1 = C + Pu, X2 = C - Pu, X3 = C - BB, X4 = C - AA;
                    const float aP = fabsf(Pu), aQ = fabsf(Qv);
                    const float g = NOCAP ? fminf(fminf(C - aP - aQ, X3 - aP), X4 - aQ)
                                          : fminf(fminf(C - aP - aQ, X3 - aP), fminf(X4 - aQ, (kCap + gmin) - C));
                    const float P2 = Pu * Pu, Q2 = Qv * Qv;
                    const float q1 = fmaf(X1, X1, -Q2), q2 = fmaf(X2, X2, -Q2);
                    const float q3 = fmaf(X3, X3, -P2), q4 = fmaf(X4, X4, -Q2);
                    const float n12 = fmaf(X1, q2, X2 * q1), d12 = q1 * q2;
                    const float n34 = fmaf(X3, q4, X4 * q3), d34 = q3 * q4;
                    float f = fmaf(n12, d34, n34 * d12) * __builtin_amdgcn_rcpf(d12 * d34);
                    // (a wave-uniform branch: the clamped form only when a lane needs it)
                    if (__builtin_expect(__ballot(g < gmin) != 0, 0)) {
                        float h[8] = {X1 + Qv, X1 - Qv, X2 + Qv, X2 - Qv, X1 - BB, X2 - BB, X4 + Qv, X4 - Qv};
#pragma unroll
                        for (int i = 0; i < 8; ++i) h[i] = clamp_h(h[i], eps);
                        const float slow = 0.5f * reciprocal_total<8>(h);
                        f = g >= gmin ? f : slow;
                    }
                    half += (Sum)f;
                });
                return (Sum)2 * half;
            });
        };
        const float bound = fmaf(2.0f, fmaf(pose.x, pose.x, pose.y * pose.y), omax2) + ss[0];
        if (__ballot(!(bound <= kCap)) == 0) return body(std::true_type{});
        return body(std::false_type{});
    } else {
        static_assert(PT == 7, "quadrotor layout: 7 points");
        // The mirrored-axis form: a_{6-i} = -a_i, and |a_0| is the largest
        // |a_i| (the host checks both): pair i shares c_i = |e|^2 - r^2 + a_i^2
        // and its two points differ in the sign of d_i = 2 a_i e.u.  o.z =
        // -r^2 + a_0^2, so c_0 = b0 = |e|^2 + o.z itself and c_i = b0 + (a_i^2 -
        // a_0^2) <= b0.  It runs when the middle point is the centre (a_3 = 0,
        // the paper's body: h_m = b0 - a_0^2 <= b0) and no obstacle of this unit
        // can pass the cap: every h is then at most 2 b0 <= 2e5, and 7 of them
        // multiply below 1.3e37.  The cap holds for the whole unit when
        // 2 |pose|^2 + 2 max_j |o_j|^2 + a_0^2 <= 1e5 on every lane, since
        // b0 <= |pose - o|^2 + a_0^2.  Any other unit, or body, runs the
        // clamped per-point form below.
        constexpr float kCap = 1.0e5f;
        const bool mirrored = p.shape_kind == kShapeMirroredAxis;
        bool fast = false;
        if (mirrored && sa2[3] == 0.0f) {
            const float bound = fmaf(2.0f, fmaf(pose.x, pose.x, pose.y * pose.y), omax2) + ss[0];
            fast = __ballot(!(bound <= kCap)) == 0;
        }
        if (fast) {
            // Four obstacles an iteration share one guard test, so the loop
            // takes no branch per obstacle.
            const AxisBody body(sa2, ss, pose, eps);
            return over_runs([&](int r) __attribute__((always_inline)) {
                Sum half = 0;
                const float4* ob = L.obs + r;
                int i = 0;
                for (; i + 4 <= q; i += 4) {
                    const float4 f = body.four(ob[0], ob[js], ob[2 * js], ob[3 * js]);
                    ob += 4 * js;
                    if constexpr (FIELD) half += (Sum)((f.x + f.y) + (f.z + f.w));
                    else half = (((half + f.x) + f.y) + f.z) + f.w;
                }
                for (; i < q; ++i) {
                    half += (Sum)body.one(ob[0]);
                    ob += js;
                }
                if (r < rem) half += (Sum)body.one(ob[0]);
                return (Sum)2 * half;
            });
        }
        // (on the mirrored-axis tile o.z carries the a_0^2 offset)
        float ssx[PM];
#pragma unroll
        for (int i = 0; i < PM; ++i) ssx[i] = mirrored ? ss[i] - ss[0] : ss[i];
        return over_runs([&](int r) __attribute__((always_inline)) {
            Sum acc = 0, acc2 = 0;
            run(r, [&](const float4 o) __attribute__((always_inline)) {
                const float ex = pose.x - o.x, ey = pose.y - o.y;
                const float ee = fmaf(ex, ex, fmaf(ey, ey, o.z));
                const float pu = fmaf(ex, cs, ey * sn);
                float h[PM];
#pragma unroll
                for (int i = 0; i < PM; ++i) h[i] = clamp_h(ee + fmaf(sa2[i], pu, ssx[i]), eps);
                if constexpr (FIELD) acc += (Sum)reciprocal_total<PM>(h);
                else reciprocal_sum<PM>(h, acc, acc2);
            });
            return acc + acc2;
        });
    }
}

// The general form of one pose against all obstacles, lane sp of a group of
// js = 2^lg lanes: any shape, h = (|e|^2 - r^2) + 2 e.d_i + |d_i|^2 with d_i
// the rotated offset.  Returns its share of sum 1/h or, with IND, the smallest
// h (the comparison controllers' constraint test, Sec. IV-A's weighted
// indicator: a pose violates a constraint where some h < 0; +inf without an
// obstacle).  Four points at a time walk the obstacles: their offsets take 12
// registers where all 16 took 48 and spilled, and four reciprocals are one.
template <bool IND, class Sum = std::conditional_t<IND, float, double>>
__device__ __forceinline__ Sum walk_points(const DevParams& p, const TileLds& L, int P, float4 pose, int sp, int lg)
{
    const int J = p.J, js = 1 << lg;
    Sum acc = IND ? (Sum)INFINITY : (Sum)0;
#pragma unroll 1
    for (int i0 = 0; i0 < P; i0 += 4) {
        float tx[4], ty[4], ss[4];      // 2 d_i, |d_i|^2
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = min(i0 + k, P - 1);
            const float a = p.shape[i][0], b = p.shape[i][1];
            tx[k] = fmaf(2.0f * a, pose.z, -(2.0f * b) * pose.w);
            ty[k] = fmaf(2.0f * a, pose.w, (2.0f * b) * pose.z);
            ss[k] = fmaf(a, a, b * b);
        }
        const int np = P - i0;
        auto h_of = [&](const float4 o, float (&h)[4]) __attribute__((always_inline)) {
            const float ex = pose.x - o.x, ey = pose.y - o.y;
            const float ee = fmaf(ex, ex, fmaf(ey, ey, o.w));
#pragma unroll
            for (int k = 0; k < 4; ++k) h[k] = fmaf(ex, tx[k], fmaf(ey, ty[k], ee + ss[k]));
        };
        const float4* ob = L.obs + sp;
        for (int j = sp; j < J; j += js, ob += js) {
            float h[4];
            h_of(ob[0], h);
            if constexpr (IND) {
                acc = fminf(acc, fminf(fminf(h[0], h[1]), fminf(h[2], h[3])));
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) h[k] = clamp_h(h[k], p.h_eps);
                acc += (Sum)reciprocal_head(h, np);
            }
        }
    }
    return acc;
}

// ---------------------------------------------------------------------------
// The fused barrier by the far field (mppi_field.hpp).
// ---------------------------------------------------------------------------
// The cell of a local position: its record, the polynomial's coordinates and
// scale.  ok: the position lies on a grid and the cell's near list is whole.
struct FieldCell {
    const float* rec;
    float u, v, iw;
    int count;          // near obstacles (0 when not ok)
    bool ok;
};

__device__ __forceinline__ FieldCell field_cell(const TileLds& L, const float* cells, float x, float y)
{
    FieldCell c{cells, 0.0f, 0.0f, 0.0f, 0, false};
#pragma unroll
    for (int l = 0; l < kFieldLevels; ++l) {
        if (l > 0 && __ballot(!c.ok) == 0) break;
        const FieldGrid g = L.grid[l];
        const float gx = fmaf(x, g.inv, g.fx), gy = fmaf(y, g.inv, g.fy);
        const float flx = floorf(gx), fly = floorf(gy);
        const float tx = (float)g.ix + flx, ty = (float)g.iy + fly;
        if (!c.ok && tx >= 0.0f && tx < (float)g.nx && ty >= 0.0f && ty < (float)g.ny) {
            c.rec = cells + (size_t)(g.base + (int)ty * g.nx + (int)tx) * kFieldWords;
            c.u = ((gx - flx) - 0.5f) * g.half;
            c.v = ((gy - fly) - 0.5f) * g.half;
            c.iw = g.iw;
            c.ok = true;
        }
    }
    if (c.ok) {
        c.count = __float_as_int(c.rec[kFieldCoefs]);
        if (c.count == kFieldFull) {
            c.ok = false;
            c.count = 0;
        }
    }
    return c;
}

// The sum over N points of the cell's polynomial (Horner's rule by rows of
// falling powers of v; the record is read in that order).  The record comes in
// three thirds, two in flight: all of it at once, beside seven points' rows,
// spilled 70 registers.
template <int N>
__device__ __forceinline__ float field_far(const float* rec, const float (&u)[N], const float (&v)[N], int n = N)
{
    constexpr int kThird = 16;
    static_assert(kFieldCoefs + 3 == 3 * kThird, "three thirds");
    const float4* r4 = reinterpret_cast<const float4*>(rec);
    float c[3 * kThird];
    auto load = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kThird / 4; ++i) {
            const float4 w = r4[t * kThird / 4 + i];
            c[t * kThird + 4 * i] = w.x;
            c[t * kThird + 4 * i + 1] = w.y;
            c[t * kThird + 4 * i + 2] = w.z;
            c[t * kThird + 4 * i + 3] = w.w;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    load(0);
    load(1);
    float acc[N], r[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = c[0];
    int q = 1;
#pragma unroll
    for (int l = kFieldDeg - 1; l >= 0; --l) {
#pragma unroll
        for (int k = kFieldDeg - l; k >= 0; --k) {
            if (q == kThird) load(2);
#pragma unroll
            for (int i = 0; i < N; ++i) r[i] = k == kFieldDeg - l ? c[q] : fmaf(r[i], u[i], c[q]);
            ++q;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = fmaf(acc[i], v[i], r[i]);
    }
    float s = acc[0];
#pragma unroll
    for (int i = 1; i < N; ++i) s += i < n ? acc[i] : 0.0f;
    return s;
}

// Near obstacles 4g .. 4g + 3 of a cell (two list words).
__device__ __forceinline__ uint2 field_near(const float* rec, int g)
{
    return reinterpret_cast<const uint2*>(rec + kFieldCoefs + 1)[g];
}

// The fused barrier of one pose of the quadrotor's axis body, lane sp of
// 2^LG: points sp, sp + 2^LG, ... of the far polynomial (the whole body is
// within the cell's margin) and every 2^LG-th group of four near obstacles.
// ok: false where the pose has no cell; the poses of a wave with such a one all
// walk the obstacles, and the result is not used.
template <int LG>
__device__ __forceinline__ float field_barrier_axis(const DevParams& p, const TileLds& L, const float* cells,
                                                    const float* sa2, const float* ss, float4 pose, int sp,
                                                    float omax2, bool& ok)
{
    constexpr int NSP = 1 << LG, N = (7 + NSP - 1) / NSP;
    const FieldCell c = field_cell(L, cells, pose.x, pose.y);
    ok = c.ok;
    if (__ballot(!ok) != 0) return 0.0f;        // (the wave's poses walk)
    float u[N], v[N];
    const float ch = 0.5f * pose.z * c.iw, sh = 0.5f * pose.w * c.iw;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        float a = sa2[i * NSP];
#pragma unroll
        for (int k = 1; k < NSP; ++k)
            if (i * NSP + k < 7) a = sp == k ? sa2[i * NSP + k] : a;
        u[i] = fmaf(a, ch, c.u);
        v[i] = fmaf(a, sh, c.v);
    }
    const int mine = (7 - sp + NSP - 1) / NSP;
    float far = field_far<N>(c.rec, u, v, mine);
    asm volatile("" : "+v"(far));       // (before the near obstacles: the compiler would hold the coefficients through them)
    const bool mirrored = p.shape_kind == kShapeMirroredAxis;
    const float bound = fmaf(2.0f, fmaf(pose.x, pose.x, pose.y * pose.y), omax2) + ss[0];
    const bool fast = mirrored && sa2[3] == 0.0f && __ballot(c.ok && !(bound <= 1.0e5f)) == 0;
    const int groups = (c.count + 3) >> 2;
    float near = 0.0f;
    if (fast) {
        const AxisBody body(sa2, ss, pose, p.h_eps);
        float half = 0.0f;
        for (int g = sp; g < groups; g += NSP) {
            const uint2 w = field_near(c.rec, g);
            const int i0 = w.x & 0xFFFF, left = c.count - 4 * g;
            // (beyond the list's end: the group's first obstacle again, taken off below)
            const int i1 = left > 1 ? w.x >> 16 : i0, i2 = left > 2 ? w.y & 0xFFFF : i0, i3 = left > 3 ? w.y >> 16 : i0;
            if (__ballot(left < 4) == 0) {
                const float4 f = body.four(L.obs[i0], L.obs[i1], L.obs[i2], L.obs[i3]);
                half += (f.x + f.y) + (f.z + f.w);
            } else {
                const float f0 = body.one(L.obs[i0]), f1 = body.one(L.obs[i1]);
                const float f2 = body.one(L.obs[i2]), f3 = body.one(L.obs[i3]);
                half += (f0 + (left > 1 ? f1 : 0.0f)) + ((left > 2 ? f2 : 0.0f) + (left > 3 ? f3 : 0.0f));
            }
        }
        near = 2.0f * half;
    } else {
        for (int k = sp; k < c.count; k += NSP) {
            const uint2 w = field_near(c.rec, k >> 2);
            const uint32_t word = (k & 2) ? w.y : w.x;
            const float4 o = L.obs[(k & 1) ? word >> 16 : word & 0xFFFF];
            const float ex = pose.x - o.x, ey = pose.y - o.y;
            const float ee = fmaf(ex, ex, fmaf(ey, ey, o.w));
            const float pu = fmaf(ex, pose.z, ey * pose.w);
#pragma unroll 1
            for (int i = 0; i < 7; ++i) {
                const float a = L.shape[i].x;
                near += barrier_rcp(fminf(ee + fmaf(2.0f * a, pu, a * a), kHMax), p.h_eps);
            }
        }
    }
    return near + far;
}

// The same for any body, a point at a time: lane sp of 2^lg takes points sp,
// sp + 2^lg, ...; each has its own cell.  IND: the smallest h over the near
// obstacles instead (a far one is never below 0).
template <bool IND>
__device__ __forceinline__ float field_barrier_points(const DevParams& p, const TileLds& L, const float* cells, int P,
                                                      float4 pose, int sp, int lg, bool& ok)
{
    float near = IND ? INFINITY : 0.0f, far = 0.0f;
    ok = true;
    for (int i = sp; i < P; i += 1 << lg) {
        const float2 ab = L.shape[i];
        const float a = ab.x, b = ab.y;
        const float dx = fmaf(a, pose.z, -b * pose.w), dy = fmaf(a, pose.w, b * pose.z);
        const FieldCell c = field_cell(L, cells, pose.x + dx, pose.y + dy);
        ok = c.ok;
        if (__ballot(!ok) != 0) break;          // (the wave's poses walk)
        if constexpr (!IND) {
            const float u[1] = {c.u}, v[1] = {c.v};
            far += field_far<1>(c.rec, u, v);
        }
        for (int g = 0; 4 * g < c.count; ++g) {
            const uint2 w = field_near(c.rec, g);
            const int left = c.count - 4 * g, i0 = w.x & 0xFFFF;
            const int id[4] = {i0, left > 1 ? (int)(w.x >> 16) : i0, left > 2 ? (int)(w.y & 0xFFFF) : i0,
                               left > 3 ? (int)(w.y >> 16) : i0};
            float h[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 o = L.obs[id[k]];
                const float ex = (pose.x - o.x) + dx, ey = (pose.y - o.y) + dy;
                h[k] = fmaf(ex, ex, fmaf(ey, ey, o.w));
            }
            if constexpr (IND) {
                near = fminf(near, fminf(fminf(h[0], h[1]), fminf(h[2], h[3])));
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) h[k] = clamp_h(h[k], p.h_eps);
                near += reciprocal_head(h, left);
            }
        }
    }
    return IND ? near : near + far;
}

// The costmap terms of one pose (every shape point): sum_i B(sdf(p_i)), or
// with the indicator the smallest sdf(p_i).  Four shape points' reads are in
// flight at a time; the body offsets come from the parameter block (uniform
// scalar loads), so the loop holds no per-point registers.
template <int PT, bool IND>
__device__ __forceinline__ float map_terms(const DevParams& p, int P, float4 pose, float inv_res, float offx,
                                           float offy)
{
    constexpr int G = 4;
    const int np = PT ? PT : P;
    const float cs = pose.z, sn = pose.w;
    float acc = IND ? INFINITY : 0.0f;
#pragma unroll 1
    for (int i0 = 0; i0 < np; i0 += G) {
        float v[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int i = min(i0 + j, np - 1);
            const float a = p.shape[i][0], b = p.shape[i][1];
            const float px = pose.x + fmaf(a, cs, -b * sn);
            const float py = pose.y + fmaf(a, sn, b * cs);
            v[j] = sdf_sample(p, fmaf(px, inv_res, offx), fmaf(py, inv_res, offy));
        }
#pragma unroll
        for (int j = 0; j < G; ++j)
            if (i0 + j < np) acc = IND ? fminf(acc, v[j]) : acc + barrier_rcp(v[j], p.h_eps);
    }
    return acc;
}

// ---------------------------------------------------------------------------
// One tile of S samples: rollout and the tile's softmax partials.
// PT = compile-time number of shape points (0: runtime P <= MPPI_PMAX; the
// fixed-P tiles use the layout form of the paper's bodies).  The standalone
// and the batched kernels run the same tile.
//
// The horizon is cut into chunks of tc steps (tile_chunk: the whole horizon
// where it fits), and each chunk runs through the phases below, one workgroup
// barrier apart.  The items of a chunk are its (step, sample) pairs, item i =
// step i / S, sample i mod S; wherever threads walk the items one by one the
// stride is a multiple of S, so a thread meets one sample only, sample tid mod
// S, and keeps its share of that sample's cost in a register (FP64).
//   1  inputs of the chunk (the waves that own no sample; every wave in the
//      first chunk); meanwhile the owner lanes run the barrier-state
//      recursion of the chunk before;
//   2  headings (owner lanes);
//   3  sines and cosines of the headings;
//   4  positions (two lanes per sample, one an axis);
//   5  the tracking cost;
//   6  the barrier and costmap units.
// Measured: carrying the whole dynamics step on one lane per sample (the
// sine, the tracking cost and a compensated sum among it) took 0.3 us a
// step; the recurrences alone take about 0.03.
// A plan is the next period's warm start, and samples that nearly tie share the
// weights, so the rounding of a cost grows from period to period.  What rounds
// it is therefore held whatever the chunks, lanes and waves: the state in FP32,
// a step's tracking and control cost one FP32 sum over the state in order, the
// barrier state in FP32, the obstacles' runs (set_splits).  Those FP32 terms
// are added up in FP64, where the order is below the rest.  (Recurrences and
// barrier sums in FP64, closer to the exact costs, moved plans of the second
// period by up to 4e-4.)
// Every (step, sample) of a chunk is split over nsp adjacent lanes, each with
// 1, 2 or 4 of its runs of obstacles; the nsp partial sums meet by wave
// shuffles.
// ---------------------------------------------------------------------------
template <int MODEL, int S, int PT, bool IND, bool MAP, bool FIELD>
__device__ void rollout_tile(const DevParams& p, const int tile, const X0& xs, unsigned char* smem)
{
    static_assert(!IND || PT == 0, "the indicator runs on the runtime-P tile");
    static_assert(!FIELD || PT != 8, "the vehicle's field takes the body a point at a time");
    constexpr int NS = Model<MODEL>::NS;
    // the vehicle's field tile, whose walk takes the layout form of its body
    constexpr bool VEHICLE = MODEL == MPPI_CAR && FIELD && !IND;
    constexpr int DW = (S + kWave - 1) / kWave;     // waves that own samples
    constexpr int POOL0 = DW * kWave;               // first thread of the other waves
    static_assert(S >= 16 && S <= kMaxTile && (S & (S - 1)) == 0, "tile size");
    static_assert(POOL0 % S == 0 || S > POOL0, "a thread's items belong to one sample");
    constexpr int RS = S + kRowPad;                 // slots from one step to the next
    auto slot = [](int item) __attribute__((always_inline)) { return item + item / S; };   // of item (step, sample)
    static_assert(kRowPad == 1, "slot()");
    static_assert(2 * S <= kRollBlock && (kRollBlock - POOL0) % S == 0, "tile size");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int J = p.J, T = p.T, K = p.K, Kp = p.Kp;
    const int P = PT ? PT : p.P;
    const int tc = tile_chunk(J, T, NS, S);
    const int nch = (T + tc - 1) / tc;
    const bool keep_noise = tile_keeps_noise(J, T, NS, S);
    const TileLds L = carve(smem, J, T, NS, S, tc, keep_noise);
    const float S_e = xs.S_e;
    const uint64_t ctr = xs.counter;
    const uint32_t c_lo = (uint32_t)ctr, c_hi = (uint32_t)(ctr >> 32);

    // the Philox words of sample kk at step t (Sec. IV-C: counter (k, t, iteration))
    // (the key words, uniform over the tile, pass through an empty asm
    // statement, so that the twenty round keys are formed per item by scalar
    // adds instead of being held in scalar registers across the whole chunk
    // loop, where they crowded out other values into reloads)
    auto philox_at = [&](int kk, int t) __attribute__((always_inline)) {
        uint32_t k0 = __builtin_amdgcn_readfirstlane(p.seed_lo), k1 = __builtin_amdgcn_readfirstlane(p.seed_hi);
        asm volatile("" : "+s"(k0), "+s"(k1));
        return philox4x32_10(make_uint4((uint32_t)kk, (uint32_t)t, c_lo, c_hi), k0, k1);
    };
    // ---- staging: local frame centred on the start position ----
    // The first element of each array is loaded before anything waits (one
    // memory round trip for all three), and this thread's first Philox words
    // are drawn meanwhile.
    const float* Uin = p.U + (size_t)(xs.parity & 1u) * T * kM;
    float ob0 = 0.0f, ob1 = 0.0f, ob2 = 0.0f, ref0 = 0.0f;
    float2 u0 = make_float2(0.0f, 0.0f);
    if (tid < J) {
        ob0 = p.obs[3 * tid];
        ob1 = p.obs[3 * tid + 1];
        ob2 = p.obs[3 * tid + 2];
    }
    if (tid < T) u0 = make_float2(Uin[2 * tid], Uin[2 * tid + 1]);
    if (tid < (T + 1) * NS) ref0 = p.xref[tid];
    const int s_mine = tid & (S - 1);       // the sample of every item this thread walks
    const uint4 w0 = philox_at(tile * S + s_mine, tid / S);

    const double ox = (double)xs.v[0], oy = (double)xs.v[1];
    float omax_mine = 0.0f;     // this thread's largest |o|^2 (local frame), for the barrier's cap bound
    if (tid < 3) L.omax[tid] = 0;           // and the unit counters
    {
        // the vehicle's layout form and the quadrotor's mirrored-axis form
        // offset |e|^2 - r^2 by |s_0|^2 (third word); the fourth word keeps
        // -r^2
        const bool offset = MODEL == MPPI_CAR ? PT != 0 || (VEHICLE && p.shape_kind == kShapeLayout)
                                              : PT != 0 && p.shape_kind == kShapeMirroredAxis;
        const double s00 = (double)p.shape[0][0], s01 = (double)p.shape[0][1];
        const double d0 = offset ? s00 * s00 + s01 * s01 : 0.0;
        for (int j = tid; j < J; j += kRollBlock) {
            if (j != tid) {
                ob0 = p.obs[3 * j];
                ob1 = p.obs[3 * j + 1];
                ob2 = p.obs[3 * j + 2];
            }
            const double cx = (double)ob0, cy = (double)ob1, r = (double)ob2;
            const float4 o = make_float4((float)(cx - ox), (float)(cy - oy), (float)(d0 - r * r), (float)(-(r * r)));
            L.obs[j] = o;
            if constexpr (PT != 0 || VEHICLE) omax_mine = fmaxf(omax_mine, fmaf(o.x, o.x, o.y * o.y));
        }
    }
    if (tid < T) L.U[tid] = u0;             // (T <= MPPI_TMAX <= the workgroup)
    for (int i = tid; i < (T + 1) * NS; i += kRollBlock) {
        const int a = i % NS;
        const float v = i == tid ? ref0 : p.xref[i];
        L.ref[i] = a == 0 ? (float)((double)v - ox) : a == 1 ? (float)((double)v - oy) : v;
    }
    if (FIELD && tid < P) L.shape[tid] = make_float2(p.shape[tid][0], p.shape[tid][1]);
    // the far field's grids from the start position
    if (FIELD && tid < kFieldLevels) {
        const FieldLevel lv = p.field->level[tid];
        FieldGrid g{};
        if (p.field->J == J) {
            const double gx = (ox - lv.x0) / lv.side, gy = (oy - lv.y0) / lv.side;
            const double cx = fmin(fmax(floor(gx), -1e9), 1e9), cy = fmin(fmax(floor(gy), -1e9), 1e9);
            const float W = (float)(0.5 * lv.side) + p.field->margin;
            g.ix = (int32_t)cx;
            g.iy = (int32_t)cy;
            g.nx = lv.nx;
            g.ny = lv.ny;
            g.base = lv.base;
            g.fx = (float)(gx - cx);
            g.fy = (float)(gy - cy);
            g.inv = (float)(1.0 / lv.side);
            g.half = (float)(lv.side / (double)W);
            g.iw = 1.0f / W;
        }
        L.grid[tid] = g;
    }
    float inv_res = 0.0f, offx = 0.0f, offy = 0.0f;
    // MAP: the controller has a costmap (p.sdf set); the tiles without one
    // carry none of its code
    if constexpr (MAP) {
        inv_res = uniform((float)(1.0 / (double)p.map_res));
        offx = uniform((float)((ox - (double)p.map_x0) / (double)p.map_res - 0.5));
        offy = uniform((float)((oy - (double)p.map_y0) / (double)p.map_res - 0.5));
    }
    lds_barrier();
    // the largest |o|^2 over the obstacles (non-negative floats order as
    // their bit patterns); read in phase 6
    if constexpr (PT != 0 || VEHICLE) {
        if (omax_mine > 0.0f) atomicMax(L.omax, __float_as_int(omax_mine));
    }

    // ---- setup: lanes 0..S-1 own one sample each ----
    const bool owner = tid < S;
    const int k = tile * S + tid;
    const bool valid = owner && k < K;

    const float sqS = sqrtf(S_e);
    const float scale0 = uniform(sqS * p.sigma[0]), scale1 = uniform(sqS * p.sigma[1]);
    const bool normal_law = p.sampling == MPPI_SAMPLE_NORMAL;
    const float cw0 = uniform(p.sigma[0] > 0.0f ? p.gamma_u / (S_e * p.sigma[0] * p.sigma[0]) : 0.0f);
    const float cw1 = uniform(p.sigma[1] > 0.0f ? p.gamma_u / (S_e * p.sigma[1] * p.sigma[1]) : 0.0f);

    // eq. barrier_update is linear in beta, so beta_t = bv_t + c_t with the
    // sample-dependent part bv_t = b_t + gamma_B bv_{t-1} (bv_0 = beta_0) and
    // the common part c_t = gamma_B (c_{t-1} - beta_d) (c_0 = 0), whose sum is
    // -beta_d gamma_B/(1-gamma_B) (T - gamma_B (1-gamma_B^T)/(1-gamma_B)).
    // The common part's cost R_B sum_t c_t is the same for every sample and is
    // added in FP64 (cshift), so a large beta_d cannot swamp the FP32 sums;
    // the host forms its factor R_B sum_t c_t / beta_d once per controller.
    double cost = 0.0;          // this thread's share of the cost of sample s_mine

    // 2 s_i and |s_i|^2 of the layout forms (uniform: kept in scalar registers)
    constexpr int PM = PT ? PT : 1;
    float sa2[PM], sb2[PM], ss[PM];
    if constexpr (PT != 0) {
#pragma unroll
        for (int i = 0; i < PM; ++i) {
            const float a = p.shape[i][0], b = p.shape[i][1];
            sa2[i] = uniform(2.0f * a);
            sb2[i] = uniform(2.0f * b);
            ss[i] = uniform(fmaf(a, a, b * b));
        }
    }
    // What a recurrence carries from one chunk to the next, in the space of
    // the partial costs: heading and companion by chunk parity, barrier state.
    float2* carry_h = reinterpret_cast<float2*>(L.red);     // [2][kMaxTile]
    float* carry_b = reinterpret_cast<float*>(L.red + 2 * kMaxTile);
    static_assert(3 * kMaxTile <= kRollBlock, "carry");

    // the noise of sample kk at step t (Sec. IV-C mixture, scaled per Alg. 1)
    auto noise_of = [&](uint4 r) __attribute__((always_inline)) {
        return nln_pair(r, scale0, scale1, p.mu_ln, p.sigma_ln, normal_law);
    };
    auto noise_at = [&](int kk, int t) __attribute__((always_inline)) { return noise_of(philox_at(kk, t)); };

    // The thread's index as the phases of a chunk use it: opaque to the
    // compiler, which otherwise forms every phase's addresses before the chunk
    // loop and holds them through the barrier units (70 registers spilled).
    auto phase_tid = [&]() __attribute__((always_inline)) {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };

    // the inputs and the control cost of item idx (step t) from its Philox words
    auto input = [&](int idx, int t, int s, uint4 words) __attribute__((always_inline)) {
        const float2 z = noise_of(words);
        const float2 u = L.U[t];
        const float v0 = u.x + z.x, v1 = u.y + z.y;
        const float s0 = fminf(fmaxf(v0, p.u_min[0]), p.u_max[0]);
        const float s1 = fminf(fmaxf(v1, p.u_min[1]), p.u_max[1]);
        float f0, f1;
        Model<MODEL>::inputs(p, s0, s1, f0, f1);
        L.a[slot(idx)] = make_float4(f0, f1, 0.0f, cw0 * u.x * v0 + cw1 * u.y * v1);
        if (keep_noise) L.nz[t * S + s] = z;
    };

    // phase 1: the inputs of the n steps from t0 on, over threads [first, block)
    auto inputs_phase = [&](int t0, int n, int first) __attribute__((always_inline)) {
        [[maybe_unused]] const int tid = phase_tid(), s_mine = tid & (S - 1);
        int idx = tid - first;
        uint4 w = w0;
        if (t0 != 0 && idx < n * S) w = philox_at(tile * S + s_mine, t0 + idx / S);
        while (idx < n * S) {
            input(idx, t0 + idx / S, s_mine, w);
            idx += kRollBlock - first;
            if (idx < n * S) w = philox_at(tile * S + s_mine, t0 + idx / S);
        }
    };

    // A recurrence over n steps, step tt from what load(tt) returns: kAhead
    // loads in flight, then their steps, without a branch between them.
    auto walk = [&](int n, auto&& load, auto&& step) __attribute__((always_inline)) {
        int tt = 0;
        for (; tt + kAhead <= n; tt += kAhead) {
            decltype(load(0)) in[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) in[i] = load(tt + i);
#pragma unroll
            for (int i = 0; i < kAhead; ++i) step(tt + i, in[i]);
        }
        for (; tt < n; ++tt) step(tt, load(tt));
    };

    // phase 2 (owner lanes): theta into a.z, its companion into a.y
    auto headings_phase = [&](int c, int n) __attribute__((always_inline)) {
        [[maybe_unused]] const int tid = phase_tid();
        constexpr int W = Model<MODEL>::W;
        float4* a = L.a + tid;
        float th = xs.v[2], hw = W ? xs.v[W] : 0.0f;
        if (c > 0) {
            const float2 h = carry_h[((c - 1) & 1) * kMaxTile + tid];
            th = h.x;
            hw = h.y;
        }
        walk(
            n, [&](int tt) __attribute__((always_inline)) { return make_float2(a[tt * RS].x, a[tt * RS].y); },
            [&](int tt, float2 in) __attribute__((always_inline)) {
                a[tt * RS].y = Model<MODEL>::heading(p.dt, th, hw, in.x, in.y);
                a[tt * RS].z = th;
            });
        if (c + 1 < nch) carry_h[(c & 1) * kMaxTile + tid] = make_float2(th, hw);
    };

    // phase 3: sines and cosines of the headings; the heading and the control
    // cost, whose places they take, wait for the tracking cost in those of the
    // barrier and the costmap's part
    auto sines_phase = [&](int n) __attribute__((always_inline)) {
        const int tid = phase_tid();
        for (int idx = tid; idx < n * S; idx += kRollBlock) {
            const int at = slot(idx);
            const float4 in = L.a[at];
            float sn, cn;
            heading_sincos(in.z, sn, cn);
            L.a[at] = make_float4(in.x, in.y, sn, cn);
            L.b[at] = in.z;
            L.mp[at] = in.w;
        }
    };

    // phase 4 (lanes 0..2S-1): positions and velocities
    auto positions_phase = [&](int c, int n) __attribute__((always_inline)) {
        [[maybe_unused]] const int tid = phase_tid(), s_mine = tid & (S - 1);
        const int axis = tid / S;
        const float4* a = L.a + s_mine;
        float* pos = (axis == 0 ? L.px : L.py) + s_mine;
        [[maybe_unused]] float* vel = (axis == 0 ? L.vx : L.vy) + s_mine;
        float q = 0.0f, v = MODEL == MPPI_CAR ? xs.v[3] : axis == 0 ? xs.v[3] : xs.v[4];
        float th = xs.v[2];
        if (c > 0) {        // (this lane's own last step of the chunk before)
            const float2 h = carry_h[((c - 1) & 1) * kMaxTile + s_mine];
            th = h.x;
            q = pos[(tc - 1) * RS];
            if constexpr (NS > 4) v = vel[(tc - 1) * RS];
            else v = h.y;
        }
        float sn, cs;       // of the heading before the step
        heading_sincos(th, sn, cs);
        walk(
            n, [&](int tt) __attribute__((always_inline)) { return a[tt * RS]; },
            [&](int tt, float4 in) __attribute__((always_inline)) {
                Model<MODEL>::position(p, axis, q, v, in.x, in.y, sn, cs);
                sn = in.z;
                cs = in.w;
                pos[tt * RS] = q;
                if constexpr (NS > 4) vel[tt * RS] = v;
            });
    };

    // phase 5: the tracking cost of every step with its control cost, one FP32
    // sum a step over the state in order, and the terminal cost
    auto tracking_cost = [&](int t0, int n) __attribute__((always_inline)) {
        const int tid = phase_tid();
        constexpr int W = Model<MODEL>::W;
        for (int idx = tid; idx < n * S; idx += kRollBlock) {
            const int t = t0 + idx / S + 1, at = slot(idx);
            const float* rf = L.ref + t * NS;
            float x[NS];
            x[0] = L.px[at];
            x[1] = L.py[at];
            x[2] = L.b[at];
            if constexpr (NS > 4) {
                x[3] = L.vx[at];
                x[4] = L.vy[at];
            }
            if constexpr (W != 0) x[W] = L.a[at].y;
            float q = 0.0f, f = 0.0f;
#pragma unroll
            for (int a = 0; a < NS; ++a) {
                const float d = x[a] - rf[a], d2 = d * d;
                q = fmaf(p.Q[a], d2, q);
                f = fmaf(p.Qf[a], d2, f);
            }
            cost += (double)(q + L.mp[at]);
            if (t == T) cost += (double)f;
        }
    };

    // phase 6: the fused barrier (or smallest h) of every item of chunk c, in
    // units of one wave; then, with a costmap, map units (one item per lane,
    // every shape point: their reads all in flight at once, away from the long
    // obstacle units).  Before them, in chunk 0, a unit for the poses of x0 and
    // x_d (32 lanes each; without a far field a lane a run, two units where each
    // has 64 runs): few lanes with long runs, whose wave taken last held the
    // chunk up.  The waves take units from a counter: the
    // oldest wave of a SIMD wins its issue slots, so with equal shares the
    // first waves finish at 68 us of a 155 us phase (K = 16384, T = 100, 400
    // obstacles) and leave the last ones alone on their SIMDs, waiting on
    // their own latencies.
    auto units_phase = [&](int c, int n) __attribute__((always_inline)) {
        const int lane = phase_tid() & (kWave - 1);
        const int items = n * S;
        int lg = (p.lg_pack >> (c == nch - 1 ? 4 : 0)) & 15;
        [[maybe_unused]] const float* cells = nullptr;
        if constexpr (FIELD) {
            // enough lanes per item to give every wave a unit
            cells = reinterpret_cast<const float*>(p.field) + 64;
            lg = 0;
            while (lg < kFieldLgMax && items << lg <= (kRollWaves - 1) * kWave) ++lg;
        }
        int ounits = ((items << lg) + kWave - 1) / kWave, xunits = (!IND && c == 0) ? 1 : 0;
        // The obstacles' runs (set_splits): the steps and the units at which the
        // second and the third part of the horizon begin in this chunk.
        constexpr bool RUNS = !IND && !FIELD;
        [[maybe_unused]] int s1 = 0, s2 = 0, u1 = 0, u2 = 0;
        if constexpr (RUNS) {
            const int t0 = c * tc;
            s1 = min(max((p.run_steps & 0xFFFF) - t0, 0), n);
            s2 = min(max((p.run_steps >> 16) - t0, s1), n);
            u1 = ((s1 * S << run_lanes(p.run_lg, 0)) + kWave - 1) / kWave;
            u2 = u1 + (((s2 - s1) * S << run_lanes(p.run_lg, 1)) + kWave - 1) / kWave;
            ounits = u2 + (((n - s2) * S << run_lanes(p.run_lg, 2)) + kWave - 1) / kWave;
        }
        if (RUNS && c == 0) xunits = ((kXSlots << run_split(p.run_lg, 0)) + kWave - 1) / kWave;
        const int munits = MAP ? (items + kWave - 1) / kWave : 0;
        const int units = ounits + munits + xunits;
        [[maybe_unused]] float omax2 = 0.0f;
        if constexpr (PT != 0 || VEHICLE) omax2 = uniform(2.0f * __int_as_float(*L.omax));
        auto pose_of = [&](int at) __attribute__((always_inline)) {
            const float4 a = L.a[at];
            return make_float4(L.px[at], L.py[at], a.w, a.z);
        };
        // With the far field the items are taken sixteen steps of a sample at
        // a time: such poses lie close, so neighbouring lanes read the same
        // cells' lines (of the records and the costmap) and have like near
        // lists, where lanes of one step read a line each.
        auto in_order = [&](int o) __attribute__((always_inline)) {
            if constexpr (FIELD) {
                constexpr int kOrder = MODEL == MPPI_CAR ? 4 : 16;
                const int blk = o / (kOrder * S), r = o - blk * (kOrder * S), left = n - blk * kOrder;
                int t = r & (kOrder - 1), s = r / kOrder;
                if (left < kOrder) {        // the last, shorter block (r < 4096: exact)
                    s = (int)(((float)r + 0.5f) * __builtin_amdgcn_rcpf((float)left));
                    t = r - s * left;
                }
                return (blk * kOrder + t) * RS + s;
            }
            return slot(o);
        };
        auto next_unit = [&]() __attribute__((always_inline)) {
            int u = 0;
            if (lane == 0) u = atomicAdd(&L.next[c & 1], 1);
            return __builtin_amdgcn_readfirstlane(u);
        };
        for (int t = next_unit(); t < units; t = next_unit()) {
            const int u = t - xunits;
            const bool ends = u < 0;
            // lane `sp` of the item's 2^lg: neighbouring lanes (one run of
            // obstacles in LDS), with the far field lanes 64 / 2^lg apart
            int lgu = lg, item, sp, at, end = items;
            [[maybe_unused]] int rlg = 0;
            if (FIELD && !ends && u < ounits) {
                const int per = kWave >> lg;
                item = u * per + (lane & (per - 1));
                sp = lane >> (6 - lg);
            } else {
                int ul = u, first = 0;
                if constexpr (RUNS) {
                    const int part = u < u1 ? 0 : u < u2 ? 1 : 2;
                    lgu = run_lanes(p.run_lg, part);
                    rlg = run_split(p.run_lg, part);
                    ul -= part == 0 ? 0 : part == 1 ? u1 : u2;
                    first = (part == 0 ? 0 : part == 1 ? s1 : s2) * S;
                    end = (part == 0 ? s1 : part == 1 ? s2 : n) * S;
                }
                item = first + ((ul * kWave + lane) >> lgu);
                sp = lane & ((1 << lgu) - 1);
            }
            if (ends || u >= ounits) {
                if constexpr (MAP) {
                    const int it = !ends ? (u - ounits) * kWave + lane : t == 0 ? lane : kXSlots;
                    if (it < (ends ? kXSlots : items)) {
                        const int ma = ends ? n * RS + it : in_order(it);
                        L.mp[ma] = map_terms<PT, IND>(p, P, pose_of(ma), inv_res, offx, offy);
                    }
                }
                if (!ends) continue;
                lgu = rlg = RUNS ? run_split(p.run_lg, 0) : 5;
                item = (t * kWave + lane) >> lgu;
                sp = lane & ((1 << lgu) - 1);
                end = kXSlots;
                at = n * RS + item;
            } else {
                at = in_order(item);
            }
            const int nsp = 1 << lgu;
            // (with a far field, walks are FP64 sums until all lanes have met)
            using Part = std::conditional_t<FIELD && !IND, double, float>;
            Part part = IND ? (Part)INFINITY : (Part)0;
            if (item < end) {
                const float4 pose = pose_of(at);
                bool walk_all = true;
                if constexpr (FIELD) {
                    if (!ends) {
                        bool ok;
                        if constexpr (PT == 7) {
                            if (lgu == 0) part = field_barrier_axis<0>(p, L, cells, sa2, ss, pose, sp, omax2, ok);
                            else if (lgu == 1) part = field_barrier_axis<1>(p, L, cells, sa2, ss, pose, sp, omax2, ok);
                            else part = field_barrier_axis<2>(p, L, cells, sa2, ss, pose, sp, omax2, ok);
                        } else {
                            part = field_barrier_points<IND>(p, L, cells, P, pose, sp, lgu, ok);
                        }
                        walk_all = __ballot(!ok) != 0;
                    }
                }
                // A wave with a pose that has no cell walks before it has read a
                // record, and by its body's layout form, so that a world whose
                // poses mostly walk costs what it costs without a field: by
                // walk_points behind the whole lookup it cost up to 2.5 times
                // that (quadrotor K=14151 T=65, 326 obstacles within 5 m, 813
                // against 321 us; now within 10 % in 300 drawn worlds).
                if (walk_all) {
                    if constexpr (FIELD) rlg = lgu;
                    if constexpr (RUNS || PT != 0) {
                        part = fused_barrier_pose<MODEL, PT, FIELD>(p, L, sa2, sb2, ss, pose, sp, lgu, rlg, omax2);
                    } else if (VEHICLE && p.shape_kind == kShapeLayout) {
                        if constexpr (VEHICLE) {
                            float va2[8], vb2[8], vs[8];
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const float a = p.shape[i][0], b = p.shape[i][1];
                                va2[i] = uniform(2.0f * a);
                                vb2[i] = uniform(2.0f * b);
                                vs[i] = uniform(fmaf(a, a, b * b));
                            }
                            part = fused_barrier_pose<MODEL, 8, FIELD>(p, L, va2, vb2, vs, pose, sp, lgu, lgu, omax2);
                        }
                    } else {
                        part = walk_points<IND>(p, L, P, pose, sp, lgu);
                    }
                }
            }
            const int step = FIELD && !ends ? kWave >> lgu : 1;
            for (int m = step; m < step * nsp; m <<= 1) {
                const Part other = __shfl_xor(part, m);
                part = IND ? fminf(part, other) : part + other;
            }
            if (sp == 0 && item < end) L.b[at] = (float)part;
        }
    };

    // the fused barrier of slot idx with its costmap part
    auto barrier_at = [&](int idx) __attribute__((always_inline)) {
        float b = L.b[idx];
        if constexpr (MAP) b = IND ? fminf(b, L.mp[idx]) : b + L.mp[idx];
        return b;
    };
    // barrier-state recursion over chunk c (owner lanes) and its cost; with the
    // indicator, the weight of every step that violates a constraint
    auto beta_phase = [&](int c, int n) __attribute__((always_inline)) {
        const int tid = phase_tid();
        const float w = IND ? p.collision_weight : p.r_b;
        float beta = 0.0f;
        if constexpr (!IND) beta = c == 0 ? barrier_at(n * RS) : carry_b[tid];      // (from beta_0)
        walk(
            n, [&](int tt) __attribute__((always_inline)) { return barrier_at(tt * RS + tid); },
            [&](int, float b) __attribute__((always_inline)) {
                if constexpr (IND) {
                    cost += (double)(b < 0.0f ? w : 0.0f);
                } else {
                    beta = fmaf(p.gamma_b, beta, b);
                    cost += (double)(w * beta);
                }
            });
        if (!IND && c + 1 < nch) carry_b[tid] = beta;
    };

    for (int c = 0; c < nch; ++c) {
        const int t0 = c * tc, n = min(tc, T - t0);
        if (c == 0) {
            inputs_phase(0, n, 0);
        } else if (wave < DW) {
            if (owner) beta_phase(c - 1, tc);
        } else {
            inputs_phase(t0, n, POOL0);
        }
        lds_barrier();
        if (tid == kRollBlock - 1) L.next[(c + 1) & 1] = 0;
        if (owner) headings_phase(c, n);
        lds_barrier();
        sines_phase(n);
        if (!IND && c == 0 && tid >= kRollBlock - kXSlots) {
            // beta_0 and beta_d are the fused barriers of the poses of x0 and
            // x_d = x_ref[T], carried in chunk 0's two extra slots
            const int i = tid - (kRollBlock - kXSlots);
            const float* xd = L.ref + T * NS;
            float sn, cn;
            heading_sincos(i == 0 ? xs.v[2] : xd[2], sn, cn);
            L.a[n * RS + i] = make_float4(0.0f, 0.0f, sn, cn);
            L.px[n * RS + i] = i == 0 ? 0.0f : xd[0];
            L.py[n * RS + i] = i == 0 ? 0.0f : xd[1];
        }
        lds_barrier();
        if (tid < 2 * S) positions_phase(c, n);
        lds_barrier();
        tracking_cost(t0, n);
        lds_barrier();          // (the units write over the headings)
        units_phase(c, n);
        lds_barrier();
    }
    if (owner) beta_phase(nch - 1, T - (nch - 1) * tc);
    // the samples' costs: lanes of one sample within a wave, then the groups
    for (int m = S; m < kWave; m <<= 1) cost += __shfl_xor(cost, m);
    constexpr int RG = S < kWave ? kRollWaves : kRollBlock / S;
    lds_barrier();          // (the carried state is spent)
    if (S >= kWave) L.red[tid] = cost;                       // [tid / S][tid % S]
    else if (lane < S) L.red[wave * S + lane] = cost;
    lds_barrier();
    // (chunk 0's extra slots lie beyond every chunk's items)
    const float beta0 = IND ? 0.0f : barrier_at(min(tc, T) * RS), beta_d = IND ? 0.0f : barrier_at(min(tc, T) * RS + 1);
    const double cshift = (double)beta_d * p.beta_d_weight;
    double total = 0.0;
    if (owner) {
#pragma unroll
        for (int g = 0; g < RG; ++g) total += L.red[g * S + tid];
    }
    const float S_hi = (float)total;
    const float S_lo = isfinite(S_hi) ? (float)(total - (double)S_hi) : 0.0f;

    // ---- tile softmax partials ----
    // (global stores come after the block reductions, whose barriers would
    // otherwise wait for them)
    const double Sd = ((double)S_hi + (double)S_lo) + cshift;
    const bool ok = valid && isfinite(Sd);
    auto wants64 = [&](double rho) {
        return isfinite(rho) && (p.normaliser == MPPI_NORM_ON ||
                                 (p.normaliser == MPPI_NORM_AUTO && fabs(rho) >= 1024.0 * (double)p.lambda));
    };
    auto weight = [&](double rho, bool u64) {
        double ek = 0.0;
        if (ok) {
            const double d = (Sd - rho) / (double)p.lambda;
            ek = u64 ? exp(-d) : (double)expf(-(float)d);
        }
        return ek;
    };
    double rho_b, eta_b, ek = 0.0;
    if constexpr (DW == 1) {
        // every sample is on wave 0: reduce over its first S lanes and
        // publish through LDS behind one barrier
        if (wave == 0) {
            double m = ok ? Sd : INFINITY;
#pragma unroll
            for (int o = S / 2; o >= 1; o >>= 1) m = fmin(m, __shfl_xor(m, o));
            m = __shfl(m, 0);
            const bool u64 = wants64(m);
            ek = weight(m, u64);
            if (owner) L.e[tid] = ek;
            double es;
            if (u64) {
                es = ek;
#pragma unroll
                for (int o = S / 2; o >= 1; o >>= 1) es += __shfl_xor(es, o);
            } else {
                float ef = (float)ek;
#pragma unroll
                for (int o = S / 2; o >= 1; o >>= 1) ef += __shfl_xor(ef, o);
                es = (double)ef;
            }
            if (tid == 0) {
                L.slots[0] = m;
                L.slots[1] = es;
            }
        }
        lds_barrier();
        rho_b = L.slots[0];
        eta_b = L.slots[1];
    } else {
        rho_b = block_min_d<kRollWaves>(ok ? Sd : INFINITY, L.slots);
        ek = weight(rho_b, wants64(rho_b));
        if (owner) L.e[tid] = ek;
        if (wants64(rho_b)) eta_b = block_sum_d<kRollWaves>(ek, L.slots);
        else eta_b = (double)block_sum_f<kRollWaves>((float)ek, L.slots);
    }
    const bool any = isfinite(rho_b);
    const bool use64 = wants64(rho_b);

    // N_b[2t + c] = sum over the tile's samples of e_k du[t][c][k].  The
    // noise is never stored in device memory on the way: it is kept in LDS
    // when it fits and otherwise drawn again from its counter, bit-identical
    // to the inputs phase (and written out here only when the controller
    // exports it).  TPT consecutive threads share a step t, each
    // summing every TPT-th sample in order, then combining across the TPT
    // threads.
    // (at least eight samples per thread: fewer shuffle rounds)
    int tpt = 1;
    while (tpt < 64 && (tpt << 1) * T <= kRollBlock && (tpt << 1) * 8 <= S) tpt <<= 1;
    const int steps_per_pass = kRollBlock / tpt;
    const int part = tid & (tpt - 1);
    const int k0 = tile * S;
    const int nk = min(S, K - k0);
    const bool store_du = p.export_noise != 0;
    // with smoothing, the unsmoothed sums gather in the (spent) chunk slots
    const bool smooth = p.sgf_m > 0;
    double* nb = reinterpret_cast<double*>(L.a);
    for (int q0 = 0; q0 < T; q0 += steps_per_pass) {
        const int t = q0 + tid / tpt;
        double o0, o1;
        if (use64) {
            double a0 = 0.0, a1 = 0.0;
            if (t < T) {
                for (int s = part; s < nk; s += tpt) {
                    const float2 z = keep_noise ? L.nz[t * S + s] : noise_at(k0 + s, t);
                    if (store_du) {
                        p.du[(size_t)(2 * t) * Kp + k0 + s] = z.x;
                        p.du[(size_t)(2 * t + 1) * Kp + k0 + s] = z.y;
                    }
                    a0 += L.e[s] * (double)z.x;
                    a1 += L.e[s] * (double)z.y;
                }
            }
            for (int m = 1; m < tpt; m <<= 1) {
                a0 += __shfl_xor(a0, m);
                a1 += __shfl_xor(a1, m);
            }
            o0 = a0;
            o1 = a1;
        } else {
            float a0 = 0.0f, a1 = 0.0f;
            if (t < T) {
                for (int s = part; s < nk; s += tpt) {
                    const float2 z = keep_noise ? L.nz[t * S + s] : noise_at(k0 + s, t);
                    if (store_du) {
                        p.du[(size_t)(2 * t) * Kp + k0 + s] = z.x;
                        p.du[(size_t)(2 * t + 1) * Kp + k0 + s] = z.y;
                    }
                    a0 = fmaf((float)L.e[s], z.x, a0);
                    a1 = fmaf((float)L.e[s], z.y, a1);
                }
            }
            for (int m = 1; m < tpt; m <<= 1) {
                a0 += __shfl_xor(a0, m);
                a1 += __shfl_xor(a1, m);
            }
            o0 = (double)a0;
            o1 = (double)a1;
        }
        if (part == 0 && t < T) {
            if (smooth) {
                nb[2 * t] = o0;
                nb[2 * t + 1] = o1;
            } else {
                p.partN[(size_t)(2 * t) * p.tiles + tile] = any ? o0 : 0.0;
                p.partN[(size_t)(2 * t + 1) * p.tiles + tile] = any ? o1 : 0.0;
            }
        }
    }
    // Algorithm 1's Savitzky-Golay smoothing of the weighted increment is
    // linear along the horizon, so it is applied to the tile's own sums:
    // N_b[t][c] <- sum_j a_tj N_b[s_t + j][c] over the window of step t.
    if (smooth) {
        __syncthreads();
        const int m = p.sgf_m, Wn = 2 * m + 1;
        for (int r = tid; r < 2 * T; r += kRollBlock) {
            const int t = r >> 1, c = r & 1;
            const int s0 = min(max(t - m, 0), T - Wn);
            const float* a = p.sgf_coef + (size_t)t * Wn;
            double v = 0.0;
            for (int j = 0; j < Wn; ++j) v += (double)a[j] * nb[2 * (s0 + j) + c];
            p.partN[(size_t)r * p.tiles + tile] = any ? v : 0.0;
        }
    }
    if (valid) {
        p.S[k] = S_hi;
        p.S[Kp + k] = S_lo;
        p.e[k] = (float)ek;
    }
    if (tid == 0) {
        p.rho_b[tile] = rho_b;
        p.eta_b[tile] = any ? eta_b : 0.0;
        p.flag_b[tile] = use64 ? 1 : 0;
        if (tile == 0) {
            // identical in every tile; the update kernel reports them
            CtrlState* st = p.st;
            st->beta0 = beta0;
            st->beta_d = beta_d;
            st->cshift = cshift;
        }
    }
}

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------
// Workgroups are handed to the chip's 8 XCDs in turn (workgroup i to XCD
// i mod 8).  The tile of workgroup i makes each XCD take a contiguous run of
// tiles, so the tiles whose partial sums share a line of the [2T][tiles]
// layout write it from one L2 (a bijection on [0, tiles) for any count).
constexpr int kXcds = 8;

__device__ __forceinline__ int xcd_tile(int i, int tiles)
{
    const int x = i % kXcds, j = i / kXcds;
    const int q = tiles / kXcds, r = tiles % kXcds;
    return x * q + min(x, r) + j;
}

// The kernel's arguments (the parameter block, then the step's arguments)
// are read field by field through the prologue, and each first touch of one
// of their lines would wait on memory in turn.  One word of every 64-byte
// line of the first Bytes bytes is loaded here, all in one batch, so the
// later loads hit the scalar cache.
template <int Bytes>
__device__ __forceinline__ void touch_kernargs()
{
    using KWord = const __attribute__((address_space(4))) uint32_t;
    KWord* kp = (KWord*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t t = 0;
#pragma unroll
    for (int i = 0; i < Bytes / 4; i += 16) t ^= kp[i];
    asm volatile("" ::"s"(t));
}

template <int MODEL, int S, int PT, bool IND, bool MAP, bool FIELD>
__global__ __launch_bounds__(kRollBlock) void k_rollout(DevParams p, StepArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NS = Model<MODEL>::NS;
    touch_kernargs<(int)(sizeof(DevParams) + sizeof(StepArgs))>();
    X0 xs;
    if (a.x0_ptr) {
        // the state's NS words, unconditionally, so the loads issue together
#pragma unroll
        for (int i = 0; i < MPPI_NMAX + 2; ++i) xs.v[i] = i < NS ? a.x0_ptr[i] : 0.0f;
    } else {
#pragma unroll
        for (int i = 0; i < MPPI_NMAX + 2; ++i) xs.v[i] = a.x0[i];
    }
    xs.parity = a.parity;
    const bool own = a.S_e > 0.0f;
    xs.S_e = own ? a.S_e : p.st->S_e;
    xs.counter = own ? a.counter : p.st->counter;
    rollout_tile<MODEL, S, PT, IND, MAP, FIELD>(p, xcd_tile((int)blockIdx.x, p.tiles), xs, smem);
}

// Persistent rollout over a work list of (controller, tile) units of one
// tile shape, taken in list order (the host sorts it longest-first): the
// tile of the standalone kernel of that shape.  Every block leaves the loop
// once the list is exhausted; the last block to leave resets the queue.
template <int MODEL, int S, int PT, bool IND, bool MAP, bool FIELD>
__global__ __launch_bounds__(kRollBlock) void k_batch_rollout(const DevParams* __restrict__ ps,
                                                              const BatchUnit* __restrict__ units, int nunits,
                                                              const BatchIn* __restrict__ in, uint32_t* queue)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_unit;
    for (;;) {
        if (threadIdx.x == 0) s_unit = (int)atomicAdd(&queue[0], 1u);
        __syncthreads();
        const int u = s_unit;
        __syncthreads();
        if (u >= nunits) break;
        const BatchUnit bu = units[u];
        const DevParams& p = ps[bu.ctrl];
        X0 xs;
#pragma unroll
        for (int i = 0; i < MPPI_NMAX + 2; ++i) xs.v[i] = in[bu.ctrl].x0[i];
        xs.parity = in[bu.ctrl].parity;
        xs.S_e = p.st->S_e;
        xs.counter = p.st->counter;
        rollout_tile<MODEL, S, PT, IND, MAP, FIELD>(p, bu.tile, xs, smem);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&queue[1], 1u) == gridDim.x - 1u) {
            queue[0] = 0u;
            queue[1] = 0u;
        }
    }
}

// The tile kinds of a model: layout form, runtime P, indicator, each without
// and with a costmap, then the same six with the obstacles' far field.  (The
// vehicle's field takes every body a point at a time: its layout form is its
// runtime-P form there.)
template <int MODEL, int S, template <int, int, int, bool, bool, bool> class K>
auto kernel_of_kind(int kind)
{
    constexpr int PD = MODEL == MPPI_CAR ? 8 : 7, PF = MODEL == MPPI_CAR ? 0 : 7;
    switch (kind) {
    case 0: return K<MODEL, S, PD, false, false, false>::get();
    case 1: return K<MODEL, S, PD, false, true, false>::get();
    case 2: return K<MODEL, S, 0, false, false, false>::get();
    case 3: return K<MODEL, S, 0, false, true, false>::get();
    case 4: return K<MODEL, S, 0, true, false, false>::get();
    case 5: return K<MODEL, S, 0, true, true, false>::get();
    case 6: return K<MODEL, S, PF, false, false, true>::get();
    case 7: return K<MODEL, S, PF, false, true, true>::get();
    case 8: return K<MODEL, S, 0, false, false, true>::get();
    case 9: return K<MODEL, S, 0, false, true, true>::get();
    case 10: return K<MODEL, S, 0, true, false, true>::get();
    default: return K<MODEL, S, 0, true, true, true>::get();
    }
}

template <int MODEL, int S, int PT, bool IND, bool MAP, bool FIELD> struct StepKernel {
    static auto get() { return &k_rollout<MODEL, S, PT, IND, MAP, FIELD>; }
};
template <int MODEL, int S, int PT, bool IND, bool MAP, bool FIELD> struct BatchKernel {
    static auto get() { return &k_batch_rollout<MODEL, S, PT, IND, MAP, FIELD>; }
};

// The kernel of `key` (kind key / kTileSizes, tile size 16 << key % kTileSizes).
template <int MODEL, template <int, int, int, bool, bool, bool> class K>
auto kernel_of(int key)
{
    const int kind = key / kTileSizes;
    switch (key % kTileSizes) {
    case 0: return kernel_of_kind<MODEL, 16, K>(kind);
    case 1: return kernel_of_kind<MODEL, 32, K>(kind);
    case 2: return kernel_of_kind<MODEL, 64, K>(kind);
    case 3: return kernel_of_kind<MODEL, 128, K>(kind);
    default: return kernel_of_kind<MODEL, 256, K>(kind);
    }
}

template <int MODEL>
BatchRolloutKernel batch_kernel_of(int key) { return kernel_of<MODEL, BatchKernel>(key); }

template <int MODEL>
hipError_t launch_rollout_m(const DevParams& p, const StepArgs& a, size_t lds, hipStream_t s)
{
    const auto k = kernel_of<MODEL, StepKernel>(tile_key(p));
    hipLaunchKernelGGL(k, dim3(p.tiles), dim3(kRollBlock), lds, s, p, a);
    return hipGetLastError();
}

}  // namespace
}  // namespace dbas
