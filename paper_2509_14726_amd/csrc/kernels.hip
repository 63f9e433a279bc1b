// Kernels of one MPPI step on gfx950 (wave64).
//
//   k_setup          once per context: problem tables -> device layout in Real
//   k_rollout4       (default for small K) a 64-sample tile per workgroup, the
//                    step pipelined over its waves: noise and clipped samples
//                    (Eq. (3)), RK4 of Eq. (2) split into body rates, attitude
//                    and translation, per-step costs fused in (gate Eq. (6)-(7),
//                    tracking Eq. (8), contouring Eq. (9)); cost write and the
//                    smallest cost of the tile
//   k_rollout_rate   the pipeline for the rate input
//   k_rollout3       three waves, chunks of steps between barriers
//   k_rollout_pair   (binary32, medium K) the one-wave rollout's arithmetic on
//                    two waves: draws and costs | motion
//   k_sample +       (large K) noise and clipped samples for all (m, k), then
//   k_rollout /      one sample per lane (k_rollout; drawing itself after k_head
//   k_rollout_split  where the sample tensor is large) or attitude and
//                    translation on two waves (k_rollout_split)
//   k_final          one block per horizon step: J_min from the tile minima,
//                    softmax weights (Eq. (4)), the weighted average (Eq. (5)),
//                    the first input, the report and the warm-start hand-over
//   kb_*             the same bodies as persistent kernels over a batch
//                    (kb_rollout_draw: the one-wave rollouts that draw)
#include <hip/hip_runtime.h>
#include <math.h>

#include <mutex>
#include <type_traits>

#include "../../include/mppi.h"

#include "device.hpp"
#include "kernels.hpp"
#include "noise.hpp"
#include "rollout.hpp"

namespace mppi {

template <typename Real> struct Vec4;
template <> struct Vec4<float> { using T = float4; };
template <> struct Vec4<double> { using T = double4; };

// Streaming (non-temporal) stores of the sample tensor from the pipelined
// rollouts: the tensor is read once, by the weighted-average kernel, and
// written this way it leaves no dirty L2 lines to write back when the rollout
// kernel ends.
__device__ __forceinline__ void store_nt(float4 *p, const float4 v)
{
    typedef float V __attribute__((ext_vector_type(4)));
    const V x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, (V *)p);
}
__device__ __forceinline__ void store_nt(double4 *p, const double4 v)
{
    typedef double V __attribute__((ext_vector_type(4)));
    const V x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, (V *)p);
}
__device__ __forceinline__ void store_nt(float *p, const float v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ void store_nt(double *p, const double v) { __builtin_nontemporal_store(v, p); }

// Arguments that a batched kernel holds in LDS.  The compiler does not know the
// address space of a pointer read from there: its accesses would be flat ones,
// each of which waits for all that went before (a load behind the streaming
// store of a sample for that store).  in_global() names it.
struct StagedArgs : KArgs {};
template <typename Args, typename T> __device__ __forceinline__ T *in_global(const Args &, T *p)
{
    if constexpr (std::is_same<Args, StagedArgs>::value) return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
    else return p;
}

// ---------------------------------------------------------------- setup

template <typename Real> __global__ void k_setup(KArgs a)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < a.G && a.gates_d) {
        // gate frame (centre, normal n, lateral h) in binary64 for the head
        // and in Real for the rollouts; the yaw's cosine and sine are taken
        // once here
        const double *g = a.gates_d + 4 * i;
        double *f = (double *)a.gates_d + 4 * a.G + 8 * i;
        const double cy = cos(g[3]), sy = sin(g[3]);
        f[0] = g[0]; f[1] = g[1]; f[2] = g[2];
        f[3] = cy; f[4] = sy;
        f[5] = -sy; f[6] = cy;
        f[7] = 0.0;
        Real *o = (Real *)a.gates_r + 8 * i;
        o[0] = (Real)g[0]; o[1] = (Real)g[1]; o[2] = (Real)g[2];
        o[3] = (Real)cy; o[4] = (Real)sy;     // normal n
        o[5] = (Real)(-sy); o[6] = (Real)cy;  // lateral h
        o[7] = Real(0);
    }
    if (i < a.P && a.path_d) {
        const double *p = a.path_d + 6 * i;
        Real *o = (Real *)a.path_r + 8 * i;
        for (int c = 0; c < 6; ++c) o[c] = (Real)p[c];
        o[6] = o[7] = Real(0);
    }
    if (i < a.R && a.xref_r) {
        // the FP64 reference was staged in the upper half of the same buffer
        const double *r = (const double *)((const char *)a.xref_r + (size_t)a.R * 16 * sizeof(Real)) + 13 * i;
        Real *o = (Real *)a.xref_r + 16 * i;
        for (int c = 0; c < 13; ++c) o[c] = (Real)r[c];
        o[13] = o[14] = o[15] = Real(0);
    }
}

// ---------------------------------------------------------------- head

// Measured gate pass x_prev -> x0 (same geometry as the in-horizon switch);
// gate = the binary64 frame (centre, n, h) written at set-up.
__device__ bool gate_cross_d(const double *pa, const double *pb, const double *gate, double half)
{
    const double nx = gate[3], ny = gate[4];
    const double hx = gate[5], hy = gate[6];
    const double sa = (pa[0] - gate[0]) * nx + (pa[1] - gate[1]) * ny;
    const double sb = (pb[0] - gate[0]) * nx + (pb[1] - gate[1]) * ny;
    if (!(sa < 0.0 && sb >= 0.0)) return false;
    const double t = sa / (sa - sb);
    const double y0 = pa[0] + t * (pb[0] - pa[0]);
    const double y1 = pa[1] + t * (pb[1] - pa[1]);
    const double y2 = pa[2] + t * (pb[2] - pa[2]);
    const double lat = (y0 - gate[0]) * hx + (y1 - gate[1]) * hy;
    const double ver = y2 - gate[2];
    return fabs(lat) <= half && fabs(ver) <= half;
}

__device__ double wrap_len_d(double th, double L)
{
    double r = fmod(th, L);
    if (r < 0.0) r += L;
    if (r >= L) r -= L;
    return r;
}

// What one solve inherits from the previous one, decided from the request and
// the warm-start state: warm-start shift, current gate and pass mask, start
// arc length, reference row, last applied input.
struct HeadVals {
    int32_t g0, i0, shift, warm;
    uint32_t s;
    uint32_t allow[kMaskWords];
    double theta0, t_now, v_prev;
    double u_prev[4];
    double x0[13];
};

// Steps the warm start is shifted by: none in an inner iteration of the same
// control step (the previous iteration ran at this time), else
// max(1, round(elapsed / dt)).
__device__ __forceinline__ int warm_shift(const KArgs &a, int warm, double t_now, double t_prev)
{
    if (a.inner && warm && t_prev == t_now) return 0;
    return solve_shift(warm, t_now, t_prev, a.dt);
}

// Rate model, contouring: the progress speed state at this solve's time, the
// previous solve's initial speed advanced over the shift by its averaged
// accelerations (clamped to [0, v_max] each step) and held beyond that
// solution's horizon; 0 at a cold start.
__device__ __forceinline__ double rate_speed0(const KArgs &a, const DevWarm *w, int warm, int shift)
{
    if (!warm) return 0.0;
    double v = w->vtheta;
    for (int j = 0; j < shift && j < a.N; ++j) v = clampT(v + a.dt * a.wV[j], 0.0, a.v_max);
    return v;
}

// Minimum over the 64 lanes of a wave (all lanes active), returned to every
// lane.  Binary32 goes through DPP moves, each a few cycles instead of an
// LDS-crossbar round trip: two quad permutes ([1,0,3,2], [2,3,0,1]), row
// shifts by 4 and 8 (lane 15 of each row then holds the row's minimum), the
// broadcast of lane 15 into rows 1 and 3 and of lane 31 into rows 2 and 3
// (lane 63 then holds the wave's minimum); a lane without a source keeps
// +inf.  Binary64 and integers use lane shuffles.  A minimum does not depend
// on the order of the comparisons, so either way every caller sees the same
// value.
template <int CTRL, int ROW_MASK = 0xf> __device__ __forceinline__ float dpp_or_inf(float v)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(INFINITY), __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}

__device__ __forceinline__ float wave_min(float v)
{
    float o;
    o = dpp_or_inf<0xb1>(v);       v = o < v ? o : v;
    o = dpp_or_inf<0x4e>(v);       v = o < v ? o : v;
    o = dpp_or_inf<0x114>(v);      v = o < v ? o : v;
    o = dpp_or_inf<0x118>(v);      v = o < v ? o : v;
    o = dpp_or_inf<0x142, 0xa>(v); v = o < v ? o : v;
    o = dpp_or_inf<0x143, 0xc>(v); v = o < v ? o : v;
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

template <typename T> __device__ __forceinline__ T wave_min(T v)
{
    for (int off = 32; off > 0; off >>= 1) {
        const T o = __shfl_xor(v, off, 64);
        v = o < v ? o : v;
    }
    return v;
}

// Run by all threads of one block (whole waves, up to 1024 threads); h is in LDS.  A
// kernel built for another objective than contouring passes CONTOUR = false
// and allocates no LDS for the projection.
template <bool CONTOUR = true> __device__ void compute_head(const KArgs &a, HeadVals &h)
{
    const int tid = threadIdx.x;
    const DevWarm *w = a.warm;
    const int warm = w->warm;

    double theta0 = 0.0;
    if (CONTOUR && a.objective == OBJ_CONTOUR) {
        __shared__ double s_d2[16], s_th[16];   // one entry per wave
        __shared__ int s_j[16];
        // the block size, read once (a read from the dispatch's implicit
        // arguments, which inside the barrier loop below would be repeated
        // at every barrier)
        const int nthr = (int)blockDim.x;
        const int P = a.P;
        const double L = a.path_len, ds = L / (double)P;
        const bool global = !warm;
        const int W = a.proj_window;
        int ic = 0;
        if (!global) {
            ic = (int)floor(wrap_len_d(w->theta0, L) / ds);
            if (ic >= P) ic = P - 1;
        }
        const int count = global ? P : 2 * W + 1;
        double best = INFINITY, best_th = 0.0;
        int best_j = 0x7fffffff;
        const double p0 = a.req[0], p1 = a.req[1], p2 = a.req[2];
        for (int j = tid; j < count; j += nthr) {
            const int i = global ? j : (((ic + (j - W)) % P) + P) % P;
            const int i1 = (i + 1) % P;
            const double *A = a.path_d + 6 * i, *B = a.path_d + 6 * i1;
            const double ab0 = B[0] - A[0], ab1 = B[1] - A[1], ab2 = B[2] - A[2];
            const double ap0 = p0 - A[0], ap1 = p1 - A[1], ap2 = p2 - A[2];
            const double l2 = ab0 * ab0 + ab1 * ab1 + ab2 * ab2;
            double t = l2 > 0.0 ? (ap0 * ab0 + ap1 * ab1 + ap2 * ab2) / l2 : 0.0;
            t = t < 0.0 ? 0.0 : (t > 1.0 ? 1.0 : t);
            const double d0 = ap0 - t * ab0, d1 = ap1 - t * ab1, d2 = ap2 - t * ab2;
            const double dd = d0 * d0 + d1 * d1 + d2 * d2;
            if (dd < best) { best = dd; best_th = ((double)i + t) * ds; best_j = j; }
        }
        // smallest distance, ties to the first candidate in search order: in
        // each wave, then over the waves' results, with one barrier (a tree of
        // barriers over all threads took nine, and 10 KB of LDS)
        const double wd = wave_min(best);
        const int wj = wave_min(best == wd ? best_j : 0x7fffffff);
        if (best == wd && best_j == wj) { s_d2[tid >> 6] = wd; s_th[tid >> 6] = best_th; s_j[tid >> 6] = wj; }
        __syncthreads();
        double md = s_d2[0], mt = s_th[0];
        int mj = s_j[0];
        for (int i = 1; i < (nthr >> 6); ++i) {
            const double d_o = s_d2[i];
            if (d_o < md || (d_o == md && s_j[i] < mj)) { md = d_o; mj = s_j[i]; mt = s_th[i]; }
        }
        theta0 = wrap_len_d(mt, L);
    }

    if (tid == 0) {
        const double t_now = a.req[13];
        int g0 = w->g0;
        uint32_t allow[kMaskWords];
        for (int j = 0; j < kMaskWords; ++j) allow[j] = warm ? w->allow[j] : 0xffffffffu;
        if (warm && a.objective == OBJ_GATE && g0 >= 0 && g0 < a.G &&
            gate_cross_d(w->x_prev, a.req, a.gates_d + 4 * a.G + 8 * g0, a.gate_half)) {
            g0 = (g0 + 1) % a.G;
            for (int j = 0; j < kMaskWords; ++j) allow[j] = 0xffffffffu;
        }
        int i0 = 0;
        if (a.objective == OBJ_TRACK) {
            double r = floor(t_now / a.ref_dt + 0.5);
            if (!(r >= 0.0)) r = 0.0;
            if (r > (double)(a.R - 1)) r = (double)(a.R - 1);
            i0 = (int)r;
        }
        h.g0 = g0;
        h.i0 = i0;
        h.shift = warm_shift(a, warm, t_now, w->t_prev);
        h.warm = warm;
        h.s = w->s;
        for (int j = 0; j < kMaskWords; ++j) h.allow[j] = allow[j];
        h.theta0 = theta0;
        h.t_now = t_now;
        // an inner iteration keeps the last applied input of the control step,
        // which the previous iteration published
        const bool same_step = a.inner && warm && w->t_prev == t_now;
        for (int i = 0; i < 4; ++i) h.u_prev[i] = same_step ? a.cur->u_prev[i] : (warm ? a.wU[i] : a.hover);
        h.v_prev = same_step ? a.cur->v_prev : (warm ? a.wV[0] : 0.0);
        // the rate model carries the progress speed state in v_prev
        if (a.input_model == INPUT_RATE) h.v_prev = rate_speed0(a, w, warm, h.shift);
        for (int i = 0; i < 13; ++i) h.x0[i] = a.req[i];
    }
    __syncthreads();
}

// Publish the head for the kernels that follow (thread 0 of one block).
__device__ void publish_head(const KArgs &a, const HeadVals &h)
{
    DevCur *c = a.cur;
    c->g0 = h.g0;
    c->i0 = h.i0;
    c->shift = h.shift;
    c->warm = h.warm;
    c->s = h.s;
    for (int j = 0; j < kMaskWords; ++j) c->allow[j] = h.allow[j];
    c->theta0 = h.theta0;
    c->t_now = h.t_now;
    for (int i = 0; i < 4; ++i) c->u_prev[i] = h.u_prev[i];
    c->v_prev = h.v_prev;
    for (int i = 0; i < 13; ++i) c->x0[i] = h.x0[i];
}

__device__ void solve_head(const KArgs &a)
{
    __shared__ HeadVals h;
    compute_head(a, h);
    if (threadIdx.x == 0) {
        publish_head(a, h);
        a.cur->J_nom = 0.0;
    }
}

// ---------------------------------------------------------------- sample

// One block of 256 samples over the steps [k0, k1); the block of the first
// samples and steps also runs the head.  The shifted warm start (R4 per step)
// is staged in LDS once, so each step is the noise and the clipped samples of
// 256 samples with one coalesced store.  Every sample and step is drawn from
// its own counters, so any split of the steps gives the same samples.
template <typename Real, bool HAS_V>
__device__ __forceinline__ void sample_body(const KArgs &a, int bx, int k0, int k1)
{
    typedef typename Vec4<Real>::T R4;
    __shared__ R4 s_us[kNMax];
    __shared__ Real s_vs[HAS_V ? kNMax : 1];
    if (bx == 0 && k0 == 0) solve_head(a);

    // nominal of this solve: the previous solution shifted, or hover (cold)
    const DevWarm *w = a.warm;
    const int warm = w->warm;
    const int shift = warm_shift(a, warm, a.req[13], w->t_prev);
    const uint32_t s = w->s;
    const int N = a.N, K = a.K;
    for (int k = k0 + (int)threadIdx.x; k < k1; k += blockDim.x) {
        int src = k + shift;
        if (src > N - 1) src = N - 1;
        R4 o;
        o.x = warm ? (Real)a.wU[4 * src + 0] : (Real)a.hover;
        o.y = warm ? (Real)a.wU[4 * src + 1] : (Real)a.hover;
        o.z = warm ? (Real)a.wU[4 * src + 2] : (Real)a.hover;
        o.w = warm ? (Real)a.wU[4 * src + 3] : (Real)a.hover;
        s_us[k] = o;
        if (HAS_V) s_vs[k] = warm ? (Real)a.wV[src] : Real(0);
    }
    __syncthreads();

    const int m = bx * 256 + threadIdx.x;
    const Real tmin = (Real)a.t_min, tmax = (Real)a.t_max;
    if (a.input_model == INPUT_RATE) {
        // the paper's input: thrust rates (and contouring's progress
        // acceleration) clipped to their bounds.  The clip to the range that
        // keeps each thrust within [t_min, t_max] (the speed within [0, v_max])
        // follows the sample's own thrust chain: the rollout applies it step
        // by step, where that chain is integrated, and writes the result back.
        if (m > K) return;
        const bool noisy = m < K;
        const Real rlo = (Real)a.rate_lim[0], rhi = (Real)a.rate_lim[1];
        const Real dlo = (Real)a.dv_lim[0], dhi = (Real)a.dv_lim[1];
        const Real sg[4] = {(Real)a.sigma[0], (Real)a.sigma[1], (Real)a.sigma[2], (Real)a.sigma[3]};
#pragma unroll 2
        for (int k = k0; k < k1; ++k) {
            const R4 us = s_us[k];
            const Real ust[4] = {us.x, us.y, us.z, us.w};
            Real z[4] = {Real(0), Real(0), Real(0), Real(0)};
            if (noisy) {
                const Normal4<Real> n4 = normals4<Real>((uint32_t)m, (uint32_t)k, s, 0u, a.seed_lo, a.seed_hi);
                z[0] = n4.z0; z[1] = n4.z1; z[2] = n4.z2; z[3] = n4.z3;
            }
            Real u[4];
            for (int i = 0; i < 4; ++i) u[i] = clamp_finite(noisy ? ust[i] + sg[i] * z[i] : ust[i], rlo, rhi);
            R4 o;
            o.x = u[0]; o.y = u[1]; o.z = u[2]; o.w = u[3];
            if (noisy) ((R4 *)a.ctrl)[(size_t)k * (size_t)K + (size_t)m] = o;
            else ((R4 *)a.nomU)[k] = o;
            if (HAS_V) {
                Real zv = Real(0);
                if (noisy) zv = normal1<Real>((uint32_t)m, (uint32_t)k, s, 1u, a.seed_lo, a.seed_hi);
                const Real acc = clamp_finite(noisy ? s_vs[k] + (Real)a.sigma_v * zv : s_vs[k], dlo, dhi);
                if (noisy) ((Real *)a.vctrl)[(size_t)k * (size_t)K + (size_t)m] = acc;
                else ((Real *)a.nomV)[k] = acc;
            }
        }
        return;
    }
    if (m == K) {  // the noise-free sample
        for (int k = k0; k < k1; ++k) {
            const R4 us = s_us[k];
            R4 o;
            o.x = clampT(us.x, tmin, tmax); o.y = clampT(us.y, tmin, tmax);
            o.z = clampT(us.z, tmin, tmax); o.w = clampT(us.w, tmin, tmax);
            ((R4 *)a.nomU)[k] = o;
            if (HAS_V) ((Real *)a.nomV)[k] = clampT(s_vs[k], Real(0), (Real)a.v_max);
        }
    } else if (m < K) {
        const Real sig0 = (Real)a.sigma[0], sig1 = (Real)a.sigma[1];
        const Real sig2 = (Real)a.sigma[2], sig3 = (Real)a.sigma[3];
#pragma unroll 2
        for (int k = k0; k < k1; ++k) {
            const R4 us = s_us[k];
            const Normal4<Real> z = normals4<Real>((uint32_t)m, (uint32_t)k, s, 0u, a.seed_lo, a.seed_hi);
            R4 o;
            o.x = clampT(us.x + sig0 * z.z0, tmin, tmax);
            o.y = clampT(us.y + sig1 * z.z1, tmin, tmax);
            o.z = clampT(us.z + sig2 * z.z2, tmin, tmax);
            o.w = clampT(us.w + sig3 * z.z3, tmin, tmax);
            const size_t idx = (size_t)k * (size_t)K + (size_t)m;
            ((R4 *)a.ctrl)[idx] = o;
            if (HAS_V) {
                const Real zv = normal1<Real>((uint32_t)m, (uint32_t)k, s, 1u, a.seed_lo, a.seed_hi);
                ((Real *)a.vctrl)[idx] = clampT(s_vs[k] + (Real)a.sigma_v * zv, Real(0), (Real)a.v_max);
            }
        }
    }
    __syncthreads();
}

// Steps per block of the sample kernel: the draws are independent, so the
// grid spreads them over (samples, steps) and every CU takes a share.
constexpr int kSampleSteps = 4;

template <typename Real, bool HAS_V> __global__ __launch_bounds__(256) void k_sample(KArgs a)
{
    const int k0 = (int)blockIdx.y * kSampleSteps;
    sample_body<Real, HAS_V>(a, blockIdx.x, k0, min(a.N, k0 + kSampleSteps));
}

// The head, for a rollout that draws its samples itself (one-wave layout): one
// block.
template <bool CONTOUR> __global__ __launch_bounds__(256) void k_head(KArgs a)
{
    __shared__ HeadVals h;
    compute_head<CONTOUR>(a, h);
    if (threadIdx.x == 0) {
        publish_head(a, h);
        a.cur->J_nom = 0.0;
    }
}

// ---------------------------------------------------------------- rollout

// Smallest finite sample cost of a 64-sample tile (+inf when there is none),
// stored by lane 0 of the wave that holds the tile's costs.  The weighted
// average takes J_min as the minimum over tiles: no atomics, nothing to reset.
template <typename Real> __device__ __forceinline__ void store_tile_min(Real v, bool use, void *tmin, int tile)
{
    v = wave_min(use ? v : Real(INFINITY));
    if ((threadIdx.x & 63) == 0) ((Real *)tmin)[tile] = v;
}

template <typename Real> struct GateRegs {
    Real cx, cy, cz, nx, ny, hx, hy;
    __device__ __forceinline__ void load(const Real *tab, int g)
    {
        const Real *r = tab + 8 * g;
        cx = r[0]; cy = r[1]; cz = r[2]; nx = r[3]; ny = r[4]; hx = r[5]; hy = r[6];
    }
};

// A value in vector registers.  Operations with a scalar-register operand
// issue at half the rate of those that read vector registers and literals
// only (4.3 against 2.5 cycles per wave and SIMD, measured with four waves),
// so the constants of the issue-bound rollout are held in vector registers.
template <typename T> __device__ __forceinline__ T in_vgpr(T x)
{
    asm volatile("" : "+v"(x));
    return x;
}
template <typename Real> __device__ __forceinline__ void in_vgpr(Model<Real> &M)
{
    M.inv_m = in_vgpr(M.inv_m); M.g = in_vgpr(M.g); M.arm_s = in_vgpr(M.arm_s); M.c_tau = in_vgpr(M.c_tau);
    M.ijx = in_vgpr(M.ijx); M.ijy = in_vgpr(M.ijy); M.ijz = in_vgpr(M.ijz);
    M.gx = in_vgpr(M.gx); M.gy = in_vgpr(M.gy); M.gz = in_vgpr(M.gz);
}

// What a wave waits for before it starts a step: each lane watches one
// counter; step k may start once every lane's counter plus its offset is
// above k (offset 0: the producer has done step k; a ring's size: the slot of
// step k has been read).  LDS operations of one wave execute in order, so a
// data read issued after the counter read sees what was written before the
// counter was, and a counter written after the data never overtakes it: the
// compiler is held to that order, the hardware needs no wait for it.
struct PipeWatch {
    const int *c;
    int off;
    __device__ __forceinline__ int peek() const
    {
        return __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) + off;
    }
    static __device__ __forceinline__ bool may_start(int seen, int k)
    {
        const bool r = __builtin_amdgcn_ballot_w64(seen > k) == ~0ull;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "singlethread");
        return r;
    }
    template <int SLEEP> __device__ __forceinline__ void wait(int k) const
    {
        while (!may_start(peek(), k)) __builtin_amdgcn_s_sleep(SLEEP);
    }
};
// Lane 0 writes the counter, the other lanes a word that nothing reads: no
// change of the execution mask, so the steps around it stay one block.
__device__ __forceinline__ void pipe_publish(int *c, int v)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "singlethread");
    __hip_atomic_store(c, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "singlethread");
}

// One tile on two waves: one wave draws the samples and sums the costs, the
// other moves the state (all in the arithmetic and order of the one-wave
// rollout, so the results are the same bit for bit).  The draws run kPairAhead
// steps ahead of the costs, the motion in between.
//
// Where the one-wave rollout leaves a single wave per SIMD (two to four tiles
// per CU), its operations issue at half the rate that two waves reach, so the
// two parts run beside each other, and no sample kernel writes what this one
// reads: K = 65000, N = 100 120 -> 98 us a solve, tracking K = 50011, N = 33
// 60 -> 42.
enum RolloutPart { PART_ALL = 0, PART_COSTS = 1, PART_MOTION = 2 };
constexpr int kPairRing = 4, kPairAhead = 3;
// Slot k mod kPairRing of a ring is written again by step k + kPairRing.  The
// costs publish the input of step i once they have read the motion of step
// i - 1 - kPairAhead, and the motion of step i is written after its input was
// published: with kPairAhead < kPairRing neither overtakes its reader, and a
// wave waits for the other's counter only to read.
template <int OBJ, typename Real> struct PairLds {
    typedef typename Vec4<Real>::T R4;
    static constexpr bool CONT = OBJ == OBJ_CONTOUR, TRACK = OBJ == OBJ_TRACK;
    R4 u[kPairRing][64];
    Real V[CONT ? kPairRing : 1][64];
    R4 dpw[kPairRing][64];              // the step's displacement and the new state's first body rate
    Real wy[kPairRing][64], wz[kPairRing][64];
    R4 q[TRACK ? kPairRing : 1][64];
    Real v[TRACK ? 3 : 1][TRACK ? kPairRing : 1][64];
    int cnt[2 + 64];                    // inputs drawn, steps moved; then words that nothing reads
};
struct NoPair {};

template <int OBJ, typename Real, bool DRAW> struct DrawLds {
    typename Vec4<Real>::T us[DRAW ? kNMax : 1];    // shifted warm-start inputs per step
    Real vs[DRAW && OBJ == OBJ_CONTOUR ? kNMax : 1];
};

// The shifted warm start of every step, staged once by the NT threads.
template <int NT, int OBJ, typename Real, bool DRAW, typename Head, typename Args>
__device__ __forceinline__ void stage_warm_start(const Args &a, int blk, const Head &h, DrawLds<OBJ, Real, DRAW> &lds)
{
    typedef typename Vec4<Real>::T R4;
    constexpr bool HAS_V = OBJ == OBJ_CONTOUR;
    auto &s_us = lds.us;
    auto &s_vs = lds.vs;
    const int K = a.K, N = a.N;
    const int shift = h.shift, warm = h.warm;
    const bool rows = a.regen && blk == (K >> 6);
    const double *const wU = in_global(a, a.wU), *const wV = in_global(a, a.wV);
    for (int k = (int)threadIdx.x; k < N; k += NT) {
        int src = k + shift;
        if (src > N - 1) src = N - 1;
        R4 o;
        o.x = warm ? (Real)wU[4 * src + 0] : (Real)a.hover;
        o.y = warm ? (Real)wU[4 * src + 1] : (Real)a.hover;
        o.z = warm ? (Real)wU[4 * src + 2] : (Real)a.hover;
        o.w = warm ? (Real)wU[4 * src + 3] : (Real)a.hover;
        s_us[k] = o;
        if (HAS_V) s_vs[k] = warm ? (Real)wV[src] : Real(0);
        // the weighted average draws the samples again from these rows
        if (rows) {
            in_global(a, (R4 *)a.nomU)[k] = o;
            if (HAS_V) in_global(a, (Real *)a.nomV)[k] = s_vs[k];
        }
    }
    __syncthreads();
}

// One wave: samples 64*blk .. 64*blk+63 (sample K is the noise-free nominal).
// DRAW: the wave draws its samples itself (the noise, perturbation and clip
// of the sample kernel, same operations) and stores them for the weighted
// average with streaming stores; the shifted warm start is staged in LDS from
// the head h.  Otherwise the wave reads the samples that the sample kernel
// stored.  PIPE: the costs are summed and the attitude step is closed as in
// the pipelined rollout, so that the results are those of k_rollout4 bit for
// bit (for launches with more tiles than the pipeline holds at once).
// NOM: the tile holds the nominal alone (K a multiple of 64) and draws nothing.
// PART: the whole rollout or one wave's part of a pair.
template <int OBJ, typename Real, bool DRAW, bool PIPE, bool RATE, bool DRAG, bool NOM, int PART = PART_ALL,
          typename Head, typename Args, typename Pair = NoPair>
__device__ __forceinline__ void rollout1_steps(const Args &a, int blk, const Head &h, DrawLds<OBJ, Real, DRAW> &lds,
                                               Pair &&pr = Pair())
{
    typedef typename Vec4<Real>::T R4;
    constexpr bool GATE = OBJ == OBJ_GATE, CONT = OBJ == OBJ_CONTOUR, TRACK = OBJ == OBJ_TRACK;
    constexpr bool HAS_V = CONT;
    static_assert(!(PIPE && RATE), "the rate input's order is the one-wave order");
    auto &s_us = lds.us;
    auto &s_vs = lds.vs;
    const int m = blk * 64 + (int)(threadIdx.x & 63);
    const int K = a.K, N = a.N;
    const bool active = m <= K;
    const bool nominal = m == K;
    Real Jfinal = Real(0);
    if (DRAW && PART == PART_ALL) stage_warm_start<64>(a, blk, h, lds);

    if (PART != PART_ALL || active) {
        Model<Real> M(a);
        in_vgpr(M);
        const Real dt = in_vgpr((Real)a.dt);
        const Real h2 = in_vgpr(Real(0.5) * (Real)a.dt);
        const Real dt6 = in_vgpr((Real)a.dt / Real(6));
        const Real h4 = in_vgpr(Real(0.5) * h2), dt12 = in_vgpr(Real(0.5) * dt6);
        const Real w_max = in_vgpr((Real)a.w_max), w_lim = in_vgpr((Real)a.w_lim);
        Real p[3], v[3], q[4], w[3];
        for (int i = 0; i < 3; ++i) { p[i] = (Real)h.x0[i]; v[i] = (Real)h.x0[3 + i]; w[i] = (Real)h.x0[10 + i]; }
        for (int i = 0; i < 4; ++i) q[i] = (Real)h.x0[6 + i];
        KSum<Real> J;                               // one-wave order: all terms of a step in one sum
        KSum<Real> J0, J1, J2;                      // pipelined order: body rates, attitude, position (J: the rest)

        // the inputs (u, V) of step k: drawn (and stored, unless the weighted
        // average draws them again) or read
        const R4 *urow = in_global(a, nominal ? (const R4 *)a.nomU : (const R4 *)a.ctrl + m);
        const size_t ustride = nominal ? 1 : (size_t)K;
        const Real *vrow = nullptr;
        if (HAS_V) vrow = in_global(a, nominal ? (const Real *)a.nomV : (const Real *)a.vctrl + m);
        const bool keep = DRAW && !a.regen && (PART == PART_ALL ? !nominal : m < K);
        const bool quiet = PART == PART_ALL ? nominal : m >= K;
        const uint32_t s_solve = h.s, key0 = a.seed_lo, key1 = a.seed_hi;
        const Real lo = (Real)(RATE ? a.rate_lim[0] : a.t_min), hi = (Real)(RATE ? a.rate_lim[1] : a.t_max);
        const Real vlo = (Real)(RATE ? a.dv_lim[0] : 0.0), vhi = (Real)(RATE ? a.dv_lim[1] : a.v_max);
        // the nominal draws with zero noise, so that no step selects
        const Real sig0 = in_vgpr(quiet ? Real(0) : (Real)a.sigma[0]), sig1 = in_vgpr(quiet ? Real(0) : (Real)a.sigma[1]);
        const Real sig2 = in_vgpr(quiet ? Real(0) : (Real)a.sigma[2]), sig3 = in_vgpr(quiet ? Real(0) : (Real)a.sigma[3]);
        const Real sigv = in_vgpr(quiet ? Real(0) : (Real)a.sigma_v);
        R4 *rec = in_global(a, (R4 *)a.ctrl + m);      // the sample's record, advanced step by step
        Real *vrec = HAS_V ? in_global(a, (Real *)a.vctrl + m) : nullptr;
        auto put = [&](const R4 &uo, const Real vo) {
            if (PART == PART_COSTS) {
                if (keep) {
                    *rec = uo;
                    if (HAS_V) *vrec = vo;
                }
            } else if (DRAW) {
                if (keep) {
                    store_nt(rec, uo);
                    if (HAS_V) store_nt(vrec, vo);
                }
            } else if (!nominal) {
                *rec = uo;
                if (HAS_V) *vrec = vo;
            }
            rec += K;
            if (HAS_V) vrec += K;
        };
        auto draw = [&](const int k, R4 &uo, Real &vo) {
            const R4 us = s_us[k];
            Normal4<Real> z = {};
            if (!NOM) z = normals4<Real>((uint32_t)m, (uint32_t)k, s_solve, 0u, key0, key1);
            uo.x = clamp_finite(us.x + sig0 * z.z0, lo, hi);
            uo.y = clamp_finite(us.y + sig1 * z.z1, lo, hi);
            uo.z = clamp_finite(us.z + sig2 * z.z2, lo, hi);
            uo.w = clamp_finite(us.w + sig3 * z.z3, lo, hi);
            if (HAS_V) {
                const Real zv = NOM ? Real(0) : normal1<Real>((uint32_t)m, (uint32_t)k, s_solve, 1u, key0, key1);
                vo = clamp_finite(s_vs[k] + sigv * zv, vlo, vhi);
            }
            if (!RATE) put(uo, vo);
        };

        // gate objective state
        const Real *gtab = in_global(a, (const Real *)a.gates_r);
        GateRegs<Real> gt, g0r;
        int g = 0, passes = 0;
        Real q_near = 0, r_near2 = 0, half = 0;
        if (GATE) {
            g = h.g0;
            gt.load(gtab, g);
            g0r = gt;
            q_near = in_vgpr((Real)a.q_near);
            r_near2 = in_vgpr((Real)(a.r_near * a.r_near));
            half = (Real)a.gate_half;
        }
        // tracking / contouring state
        Real up[4];
        for (int i = 0; i < 4; ++i) up[i] = (Real)h.u_prev[i];
        Real vp = (Real)h.v_prev;
        Real rdt[4];
        for (int i = 0; i < 4; ++i) rdt[i] = in_vgpr((Real)(a.R_dT[i] / (a.dt * a.dt)));
        const int i0 = h.i0, R = a.R;
        const Real *xref = in_global(a, (const Real *)a.xref_r);
        const Real *path = in_global(a, (const Real *)a.path_r);
        // arc length theta = th_hi + th_lo (th_lo stays 0 in binary64)
        Real th_hi = 0, th_lo = 0;
        Real ds = 0, inv_ds = 0, L = 0, q_l = 0, q_c = 0, qw[3] = {}, r_dv = 0, mu = 0;
        if (CONT) {
            th_hi = (Real)h.theta0;
            if (sizeof(Real) == 4) th_lo = (Real)(h.theta0 - (double)th_hi);
            L = in_vgpr((Real)a.path_len);
            ds = in_vgpr((Real)(a.path_len / (double)a.P));
            inv_ds = in_vgpr((Real)((double)a.P / a.path_len));
            q_l = in_vgpr((Real)a.q_l); q_c = in_vgpr((Real)a.q_c);
            for (int i = 0; i < 3; ++i) qw[i] = in_vgpr((Real)a.Q_w[i]);
            r_dv = in_vgpr(RATE ? (Real)a.r_dv : (Real)(a.r_dv / (a.dt * a.dt)));
            mu = in_vgpr((Real)a.mu);
        }

        // rate model: the thrust states and the progress speed state, carried
        // in binary64 in every precision (integrators: in binary32 their
        // rounding over the horizon reaches the attitude through the small
        // inertia and the position through the attitude)
        double T[4];
        for (int i = 0; i < 4; ++i) T[i] = RATE ? a.req[kReqThrust + i] : 0.0;
        double vs = RATE ? h.v_prev : 0.0;
        // the rate input's range clips (multiplied by 1/dt: the bound can
        // differ from the quotient in the last binary64 place)
        const double inv_dt = 1.0 / a.dt, t_min = a.t_min, t_max = a.t_max, v_max = a.v_max;
        R4 un;
        Real vn = Real(0);
        if (PART == PART_ALL && !DRAW) {
            un = urow[0];
            if (HAS_V) vn = vrow[0];
        }
        const int lane = (int)(threadIdx.x & 63);
        PipeWatch watch = {};
        int *mine = nullptr;
        int seen = 0;
        if constexpr (PART != PART_ALL) {
            watch.c = &pr.cnt[PART == PART_COSTS ? 1 : 0];
            mine = &pr.cnt[lane == 0 ? (PART == PART_COSTS ? 0 : 1) : 2 + lane];
        }
        for (int k = PART == PART_COSTS ? -kPairAhead : 0; k < N; ++k) {
            R4 u;
            Real V = Real(0);
            Real dp[3], wn[3], qn[4], vnew[3];
            if constexpr (PART == PART_COSTS) {
                // draw step k + kPairAhead while the motion of step k arrives
                const int sl = k & (kPairRing - 1);
                auto load = [&] {
                    const R4 d = pr.dpw[sl][lane];
                    dp[0] = d.x; dp[1] = d.y; dp[2] = d.z; wn[0] = d.w;
                    wn[1] = pr.wy[sl][lane];
                    wn[2] = pr.wz[sl][lane];
                    if (TRACK) {
                        const R4 t = pr.q[sl][lane];
                        qn[0] = t.x; qn[1] = t.y; qn[2] = t.z; qn[3] = t.w;
                        for (int i = 0; i < 3; ++i) vnew[i] = pr.v[i][sl][lane];
                    }
                };
                seen = watch.peek();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "singlethread");
                load();
                if (!GATE) u = pr.u[sl][lane];
                if (CONT) V = pr.V[sl][lane];
                if (k + kPairAhead < N) {
                    const int dl = (k + kPairAhead) & (kPairRing - 1);
                    R4 ud;
                    Real vd = Real(0);
                    draw(k + kPairAhead, ud, vd);
                    pr.u[dl][lane] = ud;
                    if (CONT) pr.V[dl][lane] = vd;
                    pipe_publish(mine, k + kPairAhead + 1);
                }
                if (k < 0) continue;
                if (!PipeWatch::may_start(seen, k)) {
                    watch.wait<0>(k);
                    load();
                }
            } else if constexpr (PART == PART_MOTION) {
                // the inputs of the next step are read while this one computes
                const int sl = k & (kPairRing - 1);
                if (k == 0 || !PipeWatch::may_start(seen, k)) {
                    watch.wait<0>(k);
                    un = pr.u[sl][lane];
                }
                u = un;
                seen = watch.peek();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "singlethread");
                un = pr.u[(k + 1) & (kPairRing - 1)][lane];
            } else if (DRAW) {
                draw(k, u, V);
            } else {
                // the inputs of the next step are in flight while this one computes
                u = un;
                V = vn;
                if (k + 1 < N) {
                    un = urow[(size_t)(k + 1) * ustride];
                    if (HAS_V) vn = vrow[(size_t)(k + 1) * ustride];
                }
            }
            if (RATE) {
                // clip the drawn rates to the range that keeps each thrust of
                // this sample's chain within [t_min, t_max] over the step (the
                // progress acceleration: the speed within [0, v_max]); the
                // clipped inputs are what the average weighs.  (Minimum and
                // maximum, not selects: those issue several times as slowly.)
                u.x = (Real)clamp_finite((double)u.x, (t_min - T[0]) * inv_dt, (t_max - T[0]) * inv_dt);
                u.y = (Real)clamp_finite((double)u.y, (t_min - T[1]) * inv_dt, (t_max - T[1]) * inv_dt);
                u.z = (Real)clamp_finite((double)u.z, (t_min - T[2]) * inv_dt, (t_max - T[2]) * inv_dt);
                u.w = (Real)clamp_finite((double)u.w, (t_min - T[3]) * inv_dt, (t_max - T[3]) * inv_dt);
                if (HAS_V) V = (Real)clamp_finite((double)V, (0.0 - vs) * inv_dt, (v_max - vs) * inv_dt);
            }
            if (RATE) put(u, V);
            Real term = Real(0);

            // ---- stage terms at state k
            Real ax = 0, ay = 0, az = 0;  // p_k - c_g (gate)
            if (PART == PART_MOTION) {
            } else if (GATE) {
                ax = p[0] - gt.cx;
                ay = p[1] - gt.cy;
                az = p[2] - gt.cz;
                const Real bx = p[0] - g0r.cx;
                const Real by = p[1] - g0r.cy;
                const Real bz = p[2] - g0r.cz;
                const Real d2 = bx * bx + by * by + bz * bz;
                if (d2 < r_near2) term += q_near * d2;  // Eq. (7), current gate
                if (nominal) in_global(a, a.front8)[k] = (bx * g0r.nx + by * g0r.ny) < Real(0);
            } else if (TRACK) {
                int r = i0 + k;
                if (r > R - 1) r = R - 1;
                const Real *xr = xref + 16 * r;
                if (PIPE) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = w[i] - xr[10 + i];
                        term += (Real)a.Q[10 + i] * e * e;
                    }
                    J0.add(term);
                    term = Real(0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const Real e = q[i] - xr[6 + i];
                        term += (Real)a.Q[6 + i] * e * e;
                    }
                    J1.add(term);
                    term = Real(0);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = p[i] - xr[i];
                        term += (Real)a.Q[i] * e * e;
                    }
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = v[i] - xr[3 + i];
                        term += (Real)a.Q[3 + i] * e * e;
                    }
                    J2.add(term);
                    term = Real(0);
                } else {
                    const Real x[13] = {p[0], p[1], p[2], v[0], v[1], v[2], q[0], q[1], q[2], q[3], w[0], w[1], w[2]};
#pragma unroll
                    for (int i = 0; i < 13; ++i) {
                        const Real e = x[i] - xr[i];
                        term += (Real)a.Q[i] * e * e;
                    }
                }
                if (RATE) {  // Eq. (8)'s u_k is the sampled thrust rate
                    term += (Real)a.R_dT[0] * u.x * u.x + (Real)a.R_dT[1] * u.y * u.y + (Real)a.R_dT[2] * u.z * u.z +
                            (Real)a.R_dT[3] * u.w * u.w;
                } else {
                    const Real d0 = u.x - up[0], d1 = u.y - up[1], d2 = u.z - up[2], d3 = u.w - up[3];
                    term += rdt[0] * d0 * d0 + rdt[1] * d1 * d1 + rdt[2] * d2 * d2 + rdt[3] * d3 * d3;
                }
            } else {  // contouring
                Real tq = Real(0);
                if (PIPE) {
                    tq += qw[0] * w[0] * w[0] + qw[1] * w[1] * w[1] + qw[2] * w[2] * w[2];
                    J0.add(tq);
                    const Real d0 = u.x - up[0], d1 = u.y - up[1], d2 = u.z - up[2], d3 = u.w - up[3];
                    term += rdt[0] * d0 * d0 + rdt[1] * d1 * d1 + rdt[2] * d2 * d2 + rdt[3] * d3 * d3;
                    const Real dv = V - vp;
                    term += r_dv * dv * dv;
                    term -= mu * V;
                }
                const Real fl = floor(th_hi * inv_ds);
                const Real f = ((th_hi - fl * ds) + th_lo) * inv_ds;
                // table row of theta, always inside [0, P)
                int i = (fl >= Real(0) && fl < Real(1 << 30)) ? ((int)fl % a.P) : 0;
                const int i1 = (i + 1 == a.P) ? 0 : i + 1;
                const Real *A = path + 8 * i, *B = path + 8 * i1;
                const Real g1 = Real(1) - f;
                const Real px = g1 * A[0] + f * B[0], py = g1 * A[1] + f * B[1], pz = g1 * A[2] + f * B[2];
                Real tx = g1 * A[3] + f * B[3], ty = g1 * A[4] + f * B[4], tz = g1 * A[5] + f * B[5];
                const Real tn = inv_sqrt(tx * tx + ty * ty + tz * tz);
                tx *= tn; ty *= tn; tz *= tn;
                const Real ex = p[0] - px;
                const Real ey = p[1] - py;
                const Real ez = p[2] - pz;
                const Real et = ex * tx + ey * ty + ez * tz;
                const Real lx = et * tx, ly = et * ty, lz = et * tz;
                const Real cxe = ex - lx, cye = ey - ly, cze = ez - lz;
                term += q_l * (lx * lx + ly * ly + lz * lz);
                term += q_c * (cxe * cxe + cye * cye + cze * cze);
                if (!PIPE) term += qw[0] * w[0] * w[0] + qw[1] * w[1] * w[1] + qw[2] * w[2] * w[2];
                Real adv;  // arc length advanced over the step
                if (RATE) {
                    // Eq. (9) with the progress acceleration as the input and
                    // the speed as a state, which moves linearly over the step
                    term += r_dv * V * V;
                    term += (Real)a.R_dT[0] * u.x * u.x + (Real)a.R_dT[1] * u.y * u.y + (Real)a.R_dT[2] * u.z * u.z +
                            (Real)a.R_dT[3] * u.w * u.w;
                    term -= mu * (Real)vs;
                    const double vsn = vs + a.dt * (double)V;
                    adv = (Real)(0.5 * a.dt * (vs + vsn));
                    vs = vsn;
                } else {
                    if (!PIPE) {
                        const Real dv = V - vp;
                        term += r_dv * dv * dv;
                        const Real d0 = u.x - up[0], d1 = u.y - up[1], d2 = u.z - up[2], d3 = u.w - up[3];
                        term += rdt[0] * d0 * d0 + rdt[1] * d1 * d1 + rdt[2] * d2 * d2 + rdt[3] * d3 * d3;
                        term -= mu * V;
                    }
                    adv = V * dt;
                }
                vp = V;
                {   // theta_{k+1} = theta_k + advance (mod L), compensated in binary32
                    Real y;
                    if (PIPE) y = V * dt + th_lo;
                    else y = adv + th_lo;
                    const Real t = th_hi + y;
                    th_lo = (sizeof(Real) == 4) ? y - (t - th_hi) : Real(0);
                    th_hi = t;
                    if (th_hi >= L) th_hi -= L;
                }
            }

            // ---- dynamics: RK4 of Eq. (2).  The rate model's thrusts move
            // linearly over the step: its stages see them at the start, middle
            // and end of it.
            if (PART != PART_COSTS) {
                StepInput<Real> in[3];
                if (RATE) {
                    const double h = 0.5 * a.dt, ur[4] = {(double)u.x, (double)u.y, (double)u.z, (double)u.w};
                    in[0] = step_input(M, (Real)T[0], (Real)T[1], (Real)T[2], (Real)T[3]);
                    in[1] = step_input(M, (Real)(T[0] + h * ur[0]), (Real)(T[1] + h * ur[1]), (Real)(T[2] + h * ur[2]),
                                       (Real)(T[3] + h * ur[3]));
                    in[2] = step_input(M, (Real)(T[0] + a.dt * ur[0]), (Real)(T[1] + a.dt * ur[1]),
                                       (Real)(T[2] + a.dt * ur[2]), (Real)(T[3] + a.dt * ur[3]));
                    for (int i = 0; i < 4; ++i) T[i] += a.dt * ur[i];
                } else {
                    in[0] = step_input(M, u.x, u.y, u.z, u.w);
                }
                Real dv[3], dq[4], dw[3];
                {
                    Real vst[3], qs[4], ws[3];
#pragma unroll
                    for (int i = 0; i < 3; ++i) { vst[i] = v[i]; ws[i] = w[i]; }
#pragma unroll
                    for (int i = 0; i < 4; ++i) qs[i] = q[i];
#pragma unroll
                    for (int st = 0; st < 4; ++st) {
                        const StepInput<Real> &si = in[RATE ? (st == 0 ? 0 : (st < 3 ? 1 : 2)) : 0];
                        Real kv[3], kw[3], kq[4];
                        stage_accel<DRAG>(M, si.fm, qs, vst, kv);
                        kw[0] = si.tx - M.gx * ws[1] * ws[2];
                        kw[1] = si.ty - M.gy * ws[2] * ws[0];
                        kw[2] = si.tz - M.gz * ws[0] * ws[1];
                        // kq is twice the quaternion rate; the factor 1/2 is
                        // carried by the step sizes (exact: a power of two)
                        kq[0] = -qs[1] * ws[0] - qs[2] * ws[1] - qs[3] * ws[2];
                        kq[1] = qs[0] * ws[0] + qs[2] * ws[2] - qs[3] * ws[1];
                        kq[2] = qs[0] * ws[1] - qs[1] * ws[2] + qs[3] * ws[0];
                        kq[3] = qs[0] * ws[2] + qs[1] * ws[1] - qs[2] * ws[0];
                        if (st == 0) {
#pragma unroll
                            for (int i = 0; i < 3; ++i) { dp[i] = vst[i]; dv[i] = kv[i]; dw[i] = kw[i]; }
#pragma unroll
                            for (int i = 0; i < 4; ++i) dq[i] = kq[i];
                        } else if (st < 3) {
#pragma unroll
                            for (int i = 0; i < 3; ++i) {
                                dp[i] += Real(2) * vst[i];
                                dv[i] += Real(2) * kv[i];
                                dw[i] += Real(2) * kw[i];
                            }
#pragma unroll
                            for (int i = 0; i < 4; ++i) dq[i] += Real(2) * kq[i];
                        } else {
#pragma unroll
                            for (int i = 0; i < 3; ++i) {
                                dp[i] = dt6 * (dp[i] + vst[i]);
                                dv[i] = dt6 * (dv[i] + kv[i]);
                                dw[i] = dt6 * (dw[i] + kw[i]);
                            }
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                if (PIPE) {
                                    q[i] = q[i] + dt12 * (dq[i] + kq[i]);
                                } else {
                                    dq[i] = dt12 * (dq[i] + kq[i]);
                                    q[i] += dq[i];
                                }
                            }
                        }
                        if (st < 3) {
                            const Real hh = st < 2 ? h2 : dt, hq = st < 2 ? h4 : h2;
#pragma unroll
                            for (int i = 0; i < 3; ++i) {
                                vst[i] = v[i] + hh * kv[i];
                                ws[i] = w[i] + hh * kw[i];
                            }
#pragma unroll
                            for (int i = 0; i < 4; ++i) qs[i] = q[i] + hq * kq[i];
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) { p[i] += dp[i]; v[i] += dv[i]; w[i] += dw[i]; }
                renormalize(q);
                if constexpr (PART == PART_MOTION) {
                    const int sl = k & (kPairRing - 1);
                    R4 d;
                    d.x = dp[0]; d.y = dp[1]; d.z = dp[2]; d.w = w[0];
                    pr.dpw[sl][lane] = d;
                    pr.wy[sl][lane] = w[1];
                    pr.wz[sl][lane] = w[2];
                    if (TRACK) {
                        R4 t;
                        t.x = q[0]; t.y = q[1]; t.z = q[2]; t.w = q[3];
                        pr.q[sl][lane] = t;
                        for (int i = 0; i < 3; ++i) pr.v[i][sl][lane] = v[i];
                    }
                    pipe_publish(mine, k + 1);
                    continue;
                }
            } else {
                for (int i = 0; i < 3; ++i) { p[i] += dp[i]; w[i] = wn[i]; if (TRACK) v[i] = vnew[i]; }
                if (TRACK) for (int i = 0; i < 4; ++i) q[i] = qn[i];
            }

            // ---- progress and switching (gate)
            if (GATE) {
                // |p_{k+1} - c|^2 - |p_k - c|^2 = dp . (2 (p_k - c) + dp)
                term += dp[0] * (Real(2) * ax + dp[0]) + dp[1] * (Real(2) * ay + dp[1]) +
                        dp[2] * (Real(2) * az + dp[2]);
                const Real sa = ax * gt.nx + ay * gt.ny;
                const Real sb = (ax + dp[0]) * gt.nx + (ay + dp[1]) * gt.ny;
                if (sa < Real(0) && sb >= Real(0)) {
                    const Real t = sa / (sa - sb);
                    const Real yx = ax + t * dp[0], yy = ay + t * dp[1], yz = az + t * dp[2];
                    const Real lat = yx * gt.hx + yy * gt.hy;
                    const bool inside = fabs(lat) <= half && fabs(yz) <= half;
                    const int j = k + 1;
                    const bool allowed = passes > 0 || ((h.allow[j >> 5] >> (j & 31)) & 1u);
                    if (inside && allowed) {
                        g = (g + 1 == a.G) ? 0 : g + 1;
                        ++passes;
                        gt.load(gtab, g);
                    }
                }
            }
            // ---- body-rate penalty on the new state
            if (PIPE) {
                Real rl = Real(0);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = fmax(fabs(w[i]) - w_max, Real(0));
                    rl += w_lim * e * e;
                }
                J0.add(rl);
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = fmax(fabs(w[i]) - w_max, Real(0));
                    term += w_lim * e * e;
                }
            }
            J.add(term);
            if (!GATE && !RATE) { up[0] = u.x; up[1] = u.y; up[2] = u.z; up[3] = u.w; }
        }
        if (PART == PART_MOTION) return;
        if (TRACK) {
            int r = i0 + N;
            if (r > R - 1) r = R - 1;
            const Real *xr = xref + 16 * r;
            Real term = 0;
            if (PIPE) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = w[i] - xr[10 + i];
                    term += (Real)a.QN[10 + i] * e * e;
                }
                J0.add(term);
                term = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const Real e = q[i] - xr[6 + i];
                    term += (Real)a.QN[6 + i] * e * e;
                }
                J1.add(term);
                term = 0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = p[i] - xr[i];
                    term += (Real)a.QN[i] * e * e;
                    const Real f = v[i] - xr[3 + i];
                    term += (Real)a.QN[3 + i] * f * f;
                }
                J2.add(term);
            } else {
                const Real x[13] = {p[0], p[1], p[2], v[0], v[1], v[2], q[0], q[1], q[2], q[3], w[0], w[1], w[2]};
#pragma unroll
                for (int i = 0; i < 13; ++i) {
                    const Real e = x[i] - xr[i];
                    term += (Real)a.QN[i] * e * e;
                }
                J.add(term);
            }
        }
        if (GATE && nominal) {
            const Real bx = p[0] - g0r.cx;
            const Real by = p[1] - g0r.cy;
            in_global(a, a.front8)[N] = (bx * g0r.nx + by * g0r.ny) < Real(0);
        }
        Jfinal = PIPE ? ((J0.value() + J1.value()) + J2.value()) + J.value() : J.value();
        if (nominal) in_global(a, a.cur)->J_nom = (double)Jfinal;
        else if (PART == PART_ALL || m < K) in_global(a, (Real *)a.J)[m] = Jfinal;
    }
    // smallest finite sample cost of the tile
    store_tile_min(Jfinal, active && !nominal && isfinite(Jfinal), in_global(a, (Real *)a.tmin), blk);
}

// Drag is a launch constant: the variant is chosen once.  A last tile that
// holds the nominal alone skips the draws: where K fills the chip's waves to
// the last lane it runs after them, alone (K = 262144, N = 200: 523 -> 454 us
// a solve).
template <int OBJ, typename Real, bool DRAW, bool PIPE, bool RATE, typename Head, typename Args>
__device__ __forceinline__ void rollout1_body(const Args &a, int blk, const Head &h, DrawLds<OBJ, Real, DRAW> &lds)
{
    const bool nom = DRAW && !RATE && blk * 64 == a.K;
    constexpr bool NOM = DRAW && !RATE;
    if (a.has_drag) {
        if (nom) rollout1_steps<OBJ, Real, DRAW, PIPE, RATE, true, NOM>(a, blk, h, lds);
        else rollout1_steps<OBJ, Real, DRAW, PIPE, RATE, true, false>(a, blk, h, lds);
    } else {
        if (nom) rollout1_steps<OBJ, Real, DRAW, PIPE, RATE, false, NOM>(a, blk, h, lds);
        else rollout1_steps<OBJ, Real, DRAW, PIPE, RATE, false, false>(a, blk, h, lds);
    }
}

// A pair of waves per tile (binary32, thrust input).
template <int OBJ, typename Real> __global__ __launch_bounds__(128) void k_rollout_pair(KArgs a)
{
    __shared__ HeadVals h;
    __shared__ DrawLds<OBJ, Real, true> lds;
    __shared__ PairLds<OBJ, Real> pr;
    compute_head<OBJ == OBJ_CONTOUR>(a, h);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish_head(a, h);
    if (threadIdx.x < 2) pr.cnt[threadIdx.x] = 0;
    stage_warm_start<128>(a, blockIdx.x, h, lds);
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) == 0) {
        rollout1_steps<OBJ, Real, true, false, false, false, false, PART_COSTS>(a, blockIdx.x, h, lds, pr);
    } else if (a.has_drag) {
        rollout1_steps<OBJ, Real, true, false, false, true, false, PART_MOTION>(a, blockIdx.x, h, lds, pr);
    } else {
        rollout1_steps<OBJ, Real, true, false, false, false, false, PART_MOTION>(a, blockIdx.x, h, lds, pr);
    }
}

template <int OBJ, typename Real, bool DRAW> __global__ __launch_bounds__(64) void k_rollout(KArgs a)
{
    __shared__ DrawLds<OBJ, Real, DRAW> lds;
    const DevCur &h = *(const DevCur *)a.cur;
    // (on its own a rate context reads the sample kernel's rates)
    if constexpr (DRAW) {
        rollout1_body<OBJ, Real, true, false, false>(a, blockIdx.x, h, lds);
    } else {
        if (a.input_model == INPUT_RATE) rollout1_body<OBJ, Real, false, false, true>(a, blockIdx.x, h, lds);
        else rollout1_body<OBJ, Real, false, false, false>(a, blockIdx.x, h, lds);
    }
}

// ---------------------------------------------------------------- rollout, two waves

// The rotational subsystem (q, omega) of Eq. (2) does not depend on position
// or velocity, so one sample's rollout splits over two waves of a workgroup:
// wave 0 integrates (q, omega) and hands the four RK4 stage quaternions of
// every step to wave 1 through an LDS ring of B steps; wave 1 integrates
// (p, v) from them and evaluates the position-dependent cost terms.  Each
// wave accumulates the cost terms of its own state components; the two
// partial costs are added at the end.  The arithmetic of every component is
// the same as in the one-wave rollout; only the two halves run concurrently
// on two SIMDs, which halves the critical path of a step.
template <typename Real> struct SplitRing;
template <> struct SplitRing<float> { static constexpr int B = 8; };
template <> struct SplitRing<double> { static constexpr int B = 4; };

template <int OBJ, typename Real> __device__ __forceinline__ void rollout2_body(const KArgs &a, int blk)
{
    typedef typename Vec4<Real>::T R4;
    constexpr int B = SplitRing<Real>::B;
    __shared__ R4 s_q[2][B][4][64];
    __shared__ Real s_jr[64];

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int m = blk * 64 + lane;
    const int K = a.K, N = a.N;
    const bool active = m <= K;
    const bool nominal = m == K;
    const DevCur *cur = a.cur;
    const Model<Real> M(a);
    const Real dt = (Real)a.dt;
    const Real h2 = Real(0.5) * dt;
    const Real dt6 = dt / Real(6);
    const Real h4 = Real(0.5) * h2, dt12 = Real(0.5) * dt6;
    const Real w_max = (Real)a.w_max, w_lim = (Real)a.w_lim;
    const bool use_nom = m >= K;  // lanes past K read the nominal row, results unused
    const R4 *urow = use_nom ? (const R4 *)a.nomU : (const R4 *)a.ctrl + m;
    const size_t ustride = use_nom ? 1 : (size_t)K;
    const Real *xref = (const Real *)a.xref_r;
    const int i0 = cur->i0;
    Real rdt[4];
    for (int i = 0; i < 4; ++i) rdt[i] = (Real)(a.R_dT[i] / (a.dt * a.dt));

    KSum<Real> J;
    // ---- wave 0: attitude and body rates
    Real q[4], w[3], up[4];
    // ---- wave 1: position and velocity
    Real p[3], v[3];
    GateRegs<Real> gt, g0r;
    int g = 0, passes = 0;
    Real vp = 0, th_hi = 0, th_lo = 0, ds = 0, inv_ds = 0, L = 0;
    const Real *vrow = nullptr;
    const Real *gtab = (const Real *)a.gates_r;
    const Real *path = (const Real *)a.path_r;
    {
        const double *x0 = cur->x0;
        for (int i = 0; i < 4; ++i) {
            q[i] = (Real)x0[6 + i];
        }
        for (int i = 0; i < 3; ++i) {
            w[i] = (Real)x0[10 + i];
            p[i] = (Real)x0[i];
            v[i] = (Real)x0[3 + i];
        }
        for (int i = 0; i < 4; ++i) up[i] = (Real)cur->u_prev[i];
    }
    if (wave == 1) {
        if (OBJ == OBJ_GATE) {
            g = cur->g0;
            gt.load(gtab, g);
            g0r = gt;
        }
        if (OBJ == OBJ_CONTOUR) {
            vrow = use_nom ? (const Real *)a.nomV : (const Real *)a.vctrl + m;
            vp = (Real)cur->v_prev;
            th_hi = (Real)cur->theta0;
            if (sizeof(Real) == 4) th_lo = (Real)(cur->theta0 - (double)th_hi);
            L = (Real)a.path_len;
            ds = (Real)(a.path_len / (double)a.P);
            inv_ds = (Real)((double)a.P / a.path_len);
        }
    }
    const Real q_near = (Real)a.q_near, r_near2 = (Real)(a.r_near * a.r_near), half = (Real)a.gate_half;

    const int nch = (N + B - 1) / B;
    // the control of the next step is always in flight while a step computes
    R4 u_next = urow[0];
    Real v_next = Real(0);
    if (OBJ == OBJ_CONTOUR && wave == 1) v_next = vrow[0];
    for (int c = 0; c <= nch; ++c) {
        if (wave == 0 && c < nch) {
            const int kb = c * B, ke = min(N, kb + B);
            for (int k = kb; k < ke; ++k) {
                R4 (*slot)[64] = s_q[c & 1][k - kb];
                const R4 u = u_next;
                if (k + 1 < N) u_next = urow[(size_t)(k + 1) * ustride];
                Real term = Real(0);
                if (OBJ == OBJ_TRACK) {
                    int r = i0 + k;
                    if (r > a.R - 1) r = a.R - 1;
                    const Real *xr = xref + 16 * r;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const Real e = q[i] - xr[6 + i];
                        term += (Real)a.Q[6 + i] * e * e;
                    }
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = w[i] - xr[10 + i];
                        term += (Real)a.Q[10 + i] * e * e;
                    }
                }
                if (OBJ == OBJ_CONTOUR)
                    term += (Real)a.Q_w[0] * w[0] * w[0] + (Real)a.Q_w[1] * w[1] * w[1] +
                            (Real)a.Q_w[2] * w[2] * w[2];
                if (OBJ != OBJ_GATE) {
                    const Real d0 = u.x - up[0], d1 = u.y - up[1], d2 = u.z - up[2], d3 = u.w - up[3];
                    term += rdt[0] * d0 * d0 + rdt[1] * d1 * d1 + rdt[2] * d2 * d2 + rdt[3] * d3 * d3;
                }
                const StepInput<Real> in = step_input(M, u.x, u.y, u.z, u.w);
                // RK4 on (q, omega)
                Real ws[3], qs[4], kw[3], kq[4], dw[3], dq[4];
#pragma unroll
                for (int i = 0; i < 3; ++i) ws[i] = w[i];
#pragma unroll
                for (int i = 0; i < 4; ++i) qs[i] = q[i];
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    R4 o;
                    o.x = qs[0]; o.y = qs[1]; o.z = qs[2]; o.w = qs[3];
                    slot[st][lane] = o;
                    kw[0] = in.tx - M.gx * ws[1] * ws[2];
                    kw[1] = in.ty - M.gy * ws[2] * ws[0];
                    kw[2] = in.tz - M.gz * ws[0] * ws[1];
                    // kq is twice the quaternion rate; the factor 1/2 is
                    // carried by the step sizes (exact: a power of two)
                    kq[0] = -qs[1] * ws[0] - qs[2] * ws[1] - qs[3] * ws[2];
                    kq[1] = qs[0] * ws[0] + qs[2] * ws[2] - qs[3] * ws[1];
                    kq[2] = qs[0] * ws[1] - qs[1] * ws[2] + qs[3] * ws[0];
                    kq[3] = qs[0] * ws[2] + qs[1] * ws[1] - qs[2] * ws[0];
                    if (st == 0) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] = kw[i];
#pragma unroll
                        for (int i = 0; i < 4; ++i) dq[i] = kq[i];
                    } else if (st < 3) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] += Real(2) * kw[i];
#pragma unroll
                        for (int i = 0; i < 4; ++i) dq[i] += Real(2) * kq[i];
                    } else {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] = dt6 * (dw[i] + kw[i]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) dq[i] = dt12 * (dq[i] + kq[i]);
                    }
                    if (st < 3) {
                        const Real hh = st < 2 ? h2 : dt;
                        const Real hq = st < 2 ? h4 : h2;
#pragma unroll
                        for (int i = 0; i < 3; ++i) ws[i] = w[i] + hh * kw[i];
#pragma unroll
                        for (int i = 0; i < 4; ++i) qs[i] = q[i] + hq * kq[i];
                    }
                }
                // commit the step, unit quaternion
#pragma unroll
                for (int i = 0; i < 3; ++i) w[i] += dw[i];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] += dq[i];
                renormalize(q);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = fmax(fabs(w[i]) - w_max, Real(0));
                    term += w_lim * e * e;
                }
                J.add(term);
                up[0] = u.x; up[1] = u.y; up[2] = u.z; up[3] = u.w;
            }
        } else if (wave == 1 && c >= 1) {
            const int kb = (c - 1) * B, ke = min(N, kb + B);
            for (int k = kb; k < ke; ++k) {
                R4 (*slot)[64] = s_q[(c - 1) & 1][k - kb];
                const R4 u = u_next;
                if (k + 1 < N) u_next = urow[(size_t)(k + 1) * ustride];
                R4 qstage[4];
#pragma unroll
                for (int st = 0; st < 4; ++st) qstage[st] = slot[st][lane];
                const Real fm = ((u.x + u.y) + (u.z + u.w)) * M.inv_m;
                Real term = Real(0);
                Real ax = 0, ay = 0, az = 0;
                if (OBJ == OBJ_GATE) {
                    ax = p[0] - gt.cx;
                    ay = p[1] - gt.cy;
                    az = p[2] - gt.cz;
                    const Real bx = p[0] - g0r.cx;
                    const Real by = p[1] - g0r.cy;
                    const Real bz = p[2] - g0r.cz;
                    const Real d2 = bx * bx + by * by + bz * bz;
                    if (d2 < r_near2) term += q_near * d2;
                    if (nominal) a.front8[k] = (bx * g0r.nx + by * g0r.ny) < Real(0);
                } else if (OBJ == OBJ_TRACK) {
                    int r = i0 + k;
                    if (r > a.R - 1) r = a.R - 1;
                    const Real *xr = xref + 16 * r;
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = p[i] - xr[i];
                        term += (Real)a.Q[i] * e * e;
                    }
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = v[i] - xr[3 + i];
                        term += (Real)a.Q[3 + i] * e * e;
                    }
                } else {
                    const Real fl = floor(th_hi * inv_ds);
                    const Real f = ((th_hi - fl * ds) + th_lo) * inv_ds;
                    const int i = (fl >= Real(0) && fl < Real(1 << 30)) ? ((int)fl % a.P) : 0;
                    const int i1 = (i + 1 == a.P) ? 0 : i + 1;
                    const Real *A = path + 8 * i, *Bp = path + 8 * i1;
                    const Real g1 = Real(1) - f;
                    const Real px = g1 * A[0] + f * Bp[0], py = g1 * A[1] + f * Bp[1], pz = g1 * A[2] + f * Bp[2];
                    Real tx = g1 * A[3] + f * Bp[3], ty = g1 * A[4] + f * Bp[4], tz = g1 * A[5] + f * Bp[5];
                    const Real tn = inv_sqrt(tx * tx + ty * ty + tz * tz);
                    tx *= tn; ty *= tn; tz *= tn;
                    const Real ex = p[0] - px;
                    const Real ey = p[1] - py;
                    const Real ez = p[2] - pz;
                    const Real et = ex * tx + ey * ty + ez * tz;
                    const Real lx = et * tx, ly = et * ty, lz = et * tz;
                    const Real cxe = ex - lx, cye = ey - ly, cze = ez - lz;
                    term += (Real)a.q_l * (lx * lx + ly * ly + lz * lz);
                    term += (Real)a.q_c * (cxe * cxe + cye * cye + cze * cze);
                    const Real vk = v_next;
                    if (k + 1 < N) v_next = vrow[(size_t)(k + 1) * ustride];
                    const Real dv = vk - vp;
                    term += (Real)(a.r_dv / (a.dt * a.dt)) * dv * dv;
                    term -= (Real)a.mu * vk;
                    vp = vk;
                    const Real y = vk * dt + th_lo;
                    const Real t = th_hi + y;
                    th_lo = (sizeof(Real) == 4) ? y - (t - th_hi) : Real(0);
                    th_hi = t;
                    if (th_hi >= L) th_hi -= L;
                }
                // RK4 on (p, v) with the stage quaternions of wave 0
                Real vs[3], kv[3], dpv[3], dvv[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) vs[i] = v[i];
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const R4 qq = qstage[st];
                    const Real r3x = Real(2) * (qq.y * qq.w + qq.x * qq.z);
                    const Real r3y = Real(2) * (qq.z * qq.w - qq.x * qq.y);
                    const Real r3z = Real(1) - Real(2) * (qq.y * qq.y + qq.z * qq.z);
                    kv[0] = fm * r3x;
                    kv[1] = fm * r3y;
                    kv[2] = fm * r3z - M.g;
                    if (M.drag) {
                        const Real qw = qq.x, qx = qq.y, qy = qq.z, qz = qq.w;
                        const Real r11 = Real(1) - Real(2) * (qy * qy + qz * qz), r12 = Real(2) * (qx * qy - qw * qz);
                        const Real r21 = Real(2) * (qx * qy + qw * qz), r22 = Real(1) - Real(2) * (qx * qx + qz * qz);
                        const Real r31 = Real(2) * (qx * qz - qw * qy), r32 = Real(2) * (qy * qz + qw * qx);
                        const Real b0 = M.d0 * (r11 * vs[0] + r21 * vs[1] + r31 * vs[2]);
                        const Real b1 = M.d1 * (r12 * vs[0] + r22 * vs[1] + r32 * vs[2]);
                        const Real b2 = M.d2 * (r3x * vs[0] + r3y * vs[1] + r3z * vs[2]);
                        kv[0] -= r11 * b0 + r12 * b1 + r3x * b2;
                        kv[1] -= r21 * b0 + r22 * b1 + r3y * b2;
                        kv[2] -= r31 * b0 + r32 * b1 + r3z * b2;
                    }
                    if (st == 0) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) { dpv[i] = vs[i]; dvv[i] = kv[i]; }
                    } else if (st < 3) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) { dpv[i] += Real(2) * vs[i]; dvv[i] += Real(2) * kv[i]; }
                    } else {
#pragma unroll
                        for (int i = 0; i < 3; ++i) { dpv[i] = dt6 * (dpv[i] + vs[i]); dvv[i] = dt6 * (dvv[i] + kv[i]); }
                    }
                    if (st < 3) {
                        const Real hh = st < 2 ? h2 : dt;
#pragma unroll
                        for (int i = 0; i < 3; ++i) vs[i] = v[i] + hh * kv[i];
                    }
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    p[i] += dpv[i];
                    v[i] += dvv[i];
                }
                if (OBJ == OBJ_GATE) {
                    term += dpv[0] * (Real(2) * ax + dpv[0]) + dpv[1] * (Real(2) * ay + dpv[1]) +
                            dpv[2] * (Real(2) * az + dpv[2]);
                    const Real sa = ax * gt.nx + ay * gt.ny;
                    const Real sb = (ax + dpv[0]) * gt.nx + (ay + dpv[1]) * gt.ny;
                    if (sa < Real(0) && sb >= Real(0)) {
                        const Real t = sa / (sa - sb);
                        const Real yx = ax + t * dpv[0], yy = ay + t * dpv[1], yz = az + t * dpv[2];
                        const Real lat = yx * gt.hx + yy * gt.hy;
                        const bool inside = fabs(lat) <= half && fabs(yz) <= half;
                        const int j = k + 1;
                        const bool allowed = passes > 0 || ((cur->allow[j >> 5] >> (j & 31)) & 1u);
                        if (inside && allowed) {
                            g = (g + 1 == a.G) ? 0 : g + 1;
                            ++passes;
                            gt.load(gtab, g);
                        }
                    }
                }
                J.add(term);
            }
        }
        __syncthreads();
    }

    // terminal terms, then the two partial costs are added
    if (OBJ == OBJ_TRACK) {
        int r = i0 + N;
        if (r > a.R - 1) r = a.R - 1;
        const Real *xr = xref + 16 * r;
        Real term = 0;
        if (wave == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const Real e = q[i] - xr[6 + i];
                term += (Real)a.QN[6 + i] * e * e;
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const Real e = w[i] - xr[10 + i];
                term += (Real)a.QN[10 + i] * e * e;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const Real e = p[i] - xr[i];
                term += (Real)a.QN[i] * e * e;
                const Real f = v[i] - xr[3 + i];
                term += (Real)a.QN[3 + i] * f * f;
            }
        }
        J.add(term);
    }
    if (wave == 0) s_jr[lane] = J.value();
    __syncthreads();
    if (wave == 1) {
        Real Jfinal = Real(0);
        if (active) {
            Jfinal = J.value() + s_jr[lane];
            if (OBJ == OBJ_GATE && nominal) {
                const Real bx = p[0] - g0r.cx;
                const Real by = p[1] - g0r.cy;
                a.front8[N] = (bx * g0r.nx + by * g0r.ny) < Real(0);
            }
            if (nominal) a.cur->J_nom = (double)Jfinal;
            else ((Real *)a.J)[m] = Jfinal;
        }
        store_tile_min(Jfinal, active && !nominal && isfinite(Jfinal), a.tmin, blk);
    }
}

template <int OBJ, typename Real> __global__ __launch_bounds__(128) void k_rollout_split(KArgs a)
{
    rollout2_body<OBJ, Real>(a, blockIdx.x);
}

// ---------------------------------------------------------------- rollout, three waves

// Sampling joins the rollout: per 64-sample tile, wave 0 draws the noise and
// the clipped controls of every step (Eq. (3)), stores them in the sample
// tensor for the weighted average and hands the step's collective thrust over
// mass and torques over inertia to the other waves through an LDS ring;
// wave 1 integrates (q, omega) and hands on the RK4 stage quaternions; wave 2
// integrates (p, v) and evaluates the position costs.  Each wave accumulates
// the cost terms of what it computes (wave 0: control-rate and progress-speed
// terms; wave 1: attitude and body-rate terms; wave 2: position terms); the
// three partial costs are added at the end.  Every workgroup derives the
// per-solve head itself; workgroup 0 publishes it for the tail.
template <typename Real> struct Ring3;
template <> struct Ring3<float> { static constexpr int B = 8; };
template <> struct Ring3<double> { static constexpr int B = 4; };

template <int OBJ, typename Real>
__device__ __forceinline__ void rollout3_body(const KArgs &a, int blk, const HeadVals &h)
{
    typedef typename Vec4<Real>::T R4;
    constexpr int B = Ring3<Real>::B;
    constexpr bool HAS_V = OBJ == OBJ_CONTOUR;
    __shared__ R4 s_in[3][B][64];                  // (F/m, tau_x/J_x, tau_y/J_y, tau_z/J_z)
    __shared__ Real s_v[HAS_V ? 3 : 1][B][64];     // progress speed
    __shared__ R4 s_q[2][B][4][64];                // stage quaternions
    __shared__ Real s_jp[2][64];                   // partial costs of waves 0 and 1
    __shared__ R4 s_us[kNMax];                     // shifted warm-start thrusts per step
    __shared__ Real s_vs[HAS_V ? kNMax : 1];       // shifted warm-start progress speed
    __shared__ Real s_gtab[OBJ == OBJ_GATE ? 8 * kGMax : 1];   // the gate table, staged once
    __shared__ uint8_t s_f8[OBJ == OBJ_GATE ? kNMax : 1];      // front flags of the nominal, steps 0..N-1

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int m = blk * 64 + lane;
    const int K = a.K, N = a.N;
    const bool active = m <= K;
    const bool nominal = m == K;
    const bool sampled = m < K;
    const Model<Real> M(a);
    const Real dt = (Real)a.dt;
    const Real h2 = Real(0.5) * dt;
    const Real dt6 = dt / Real(6);
    const Real h4 = Real(0.5) * h2, dt12 = Real(0.5) * dt6;
    const Real w_max = (Real)a.w_max, w_lim = (Real)a.w_lim;
    const Real *xref = (const Real *)a.xref_r;
    const int i0 = h.i0;
    Real rdt[4];
    for (int i = 0; i < 4; ++i) rdt[i] = (Real)(a.R_dT[i] / (a.dt * a.dt));
    const Real r_dv = (Real)(a.r_dv / (a.dt * a.dt));

    KSum<Real> J;
    // wave 0: sampling
    Real up[4], vp = (Real)h.v_prev;
    for (int i = 0; i < 4; ++i) up[i] = (Real)h.u_prev[i];
    // wave 1: attitude and body rates; wave 2: position and velocity
    Real q[4], w[3], p[3], v[3];
    for (int i = 0; i < 4; ++i) {
        q[i] = (Real)h.x0[6 + i];
    }
    for (int i = 0; i < 3; ++i) {
        w[i] = (Real)h.x0[10 + i];
        p[i] = (Real)h.x0[i];
        v[i] = (Real)h.x0[3 + i];
    }
    GateRegs<Real> gt, g0r;
    int g = 0, passes = 0;
    const Real *gtab = (const Real *)a.gates_r;
    const Real *path = (const Real *)a.path_r;
    Real th_hi = 0, th_lo = 0, ds = 0, inv_ds = 0, L = 0;
    if (OBJ == OBJ_GATE) g = h.g0;
    if (OBJ == OBJ_CONTOUR) {
        th_hi = (Real)h.theta0;
        if (sizeof(Real) == 4) th_lo = (Real)(h.theta0 - (double)th_hi);
        L = (Real)a.path_len;
        ds = (Real)(a.path_len / (double)a.P);
        inv_ds = (Real)((double)a.P / a.path_len);
    }
    const Real q_near = (Real)a.q_near, r_near2 = (Real)(a.r_near * a.r_near), half = (Real)a.gate_half;
    const Real tmin = (Real)a.t_min, tmax = (Real)a.t_max, vmax = (Real)a.v_max;
    const Real sig0 = (Real)a.sigma[0], sig1 = (Real)a.sigma[1], sig2 = (Real)a.sigma[2], sig3 = (Real)a.sigma[3];
    const Real sigv = (Real)a.sigma_v, hover = (Real)a.hover;
    typedef typename Vec4<Real>::T R4g;
    R4g *ctrl = (R4g *)a.ctrl;
    Real *vctrl = (Real *)a.vctrl;

    // the gate table in LDS: a gate switch inside the pipeline then waits on
    // no global load (which would also wait on the wave's sample stores)
    if (OBJ == OBJ_GATE)
        for (int i = threadIdx.x; i < 8 * a.G; i += blockDim.x) s_gtab[i] = gtab[i];
    // the shifted warm start (Alg. 1, warm start) of every step, staged once
    // so that the sampling wave reads it from LDS instead of waiting on a
    // dependent global load per step
    for (int k = threadIdx.x; k < N; k += blockDim.x) {
        int src = k + h.shift;
        if (src > N - 1) src = N - 1;
        R4 o;
        o.x = h.warm ? (Real)a.wU[4 * src + 0] : hover;
        o.y = h.warm ? (Real)a.wU[4 * src + 1] : hover;
        o.z = h.warm ? (Real)a.wU[4 * src + 2] : hover;
        o.w = h.warm ? (Real)a.wU[4 * src + 3] : hover;
        s_us[k] = o;
        if (HAS_V) s_vs[k] = h.warm ? (Real)a.wV[src] : Real(0);
        // the weighted average regenerates the samples from these rows
        if (a.regen && blk == (K >> 6)) {
            ((R4 *)a.nomU)[k] = o;
            if (HAS_V) ((Real *)a.nomV)[k] = s_vs[k];
        }
    }
    __syncthreads();
    if (OBJ == OBJ_GATE) {
        gt.load(s_gtab, g);
        g0r = gt;
    }

    const int nch = (N + B - 1) / B;
    for (int c = 0; c <= nch + 1; ++c) {
        if (wave == 0 && c < nch) {
            const int kb = c * B, ke = min(N, kb + B);
            auto noise_step = [&](const int k, const int j) {
                const R4 w4 = s_us[k];
                const Real us[4] = {w4.x, w4.y, w4.z, w4.w};
                const Real vs = HAS_V ? s_vs[k] : Real(0);
                R4 u;
                Real V = Real(0);
                if (sampled) {
                    const Normal4<Real> z = normals4<Real>((uint32_t)m, (uint32_t)k, h.s, 0u, a.seed_lo, a.seed_hi);
                    u.x = clampT(us[0] + sig0 * z.z0, tmin, tmax);
                    u.y = clampT(us[1] + sig1 * z.z1, tmin, tmax);
                    u.z = clampT(us[2] + sig2 * z.z2, tmin, tmax);
                    u.w = clampT(us[3] + sig3 * z.z3, tmin, tmax);
                    const size_t idx = (size_t)k * (size_t)K + (size_t)m;
                    if (!a.regen) store_nt(&ctrl[idx], u);
                    if (HAS_V) {
                        const Real zv = normal1<Real>((uint32_t)m, (uint32_t)k, h.s, 1u, a.seed_lo, a.seed_hi);
                        V = clampT(vs + sigv * zv, Real(0), vmax);
                        if (!a.regen) store_nt(&vctrl[idx], V);
                    }
                } else {  // the noise-free nominal (and idle lanes past it)
                    u.x = clampT(us[0], tmin, tmax);
                    u.y = clampT(us[1], tmin, tmax);
                    u.z = clampT(us[2], tmin, tmax);
                    u.w = clampT(us[3], tmin, tmax);
                    if (HAS_V) V = clampT(vs, Real(0), vmax);
                }
                if (HAS_V) s_v[c % 3][j][lane] = V;
                if (OBJ != OBJ_GATE) {
                    const Real d0 = u.x - up[0], d1 = u.y - up[1], d2 = u.z - up[2], d3 = u.w - up[3];
                    Real term = rdt[0] * d0 * d0 + rdt[1] * d1 * d1 + rdt[2] * d2 * d2 + rdt[3] * d3 * d3;
                    if (HAS_V) {
                        const Real dv = V - vp;
                        term += r_dv * dv * dv;
                        term -= (Real)a.mu * V;
                        vp = V;
                    }
                    J.add(term);
                    up[0] = u.x; up[1] = u.y; up[2] = u.z; up[3] = u.w;
                }
                const StepInput<Real> in = step_input(M, u.x, u.y, u.z, u.w);
                R4 o;
                o.x = in.fm; o.y = in.tx; o.z = in.ty; o.w = in.tz;
                s_in[c % 3][j][lane] = o;
            };
            if (ke - kb == B) {
#pragma unroll
                for (int j = 0; j < B; ++j) noise_step(kb + j, j);
            } else {
                for (int k = kb; k < ke; ++k) noise_step(k, k - kb);
            }
        } else if (wave == 1 && c >= 1 && c <= nch) {
            const int kb = (c - 1) * B, ke = min(N, kb + B);
            auto rot_step = [&](const int k, const int j) {
                const R4 in = s_in[(c - 1) % 3][j][lane];
                R4 (*slot)[64] = s_q[(c - 1) & 1][j];
                Real term = Real(0);
                if (OBJ == OBJ_TRACK) {
                    int r = i0 + k;
                    if (r > a.R - 1) r = a.R - 1;
                    const Real *xr = xref + 16 * r;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const Real e = q[i] - xr[6 + i];
                        term += (Real)a.Q[6 + i] * e * e;
                    }
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = w[i] - xr[10 + i];
                        term += (Real)a.Q[10 + i] * e * e;
                    }
                }
                if (OBJ == OBJ_CONTOUR)
                    term += (Real)a.Q_w[0] * w[0] * w[0] + (Real)a.Q_w[1] * w[1] * w[1] +
                            (Real)a.Q_w[2] * w[2] * w[2];
                Real ws[3], qs[4], kw[3], kq[4], dw[3], dq[4];
#pragma unroll
                for (int i = 0; i < 3; ++i) ws[i] = w[i];
#pragma unroll
                for (int i = 0; i < 4; ++i) qs[i] = q[i];
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    R4 o;
                    o.x = qs[0]; o.y = qs[1]; o.z = qs[2]; o.w = qs[3];
                    slot[st][lane] = o;
                    kw[0] = in.y - M.gx * ws[1] * ws[2];
                    kw[1] = in.z - M.gy * ws[2] * ws[0];
                    kw[2] = in.w - M.gz * ws[0] * ws[1];
                    // kq is twice the quaternion rate; the factor 1/2 is
                    // carried by the step sizes (exact: a power of two)
                    kq[0] = -qs[1] * ws[0] - qs[2] * ws[1] - qs[3] * ws[2];
                    kq[1] = qs[0] * ws[0] + qs[2] * ws[2] - qs[3] * ws[1];
                    kq[2] = qs[0] * ws[1] - qs[1] * ws[2] + qs[3] * ws[0];
                    kq[3] = qs[0] * ws[2] + qs[1] * ws[1] - qs[2] * ws[0];
                    if (st == 0) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] = kw[i];
#pragma unroll
                        for (int i = 0; i < 4; ++i) dq[i] = kq[i];
                    } else if (st < 3) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] += Real(2) * kw[i];
#pragma unroll
                        for (int i = 0; i < 4; ++i) dq[i] += Real(2) * kq[i];
                    } else {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] = dt6 * (dw[i] + kw[i]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) dq[i] = dt12 * (dq[i] + kq[i]);
                    }
                    if (st < 3) {
                        const Real hh = st < 2 ? h2 : dt;
                        const Real hq = st < 2 ? h4 : h2;
#pragma unroll
                        for (int i = 0; i < 3; ++i) ws[i] = w[i] + hh * kw[i];
#pragma unroll
                        for (int i = 0; i < 4; ++i) qs[i] = q[i] + hq * kq[i];
                    }
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) w[i] += dw[i];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] += dq[i];
                renormalize(q);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = fmax(fabs(w[i]) - w_max, Real(0));
                    term += w_lim * e * e;
                }
                J.add(term);
            };
            if (ke - kb == B) {
#pragma unroll
                for (int j = 0; j < B; ++j) rot_step(kb + j, j);
            } else {
                for (int k = kb; k < ke; ++k) rot_step(k, k - kb);
            }
        } else if (wave == 2 && c >= 2) {
            const int kb = (c - 2) * B, ke = min(N, kb + B);
            auto trans_step = [&](const int k, const int j) {
                const R4 in = s_in[(c - 2) % 3][j][lane];
                R4 qstage[4];
#pragma unroll
                for (int st = 0; st < 4; ++st) qstage[st] = s_q[(c - 2) & 1][j][st][lane];
                const Real fm = in.x;
                Real term = Real(0);
                Real ax = 0, ay = 0, az = 0;
                if (OBJ == OBJ_GATE) {
                    ax = p[0] - gt.cx;
                    ay = p[1] - gt.cy;
                    az = p[2] - gt.cz;
                    const Real bx = p[0] - g0r.cx;
                    const Real by = p[1] - g0r.cy;
                    const Real bz = p[2] - g0r.cz;
                    const Real d2 = bx * bx + by * by + bz * bz;
                    if (d2 < r_near2) term += q_near * d2;
                    if (nominal) s_f8[k] = (bx * g0r.nx + by * g0r.ny) < Real(0);
                } else if (OBJ == OBJ_TRACK) {
                    int r = i0 + k;
                    if (r > a.R - 1) r = a.R - 1;
                    const Real *xr = xref + 16 * r;
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = p[i] - xr[i];
                        term += (Real)a.Q[i] * e * e;
                    }
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const Real e = v[i] - xr[3 + i];
                        term += (Real)a.Q[3 + i] * e * e;
                    }
                } else {
                    const Real vk = s_v[(c - 2) % 3][j][lane];
                    const Real fl = floor(th_hi * inv_ds);
                    const Real f = ((th_hi - fl * ds) + th_lo) * inv_ds;
                    const int i = (fl >= Real(0) && fl < Real(1 << 30)) ? ((int)fl % a.P) : 0;
                    const int i1 = (i + 1 == a.P) ? 0 : i + 1;
                    const Real *A = path + 8 * i, *Bp = path + 8 * i1;
                    const Real g1 = Real(1) - f;
                    const Real px = g1 * A[0] + f * Bp[0], py = g1 * A[1] + f * Bp[1], pz = g1 * A[2] + f * Bp[2];
                    Real tx = g1 * A[3] + f * Bp[3], ty = g1 * A[4] + f * Bp[4], tz = g1 * A[5] + f * Bp[5];
                    const Real tn = inv_sqrt(tx * tx + ty * ty + tz * tz);
                    tx *= tn; ty *= tn; tz *= tn;
                    const Real ex = p[0] - px;
                    const Real ey = p[1] - py;
                    const Real ez = p[2] - pz;
                    const Real et = ex * tx + ey * ty + ez * tz;
                    const Real lx = et * tx, ly = et * ty, lz = et * tz;
                    const Real cxe = ex - lx, cye = ey - ly, cze = ez - lz;
                    term += (Real)a.q_l * (lx * lx + ly * ly + lz * lz);
                    term += (Real)a.q_c * (cxe * cxe + cye * cye + cze * cze);
                    const Real y = vk * dt + th_lo;
                    const Real t = th_hi + y;
                    th_lo = (sizeof(Real) == 4) ? y - (t - th_hi) : Real(0);
                    th_hi = t;
                    if (th_hi >= L) th_hi -= L;
                }
                Real vs[3], kv[3], dpv[3], dvv[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) vs[i] = v[i];
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const R4 qq = qstage[st];
                    const Real r3x = Real(2) * (qq.y * qq.w + qq.x * qq.z);
                    const Real r3y = Real(2) * (qq.z * qq.w - qq.x * qq.y);
                    const Real r3z = Real(1) - Real(2) * (qq.y * qq.y + qq.z * qq.z);
                    kv[0] = fm * r3x;
                    kv[1] = fm * r3y;
                    kv[2] = fm * r3z - M.g;
                    if (M.drag) {
                        const Real qw = qq.x, qx = qq.y, qy = qq.z, qz = qq.w;
                        const Real r11 = Real(1) - Real(2) * (qy * qy + qz * qz), r12 = Real(2) * (qx * qy - qw * qz);
                        const Real r21 = Real(2) * (qx * qy + qw * qz), r22 = Real(1) - Real(2) * (qx * qx + qz * qz);
                        const Real r31 = Real(2) * (qx * qz - qw * qy), r32 = Real(2) * (qy * qz + qw * qx);
                        const Real b0 = M.d0 * (r11 * vs[0] + r21 * vs[1] + r31 * vs[2]);
                        const Real b1 = M.d1 * (r12 * vs[0] + r22 * vs[1] + r32 * vs[2]);
                        const Real b2 = M.d2 * (r3x * vs[0] + r3y * vs[1] + r3z * vs[2]);
                        kv[0] -= r11 * b0 + r12 * b1 + r3x * b2;
                        kv[1] -= r21 * b0 + r22 * b1 + r3y * b2;
                        kv[2] -= r31 * b0 + r32 * b1 + r3z * b2;
                    }
                    if (st == 0) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) { dpv[i] = vs[i]; dvv[i] = kv[i]; }
                    } else if (st < 3) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) { dpv[i] += Real(2) * vs[i]; dvv[i] += Real(2) * kv[i]; }
                    } else {
#pragma unroll
                        for (int i = 0; i < 3; ++i) { dpv[i] = dt6 * (dpv[i] + vs[i]); dvv[i] = dt6 * (dvv[i] + kv[i]); }
                    }
                    if (st < 3) {
                        const Real hh = st < 2 ? h2 : dt;
#pragma unroll
                        for (int i = 0; i < 3; ++i) vs[i] = v[i] + hh * kv[i];
                    }
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    p[i] += dpv[i];
                    v[i] += dvv[i];
                }
                if (OBJ == OBJ_GATE) {
                    term += dpv[0] * (Real(2) * ax + dpv[0]) + dpv[1] * (Real(2) * ay + dpv[1]) +
                            dpv[2] * (Real(2) * az + dpv[2]);
                    const Real sa = ax * gt.nx + ay * gt.ny;
                    const Real sb = (ax + dpv[0]) * gt.nx + (ay + dpv[1]) * gt.ny;
                    if (sa < Real(0) && sb >= Real(0)) {
                        const Real t = sa / (sa - sb);
                        const Real yx = ax + t * dpv[0], yy = ay + t * dpv[1], yz = az + t * dpv[2];
                        const Real lat = yx * gt.hx + yy * gt.hy;
                        const bool inside = fabs(lat) <= half && fabs(yz) <= half;
                        const int jj = k + 1;
                        const bool allowed = passes > 0 || ((h.allow[jj >> 5] >> (jj & 31)) & 1u);
                        if (inside && allowed) {
                            g = (g + 1 == a.G) ? 0 : g + 1;
                            ++passes;
                            gt.load(s_gtab, g);
                        }
                    }
                }
                J.add(term);
            };
            if (ke - kb == B) {
#pragma unroll
                for (int j = 0; j < B; ++j) trans_step(kb + j, j);
            } else {
                for (int k = kb; k < ke; ++k) trans_step(k, k - kb);
            }
        }
        __syncthreads();
    }

    if (OBJ == OBJ_TRACK && wave > 0) {
        int r = i0 + N;
        if (r > a.R - 1) r = a.R - 1;
        const Real *xr = xref + 16 * r;
        Real term = 0;
        if (wave == 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const Real e = q[i] - xr[6 + i];
                term += (Real)a.QN[6 + i] * e * e;
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const Real e = w[i] - xr[10 + i];
                term += (Real)a.QN[10 + i] * e * e;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const Real e = p[i] - xr[i];
                term += (Real)a.QN[i] * e * e;
                const Real f = v[i] - xr[3 + i];
                term += (Real)a.QN[3 + i] * f * f;
            }
        }
        J.add(term);
    }
    if (wave < 2) s_jp[wave][lane] = J.value();
    __syncthreads();
    if (wave == 2) {
        Real Jfinal = Real(0);
        if (active) {
            Jfinal = (s_jp[0][lane] + s_jp[1][lane]) + J.value();
            if (OBJ == OBJ_GATE && nominal) {
                const Real bx = p[0] - g0r.cx;
                const Real by = p[1] - g0r.cy;
                a.front8[N] = (bx * g0r.nx + by * g0r.ny) < Real(0);
            }
            if (nominal) a.cur->J_nom = (double)Jfinal;
            else ((Real *)a.J)[m] = Jfinal;
        }
        // the tile of the nominal writes its front flags of steps 0..N-1
        if (OBJ == OBJ_GATE && blk == (K >> 6))
            for (int i = lane; i < N; i += 64) a.front8[i] = s_f8[i];
        store_tile_min(Jfinal, active && !nominal && isfinite(Jfinal), a.tmin, blk);
    }
    __syncthreads();
}

// ---------------------------------------------------------------- rollout, pipelined

// The step of Eq. (2) split into pipeline stages over the waves of one
// workgroup, a 64-sample tile per workgroup:
//   rates        integrates the body rates (they depend on the torques only),
//                for the gate objective with their rate-limit term;
//   attitude     integrates the attitude from the stage body rates;
//   position     integrates position and velocity from the stage attitudes;
//   costs        adds the cost terms of position (gate progress, near-gate
//                term, crossing and switch; contouring; tracking of position
//                and velocity) and, for contouring, of the body rates;
//   terms        (tracking) the cost terms of attitude and body rates;
//                (contouring) the path point and tangent of each step, which
//                depend on the drawn progress speeds only, and the input terms;
//   draws        the noise and the clipped inputs (Eq. (3)), four waves.
// Each stage hands its stage values on through an LDS ring of steps and runs
// as far ahead as the rings allow: a stage publishes how many steps it has
// done in a counter in LDS, its consumer starts a step once the counter has
// passed it, and a producer waits while the ring slot that it would overwrite
// has not been read.  No workgroup barrier falls inside the horizon: with
// barriers between chunks of 4 steps every stage paid about 1,100 cycles per
// chunk for the handoff (LDS latency at its start, the drain at its end, the
// slowest stage).  What bounds a step now is the issue of the busiest wave:
// the attitude's 85 operations at 5 cycles and its 4 LDS writes at 28 make
// 630 cycles a step (binary32).  Solves on 129 tiles, gate, N = 100: 46.5 ->
// 43.0 us; contouring, 94 tiles: 53.8 -> 50.5; tracking, 470 tiles, N = 50:
// 53.5 -> 43.9; binary64, 129 tiles, N = 100: 130 -> 64 us (there the draws
// moved to waves of their own as well).

// Progress counters of the pipeline, one set per workgroup in LDS.  The
// drawing waves publish the next step they will draw, the stages the number
// of steps they have done.
enum PipeCounter { PC_DRAW = 0, PC_RATE = 4, PC_ATT = 5, PC_POS = 6, PC_COST = 7, PC_TERM = 8, PC_CHAIN = 9, PC_N = 16 };

// One stage of the pipeline over the steps 0..N-1: load(k, in) reads the
// inputs of step k from the rings, step(k, in) computes it and writes its
// output.  The counters and then the inputs of step k + 1 are read while step
// k computes: if the counters show that the inputs were there, the next step
// finds them in registers, else both are read again.
// A step may also prepare its successor's inputs (nxt); first does so for step 0.
template <typename In, typename Load, typename Step, typename First>
__device__ __forceinline__ void pipe_run(const int N, const PipeWatch watch, int *const mine, Load load, Step step,
                                         First first)
{
    In a, b;
    watch.wait<0>(0);
    load(0, a);
    first(a);
    int k = 0;
    auto one = [&](In &cur, In &nxt) {
        int seen = watch.peek();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "singlethread");
        load(k + 1, nxt);
        step(k, cur, nxt);
        pipe_publish(mine, ++k);
        if (k == N) return false;
        __builtin_amdgcn_sched_barrier(0);
        if (!PipeWatch::may_start(seen, k)) {
            watch.wait<0>(k);
            load(k, nxt);
        }
        return true;
    };
    while (one(a, b) && one(b, a)) {}
}
template <typename In, typename Load, typename Step>
__device__ __forceinline__ void pipe_run(const int N, const PipeWatch watch, int *const mine, Load load, Step step)
{
    pipe_run<In>(N, watch, mine, load, step, [](In &) {});
}

// Drawing waves of the pipeline: as many as keep the workgroup at eight waves
// in binary32 (two workgroups then share a CU), four in binary64, whose draws
// take several times as long.
constexpr int pipe_draws(int obj, size_t real) { return obj == OBJ_GATE || real == 8 ? 4 : 3; }
// waves of a workgroup: rates, attitude, position, costs, terms (not for the
// gate objective), draws
constexpr int pipe_waves(int obj, size_t real) { return (obj == OBJ_GATE ? 4 : 5) + pipe_draws(obj, real); }

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
// The scheduler would otherwise place an operation right behind the one it
// depends on: a wave issues independent operations every 5 cycles, dependent
// ones every 10 (measured), so the recurrences are written level by level.
template <typename Real> __device__ __forceinline__ void level()
{
    if (sizeof(Real) == 8) __builtin_amdgcn_sched_barrier(0);
}

// R: steps of the stage rings (a power of two); the input rings, which span
// all stages, hold 2 R.
template <int OBJ, typename Real, int R>
__device__ __forceinline__ void rollout4_body(const KArgs &a, int blk, const HeadVals &h)
{
    typedef typename Vec4<Real>::T R4;
    constexpr bool GATE = OBJ == OBJ_GATE, CONT = OBJ == OBJ_CONTOUR, TRACK = OBJ == OBJ_TRACK;
    constexpr bool HAS_V = CONT;
    constexpr int RS = R, RI = 2 * R;
    static_assert((R & (R - 1)) == 0, "slots are taken modulo a power of two");
    constexpr int kDrawWaves = pipe_draws(OBJ, sizeof(Real));
    constexpr int W_DRAW = GATE ? 4 : 5;           // first drawing wave
    __shared__ R4 s_in[RI][64];                    // (F/m, tau_x/J_x, tau_y/J_y, tau_z/J_z)
    __shared__ R4 s_w[RS][4][64];                  // stage body rates
    __shared__ R4 s_q[RS][4][64];                  // stage quaternions
    __shared__ R4 s_p[RS][2][64];                  // p_k and its increment (tracking: v_k)
    __shared__ R4 s_u[GATE ? 1 : RI][64];          // clipped inputs
    __shared__ Real s_v[HAS_V ? RI : 1][64];       // progress speed
    __shared__ R4 s_t[CONT ? RS : 1][2][64];      // path point and input term; path tangent (tracking: p_N, v_N)
    __shared__ R4 s_us[kNMax];                     // shifted warm-start thrusts per step
    __shared__ Real s_vs[HAS_V ? kNMax : 1];       // shifted warm-start progress speed
    __shared__ Real s_jp[3][64];                   // partial costs of the other waves
    __shared__ R4 s_pN[64];                        // p_N (front flag of the nominal)
    __shared__ Real s_gtab[GATE ? 8 * kGMax : 1];  // the gate table, staged once
    __shared__ uint8_t s_f8[GATE ? kNMax : 1];     // front flags of the nominal, steps 0..N-1
    __shared__ int s_cnt[PC_N + 64];               // progress counters; then a word per lane that nothing reads

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int m = blk * 64 + lane;
    const int K = a.K, N = a.N;
    const bool active = m <= K;
    const bool nominal = m == K;
    const bool sampled = m < K;
    const Real dt = (Real)a.dt;
    const Real h2 = Real(0.5) * dt;
    const Real dt6 = dt / Real(6);
    const Real h4 = Real(0.5) * h2, dt12 = Real(0.5) * dt6;
    const Real *xref = (const Real *)a.xref_r;
    const int i0 = h.i0;
    const Real hover = (Real)a.hover;

    // the gate table in LDS: a gate switch inside the pipeline then waits on
    // no global load (which would also wait on the wave's sample stores)
    if (GATE)
        for (int i = threadIdx.x; i < 8 * a.G; i += blockDim.x) s_gtab[i] = ((const Real *)a.gates_r)[i];
    // the shifted warm start of every step, staged once
    for (int k = threadIdx.x; k < N; k += blockDim.x) {
        int src = k + h.shift;
        if (src > N - 1) src = N - 1;
        R4 o;
        o.x = h.warm ? (Real)a.wU[4 * src + 0] : hover;
        o.y = h.warm ? (Real)a.wU[4 * src + 1] : hover;
        o.z = h.warm ? (Real)a.wU[4 * src + 2] : hover;
        o.w = h.warm ? (Real)a.wU[4 * src + 3] : hover;
        s_us[k] = o;
        if (HAS_V) s_vs[k] = h.warm ? (Real)a.wV[src] : Real(0);
        // the weighted average regenerates the samples from these rows
        if (a.regen && blk == (K >> 6)) {
            ((R4 *)a.nomU)[k] = o;
            if (HAS_V) ((Real *)a.nomV)[k] = s_vs[k];
        }
    }
    if (threadIdx.x < PC_N) s_cnt[threadIdx.x] = (int)threadIdx.x < kDrawWaves ? (int)threadIdx.x : 0;
    __syncthreads();

    auto counter = [&](const int c) { return lane == 0 ? &s_cnt[c] : &s_cnt[PC_N + lane]; };
    // rate limit on the body rates after a step
    const Real w_max = (Real)a.w_max, w_lim = (Real)a.w_lim;
    auto rate_limit = [&](const Real wx, const Real wy, const Real wz) {
        const Real ww[3] = {wx, wy, wz};
        Real rl = Real(0);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const Real e = fmax(fabs(ww[i]) - w_max, Real(0));
            rl += w_lim * e * e;
        }
        return rl;
    };
    // row of the tracking reference at state k
    auto ref_row = [&](const int k) {
        int r = i0 + k;
        if (r > a.R - 1) r = a.R - 1;
        return xref + 16 * r;
    };

    KSum<Real> J;       // costs: this wave's own part of the cost (wave 3 holds J_3)
    // two workgroups on a CU: the stages ahead of the draws (tracking, 470
    // tiles, N = 50: 45.4 -> 43.9 us a solve); with one workgroup the issue
    // slots are not short (binary64: 64.6 -> 69.9 us, gate 42.9 -> 43.4)
    if (sizeof(Real) == 4 && R == 4 && wave < W_DRAW) __builtin_amdgcn_s_setprio(3);
    if (wave >= W_DRAW) {
        // the draws: drawing wave i takes the steps i, i + kDrawWaves, ...
        const Model<Real> M(a);
        const Real tmin = (Real)a.t_min, tmax = (Real)a.t_max, vmax = (Real)a.v_max;
        // the noise-free nominal and the idle lanes past it draw with zero
        // noise, so that no step selects between two values
        const Real sig0 = sampled ? (Real)a.sigma[0] : Real(0), sig1 = sampled ? (Real)a.sigma[1] : Real(0);
        const Real sig2 = sampled ? (Real)a.sigma[2] : Real(0), sig3 = sampled ? (Real)a.sigma[3] : Real(0);
        const Real sigv = sampled ? (Real)a.sigma_v : Real(0);
        R4 *ctrl = (R4 *)a.ctrl;
        Real *vctrl = (Real *)a.vctrl;
        const uint32_t s_solve = __builtin_amdgcn_readfirstlane(h.s);
        const uint32_t key0 = __builtin_amdgcn_readfirstlane(a.seed_lo);
        const uint32_t key1 = __builtin_amdgcn_readfirstlane(a.seed_hi);
        const bool keep = sampled && !a.regen;
        // the slot is free once the position stage and the reader of the inputs have read it
        const PipeWatch watch = {&s_cnt[GATE || (lane & 1) == 0 ? PC_POS : (CONT ? PC_TERM : PC_COST)], RI};
        int *const mine = counter(PC_DRAW + wave - W_DRAW);
        for (int k = wave - W_DRAW; k < N; k += kDrawWaves) {
            const R4 us = s_us[k];
            const Normal4<Real> z = normals4<Real>((uint32_t)m, (uint32_t)k, s_solve, 0u, key0, key1);
            R4 u;
            u.x = clamp_finite(us.x + sig0 * z.z0, tmin, tmax);
            u.y = clamp_finite(us.y + sig1 * z.z1, tmin, tmax);
            u.z = clamp_finite(us.z + sig2 * z.z2, tmin, tmax);
            u.w = clamp_finite(us.w + sig3 * z.z3, tmin, tmax);
            Real V = Real(0);
            if (HAS_V) {
                const Real zv = normal1<Real>((uint32_t)m, (uint32_t)k, s_solve, 1u, key0, key1);
                V = clamp_finite(s_vs[k] + sigv * zv, Real(0), vmax);
            }
            // store the samples, hand the inputs on
            if (keep) {
                const size_t idx = (size_t)k * (size_t)K + (size_t)m;
                store_nt(&ctrl[idx], u);
                if (HAS_V) store_nt(&vctrl[idx], V);
            }
            const StepInput<Real> in = step_input(M, u.x, u.y, u.z, u.w);
            R4 o;
            o.x = in.fm; o.y = in.tx; o.z = in.ty; o.w = in.tz;
            watch.wait<2>(k);
            s_in[k & (RI - 1)][lane] = o;
            if (HAS_V) s_v[k & (RI - 1)][lane] = V;
            if (!GATE) s_u[k & (RI - 1)][lane] = u;
            pipe_publish(mine, k + kDrawWaves);
        }
    } else if (wave == 0) {
        // body rates
        const Model<Real> M(a);
        Real w[3];
        for (int i = 0; i < 3; ++i) w[i] = (Real)h.x0[10 + i];
        // inputs drawn; stage slots read by the attitude, the first of them by the rate costs
        const int reader = TRACK ? PC_TERM : PC_COST;
        const PipeWatch watch = {&s_cnt[lane < kDrawWaves ? PC_DRAW + lane : (GATE || (lane & 1) ? PC_ATT : reader)],
                                 lane < kDrawWaves ? 0 : RS};
        auto omega_step = [&](const int k, const R4 &in, R4 &) {
            R4 (*slot)[64] = s_w[k & (RS - 1)];
            Real ws[3], kw[3], dw[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) ws[i] = w[i];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                slot[st][lane].x = ws[0]; slot[st][lane].y = ws[1]; slot[st][lane].z = ws[2];
                kw[0] = in.y - M.gx * ws[1] * ws[2];
                kw[1] = in.z - M.gy * ws[2] * ws[0];
                kw[2] = in.w - M.gz * ws[0] * ws[1];
                if (st == 0) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) dw[i] = kw[i];
                } else if (st < 3) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) dw[i] += Real(2) * kw[i];
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i) dw[i] = dt6 * (dw[i] + kw[i]);
                }
                if (st < 3) {
                    const Real hh = st < 2 ? h2 : dt;
#pragma unroll
                    for (int i = 0; i < 3; ++i) ws[i] = w[i] + hh * kw[i];
                }
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) w[i] += dw[i];
            if (GATE) J.add(rate_limit(w[0], w[1], w[2]));
        };
        pipe_run<R4>(N, watch, counter(PC_RATE), [&](const int k, R4 &in) { in = s_in[k & (RI - 1)][lane]; }, omega_step);
        if (GATE) {
            s_jp[0][lane] = J.value();
        } else {
            // w_N, as the first stage of a step N
            const PipeWatch last = {&s_cnt[lane & 1 ? PC_ATT : reader], RS};
            last.wait<0>(N);
            R4 *const o = s_w[N & (RS - 1)][0];
            o[lane].x = w[0]; o[lane].y = w[1]; o[lane].z = w[2];
            pipe_publish(counter(PC_RATE), N + 1);
        }
    } else if (wave == 1) {
        // attitude
        Real q[4];
        for (int i = 0; i < 4; ++i) q[i] = (Real)h.x0[6 + i];
        struct In { R4 w[4]; };
        const PipeWatch watch = {&s_cnt[lane == 0 ? PC_RATE : (TRACK && (lane & 1) ? PC_TERM : PC_POS)], lane == 0 ? 0 : RS};
        auto quat_step = [&](const int k, const In &wst, In &) {
            R4 (*slot)[64] = s_q[k & (RS - 1)];
            Real qs[4], dq[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) qs[i] = q[i];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const R4 ws = wst.w[st];
                // kq is twice the quaternion rate; the factor 1/2 is
                // carried by the step sizes (exact: a power of two)
                Real kq[4];
                level<Real>();
                kq[0] = -(qs[2] * ws.y);
                kq[1] = qs[2] * ws.z;
                kq[2] = -(qs[1] * ws.z);
                kq[3] = qs[1] * ws.y;
                level<Real>();
                kq[0] = fma_t(-qs[1], ws.x, kq[0]);
                kq[1] = fma_t(qs[0], ws.x, kq[1]);
                kq[2] = fma_t(qs[0], ws.y, kq[2]);
                kq[3] = fma_t(qs[0], ws.z, kq[3]);
                level<Real>();
                kq[0] = fma_t(-qs[3], ws.z, kq[0]);
                kq[1] = fma_t(-qs[3], ws.y, kq[1]);
                kq[2] = fma_t(qs[3], ws.x, kq[2]);
                kq[3] = fma_t(-qs[2], ws.x, kq[3]);
                level<Real>();
                R4 o;
                o.x = qs[0]; o.y = qs[1]; o.z = qs[2]; o.w = qs[3];
                slot[st][lane] = o;
                if (st < 3) {
                    const Real hq = st < 2 ? h4 : h2;
#pragma unroll
                    for (int i = 0; i < 4; ++i) qs[i] = fma_t(hq, kq[i], q[i]);
                }
                level<Real>();
                if (st == 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) dq[i] = kq[i];
                } else if (st < 3) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) dq[i] = fma_t(Real(2), kq[i], dq[i]);
                } else {
                    // the last stage closes the step in one multiply-add
                    // per component (this wave's recurrence sets the pace)
#pragma unroll
                    for (int i = 0; i < 4; ++i) dq[i] = dq[i] + kq[i];
                    level<Real>();
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[i] = fma_t(dt12, dq[i], q[i]);
                }
            }
            level<Real>();
            renormalize(q);
        };
        pipe_run<In>(N, watch, counter(PC_ATT),
                     [&](const int k, In &in) {
#pragma unroll
                         for (int st = 0; st < 4; ++st) in.w[st] = s_w[k & (RS - 1)][st][lane];
                     },
                     quat_step);
        if (TRACK) {
            R4 o;
            o.x = q[0]; o.y = q[1]; o.z = q[2]; o.w = q[3];
            s_pN[lane] = o;     // q_N, for the terminal term
        }
    } else if (wave == 2) {
        // position and velocity
        const Model<Real> M(a);
        Real p[3], v[3];
        for (int i = 0; i < 3; ++i) {
            p[i] = (Real)h.x0[i];
            v[i] = (Real)h.x0[3 + i];
        }
        struct In { Real fm; R4 q[4]; };
        const PipeWatch watch = {&s_cnt[lane == 0 ? PC_ATT : PC_COST], lane == 0 ? 0 : RS};
        // drag is a launch constant: the branch sits outside the step, so the
        // stages of a step (independent without drag) schedule together
        auto trans_step = [&](const int k, const In &in, auto drag_tag) {
            constexpr bool DRAG = decltype(drag_tag)::value;
            const Real fm = in.fm;
            Real vs[3], kv[3], dpv[3], dvv[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) vs[i] = v[i];
            // F/m times the thrust direction; the factor 2 of its first
            // two components rides on F/m (exact: a power of two)
            const Real fm2 = Real(2) * fm;
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const R4 qq = in.q[st];
                const Real r3z = Real(1) - Real(2) * (qq.y * qq.y + qq.z * qq.z);
                kv[0] = fm2 * (qq.y * qq.w + qq.x * qq.z);
                kv[1] = fm2 * (qq.z * qq.w - qq.x * qq.y);
                kv[2] = fm * r3z - M.g;
                if (DRAG) {
                    const Real qw = qq.x, qx = qq.y, qy = qq.z, qz = qq.w;
                    const Real r3x = Real(2) * (qq.y * qq.w + qq.x * qq.z);
                    const Real r3y = Real(2) * (qq.z * qq.w - qq.x * qq.y);
                    const Real r11 = Real(1) - Real(2) * (qy * qy + qz * qz), r12 = Real(2) * (qx * qy - qw * qz);
                    const Real r21 = Real(2) * (qx * qy + qw * qz), r22 = Real(1) - Real(2) * (qx * qx + qz * qz);
                    const Real r31 = Real(2) * (qx * qz - qw * qy), r32 = Real(2) * (qy * qz + qw * qx);
                    const Real b0 = M.d0 * (r11 * vs[0] + r21 * vs[1] + r31 * vs[2]);
                    const Real b1 = M.d1 * (r12 * vs[0] + r22 * vs[1] + r32 * vs[2]);
                    const Real b2 = M.d2 * (r3x * vs[0] + r3y * vs[1] + r3z * vs[2]);
                    kv[0] -= r11 * b0 + r12 * b1 + r3x * b2;
                    kv[1] -= r21 * b0 + r22 * b1 + r3y * b2;
                    kv[2] -= r31 * b0 + r32 * b1 + r3z * b2;
                }
                if (st == 0) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) { dpv[i] = vs[i]; dvv[i] = kv[i]; }
                } else if (st < 3) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) { dpv[i] += Real(2) * vs[i]; dvv[i] += Real(2) * kv[i]; }
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i) { dpv[i] = dt6 * (dpv[i] + vs[i]); dvv[i] = dt6 * (dvv[i] + kv[i]); }
                }
                if (st < 3) {
                    const Real hh = st < 2 ? h2 : dt;
#pragma unroll
                    for (int i = 0; i < 3; ++i) vs[i] = v[i] + hh * kv[i];
                }
            }
            R4 (*ps)[64] = s_p[k & (RS - 1)];
            ps[0][lane].x = p[0]; ps[0][lane].y = p[1]; ps[0][lane].z = p[2];
            const Real *const o2 = TRACK ? v : dpv;
            ps[1][lane].x = o2[0]; ps[1][lane].y = o2[1]; ps[1][lane].z = o2[2];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                p[i] += dpv[i];
                v[i] += dvv[i];
            }
        };
        auto load = [&](const int k, In &in) {
            in.fm = s_in[k & (RI - 1)][lane].x;
#pragma unroll
            for (int st = 0; st < 4; ++st) in.q[st] = s_q[k & (RS - 1)][st][lane];
        };
        if (M.drag)
            pipe_run<In>(N, watch, counter(PC_POS), load,
                         [&](const int k, const In &in, In &) { trans_step(k, in, std::true_type{}); });
        else
            pipe_run<In>(N, watch, counter(PC_POS), load,
                         [&](const int k, const In &in, In &) { trans_step(k, in, std::false_type{}); });
        if (GATE) {
            R4 o;
            o.x = p[0]; o.y = p[1]; o.z = p[2]; o.w = Real(0);
            s_pN[lane] = o;
        }
        if (TRACK) {
            // the terminal term of position and velocity closes the sum of its
            // stage terms, which the cost wave keeps
            s_t[0][0][lane].x = p[0]; s_t[0][0][lane].y = p[1]; s_t[0][0][lane].z = p[2];
            s_t[0][1][lane].x = v[0]; s_t[0][1][lane].y = v[1]; s_t[0][1][lane].z = v[2];
        }
    } else if (wave == 3 && TRACK) {
        // input-rate terms (J) and the tracking terms of position and velocity (J2)
        KSum<Real> J2;
        Real up[4];
        for (int i = 0; i < 4; ++i) up[i] = (Real)h.u_prev[i];
        Real rdt[4];
        for (int i = 0; i < 4; ++i) rdt[i] = (Real)(a.R_dT[i] / (a.dt * a.dt));
        struct In { R4 p, v, u; Real x[6]; };
        const PipeWatch watch = {&s_cnt[PC_POS], 0};
        pipe_run<In>(
            N, watch, counter(PC_COST),
            [&](const int k, In &in) {
                in.p = s_p[k & (RS - 1)][0][lane];
                in.v = s_p[k & (RS - 1)][1][lane];
                in.u = s_u[k & (RI - 1)][lane];
                const Real *xr = ref_row(k);
#pragma unroll
                for (int i = 0; i < 6; ++i) in.x[i] = xr[i];
            },
            [&](const int, const In &in, In &) {
                const Real *xr = in.x;
                const Real p[3] = {in.p.x, in.p.y, in.p.z}, v[3] = {in.v.x, in.v.y, in.v.z};
                Real term = Real(0);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = p[i] - xr[i];
                    term += (Real)a.Q[i] * e * e;
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = v[i] - xr[3 + i];
                    term += (Real)a.Q[3 + i] * e * e;
                }
                J2.add(term);
                const R4 u = in.u;
                const Real d0 = u.x - up[0], d1 = u.y - up[1], d2 = u.z - up[2], d3 = u.w - up[3];
                term = Real(0);
                term += rdt[0] * d0 * d0 + rdt[1] * d1 * d1 + rdt[2] * d2 * d2 + rdt[3] * d3 * d3;
                up[0] = u.x; up[1] = u.y; up[2] = u.z; up[3] = u.w;
                J.add(term);
            });
        __syncthreads();
        const Real *xr = ref_row(N);
        const R4 pN = s_t[0][0][lane], vN = s_t[0][1][lane];
        const Real p[3] = {pN.x, pN.y, pN.z}, v[3] = {vN.x, vN.y, vN.z};
        Real term = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const Real e = p[i] - xr[i];
            term += (Real)a.QN[i] * e * e;
            const Real f = v[i] - xr[3 + i];
            term += (Real)a.QN[3 + i] * f * f;
        }
        J2.add(term);
        s_jp[2][lane] = J2.value();
    } else if (wave == 4 && TRACK) {
        // tracking terms of the body rates with the rate limit (J), and of the attitude (J1)
        KSum<Real> J1;
        R4 w;
        w.x = (Real)h.x0[10]; w.y = (Real)h.x0[11]; w.z = (Real)h.x0[12];
        struct In { R4 q, w; Real x[7]; };
        const PipeWatch watch = {&s_cnt[lane == 0 ? PC_RATE : PC_ATT], lane == 0 ? -1 : 0};
        pipe_run<In>(
            N, watch, counter(PC_TERM),
            [&](const int k, In &in) {
                in.q = s_q[k & (RS - 1)][0][lane];
                in.w = s_w[(k + 1) & (RS - 1)][0][lane];
                const Real *xr = ref_row(k);
#pragma unroll
                for (int i = 0; i < 7; ++i) in.x[i] = xr[6 + i];
            },
            [&](const int, const In &in, In &) {
                const Real *xr = in.x;
                const Real q[4] = {in.q.x, in.q.y, in.q.z, in.q.w}, ww[3] = {w.x, w.y, w.z};
                Real term = Real(0);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const Real e = ww[i] - xr[4 + i];
                    term += (Real)a.Q[10 + i] * e * e;
                }
                J.add(term);
                J.add(rate_limit(in.w.x, in.w.y, in.w.z));
                term = Real(0);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const Real e = q[i] - xr[i];
                    term += (Real)a.Q[6 + i] * e * e;
                }
                J1.add(term);
                w = in.w;
            });
        __syncthreads();
        const Real *xr = ref_row(N);
        const R4 qN = s_pN[lane];
        const Real q[4] = {qN.x, qN.y, qN.z, qN.w}, ww[3] = {w.x, w.y, w.z};
        Real term = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const Real e = ww[i] - xr[10 + i];
            term += (Real)a.QN[10 + i] * e * e;
        }
        J.add(term);
        term = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const Real e = q[i] - xr[6 + i];
            term += (Real)a.QN[6 + i] * e * e;
        }
        J1.add(term);
        s_jp[0][lane] = J.value();
        s_jp[1][lane] = J1.value();
    } else if (wave == 4 && CONT) {
        // path point and tangent of every step, and the terms of the inputs
        Real up[4], vp = (Real)h.v_prev;
        for (int i = 0; i < 4; ++i) up[i] = (Real)h.u_prev[i];
        Real rdt[4];
        for (int i = 0; i < 4; ++i) rdt[i] = (Real)(a.R_dT[i] / (a.dt * a.dt));
        const Real r_dv = (Real)(a.r_dv / (a.dt * a.dt)), mu = (Real)a.mu;
        const Real *path = (const Real *)a.path_r;
        Real th_hi = (Real)h.theta0, th_lo = 0;
        if (sizeof(Real) == 4) th_lo = (Real)(h.theta0 - (double)th_hi);
        const Real L = (Real)a.path_len;
        const Real ds = (Real)(a.path_len / (double)a.P), inv_ds = (Real)((double)a.P / a.path_len);
        // u, V and the table rows around theta_k with its place between them
        struct In { R4 u; Real V, f; R4 A0, A1, B0, B1; };
        auto rows = [&](In &in) {
            const Real fl = floor(th_hi * inv_ds);
            in.f = ((th_hi - fl * ds) + th_lo) * inv_ds;
            const int i = (fl >= Real(0) && fl < Real(1 << 30)) ? ((int)fl % a.P) : 0;
            const int i1 = (i + 1 == a.P) ? 0 : i + 1;
            const R4 *A = (const R4 *)(path + 8 * i), *B = (const R4 *)(path + 8 * i1);
            in.A0 = A[0]; in.A1 = A[1]; in.B0 = B[0]; in.B1 = B[1];
        };
        const PipeWatch watch = {&s_cnt[lane < kDrawWaves ? PC_DRAW + lane : PC_COST], lane < kDrawWaves ? 0 : RS};
        pipe_run<In>(
            N, watch, counter(PC_TERM),
            [&](const int k, In &in) {
                in.u = s_u[k & (RI - 1)][lane];
                in.V = s_v[k & (RI - 1)][lane];
            },
            [&](const int k, const In &in, In &nxt) {
                const Real V = in.V;
                {   // theta_{k+1}; its table rows are in flight while this step computes
                    const Real y = V * dt + th_lo;
                    const Real t = th_hi + y;
                    th_lo = (sizeof(Real) == 4) ? y - (t - th_hi) : Real(0);
                    th_hi = t;
                    if (th_hi >= L) th_hi -= L;
                    rows(nxt);
                }
                Real term = Real(0);
                const R4 u = in.u;
                const Real d0 = u.x - up[0], d1 = u.y - up[1], d2 = u.z - up[2], d3 = u.w - up[3];
                term += rdt[0] * d0 * d0 + rdt[1] * d1 * d1 + rdt[2] * d2 * d2 + rdt[3] * d3 * d3;
                up[0] = u.x; up[1] = u.y; up[2] = u.z; up[3] = u.w;
                const Real dv = V - vp;
                term += r_dv * dv * dv;
                term -= mu * V;
                vp = V;
                const Real f = in.f, g1 = Real(1) - f;
                const Real A[6] = {in.A0.x, in.A0.y, in.A0.z, in.A0.w, in.A1.x, in.A1.y};
                const Real Bp[6] = {in.B0.x, in.B0.y, in.B0.z, in.B0.w, in.B1.x, in.B1.y};
                const Real px = g1 * A[0] + f * Bp[0], py = g1 * A[1] + f * Bp[1], pz = g1 * A[2] + f * Bp[2];
                Real tx = g1 * A[3] + f * Bp[3], ty = g1 * A[4] + f * Bp[4], tz = g1 * A[5] + f * Bp[5];
                const Real tn = inv_sqrt(tx * tx + ty * ty + tz * tz);
                tx *= tn; ty *= tn; tz *= tn;
                R4 (*o)[64] = s_t[k & (RS - 1)];
                R4 c;
                c.x = px; c.y = py; c.z = pz; c.w = term;
                o[0][lane] = c;
                o[1][lane].x = tx; o[1][lane].y = ty; o[1][lane].z = tz;
            },
            rows);
    } else if (CONT) {
        // contouring errors (J), body-rate terms (J0)
        KSum<Real> J0;
        const Real q_l = (Real)a.q_l, q_c = (Real)a.q_c;
        const Real qw0 = (Real)a.Q_w[0], qw1 = (Real)a.Q_w[1], qw2 = (Real)a.Q_w[2];
        R4 w;
        w.x = (Real)h.x0[10]; w.y = (Real)h.x0[11]; w.z = (Real)h.x0[12];
        struct In { R4 p, c, t, w; };
        const PipeWatch watch = {&s_cnt[lane == 0 ? PC_RATE : (lane & 1 ? PC_POS : PC_TERM)], lane == 0 ? -1 : 0};
        pipe_run<In>(
            N, watch, counter(PC_COST),
            [&](const int k, In &in) {
                in.p = s_p[k & (RS - 1)][0][lane];
                in.c = s_t[k & (RS - 1)][0][lane];
                in.t = s_t[k & (RS - 1)][1][lane];
                in.w = s_w[(k + 1) & (RS - 1)][0][lane];
            },
            [&](const int, const In &in, In &) {
                Real term = Real(0);
                term += qw0 * w.x * w.x + qw1 * w.y * w.y + qw2 * w.z * w.z;
                J0.add(term);
                J0.add(rate_limit(in.w.x, in.w.y, in.w.z));
                w = in.w;
                term = in.c.w;
                const Real tx = in.t.x, ty = in.t.y, tz = in.t.z;
                const Real ex = in.p.x - in.c.x;
                const Real ey = in.p.y - in.c.y;
                const Real ez = in.p.z - in.c.z;
                const Real et = ex * tx + ey * ty + ez * tz;
                const Real lx = et * tx, ly = et * ty, lz = et * tz;
                const Real cxe = ex - lx, cye = ey - ly, cze = ez - lz;
                term += q_l * (lx * lx + ly * ly + lz * lz);
                term += q_c * (cxe * cxe + cye * cye + cze * cze);
                J.add(term);
            });
        __syncthreads();
        s_jp[0][lane] = J0.value();
        s_jp[1][lane] = Real(0);
        s_jp[2][lane] = Real(0);
    } else if (GATE) {
        // gate progress, near-gate term, crossing and switch
        const Real q_near = (Real)a.q_near, r_near2 = (Real)(a.r_near * a.r_near), half = (Real)a.gate_half;
        GateRegs<Real> gt, g0r;
        int g = h.g0, passes = 0;
        gt.load(s_gtab, g);
        g0r = gt;
        struct In { R4 p, d; };
        const PipeWatch watch = {&s_cnt[PC_POS], 0};
        pipe_run<In>(
            N, watch, counter(PC_COST),
            [&](const int k, In &in) {
                in.p = s_p[k & (RS - 1)][0][lane];
                in.d = s_p[k & (RS - 1)][1][lane];
            },
            [&](const int k, const In &in, In &) {
                Real term = Real(0);
                const Real pk[3] = {in.p.x, in.p.y, in.p.z};
                const Real dpv[3] = {in.d.x, in.d.y, in.d.z};
                const Real ax = pk[0] - gt.cx;
                const Real ay = pk[1] - gt.cy;
                const Real az = pk[2] - gt.cz;
                const Real bx = pk[0] - g0r.cx;
                const Real by = pk[1] - g0r.cy;
                const Real bz = pk[2] - g0r.cz;
                const Real d2 = bx * bx + by * by + bz * bz;
                if (d2 < r_near2) term += q_near * d2;
                if (nominal) s_f8[k] = (bx * g0r.nx + by * g0r.ny) < Real(0);
                term += dpv[0] * (Real(2) * ax + dpv[0]) + dpv[1] * (Real(2) * ay + dpv[1]) +
                        dpv[2] * (Real(2) * az + dpv[2]);
                const Real sa = ax * gt.nx + ay * gt.ny;
                const Real sb = (ax + dpv[0]) * gt.nx + (ay + dpv[1]) * gt.ny;
                if (sa < Real(0) && sb >= Real(0)) {
                    const Real t = sa / (sa - sb);
                    const Real yx = ax + t * dpv[0], yy = ay + t * dpv[1], yz = az + t * dpv[2];
                    const Real lat = yx * gt.hx + yy * gt.hy;
                    const bool inside = fabs(lat) <= half && fabs(yz) <= half;
                    const int jj = k + 1;
                    const bool allowed = passes > 0 || ((h.allow[jj >> 5] >> (jj & 31)) & 1u);
                    if (inside && allowed) {
                        g = (g + 1 == a.G) ? 0 : g + 1;
                        ++passes;
                        gt.load(s_gtab, g);
                    }
                }
                J.add(term);
            });
        __syncthreads();
        if (nominal) {
            const R4 ph = s_pN[lane];
            const Real bx = ph.x - g0r.cx;
            const Real by = ph.y - g0r.cy;
            a.front8[N] = (bx * g0r.nx + by * g0r.ny) < Real(0);
        }
        // the tile of the nominal writes its front flags of steps 0..N-1
        if (blk == (K >> 6))
            for (int i = lane; i < N; i += 64) a.front8[i] = s_f8[i];
        s_jp[1][lane] = Real(0);
        s_jp[2][lane] = Real(0);
    }
    // (the cost waves meet the others at their own first barrier above)
    if (!((wave == 3) || (wave == 4 && TRACK))) __syncthreads();
    __syncthreads();
    if (wave == 3) {
        Real Jfinal = Real(0);
        if (active) {
            Jfinal = ((s_jp[0][lane] + s_jp[1][lane]) + s_jp[2][lane]) + J.value();
            if (nominal) a.cur->J_nom = (double)Jfinal;
            else ((Real *)a.J)[m] = Jfinal;
        }
        store_tile_min(Jfinal, active && !nominal && isfinite(Jfinal), a.tmin, blk);
    }
    __syncthreads();
}

template <int OBJ, typename Real, int R>
__global__ __launch_bounds__(64 * pipe_waves(OBJ, sizeof(Real))) void k_rollout4(KArgs a)
{
    __shared__ HeadVals h;
    compute_head<OBJ == OBJ_CONTOUR>(a, h);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish_head(a, h);
    rollout4_body<OBJ, Real, R>(a, blockIdx.x, h);
}

// ---------------------------------------------------------------- rollout, pipelined, rate input

// The pipeline for the rate input (17 states), with the order of operations
// of the one-wave rollout, so that its results are those bit for bit (a batch
// steps rate contexts with one-wave rollouts).  One stage more than above:
//   draws        the rates (and contouring's progress acceleration), clipped
//                to their bounds;
//   chain        the thrust chain in binary64: the clip to the range that
//                keeps each thrust in [t_min, t_max], the sample tensor, the
//                thrusts at the middle and the end of the step;
//   rates, attitude, position as above, from the stage thrusts;
//   terms        (contouring) the speed chain and its clip, the path point and
//                tangent, the input terms;
//   costs        all cost terms of a step, in the one-wave order.
// A lone wave took 1.1 us a step (K = 8192, N = 20: 22 us behind a 5.6 us
// sample pass); the stages overlap to about 0.3 us a step.  Calls through the
// host entry point at K = 8192, N = 20: gate 49.5 -> 39.5 us, contouring 60.8
// -> 45.4, tracking 52.7 -> 40.0; binary64 gate, K = 4001, N = 33: 72.8 -> 58.9.
constexpr int rate_pipe_draws = 3;
constexpr int rate_pipe_waves(int obj) { return (obj == OBJ_CONTOUR ? 6 : 5) + rate_pipe_draws; }

template <int OBJ, typename Real, int R>
__device__ __forceinline__ void rollout_rate_body(const KArgs &a, int blk, const HeadVals &h)
{
    typedef typename Vec4<Real>::T R4;
    constexpr bool GATE = OBJ == OBJ_GATE, CONT = OBJ == OBJ_CONTOUR, TRACK = OBJ == OBJ_TRACK;
    constexpr int RS = R, RI = 2 * R;
    static_assert((R & (R - 1)) == 0, "slots are taken modulo a power of two");
    constexpr int kDrawWaves = rate_pipe_draws;
    constexpr int W_DRAW = CONT ? 6 : 5;
    __shared__ R4 s_r[RI][64];                     // drawn rates within their bounds
    __shared__ R4 s_T[RI][2][64];                  // thrusts at the middle and the end of the step
    __shared__ R4 s_w[RS][4][64];                  // stage body rates
    __shared__ R4 s_q[RS][4][64];                  // stage quaternions
    __shared__ R4 s_p[RS][CONT ? 1 : 2][64];       // p_k and (gate) its increment, (tracking) v_k
    __shared__ R4 s_u[GATE ? 1 : RI][64];          // clipped rates
    __shared__ Real s_v[CONT ? RI : 1][64];        // drawn progress acceleration
    __shared__ R4 s_t[CONT ? RS : 1][3][64];       // path point, tangent, input terms; acceleration, speed
    __shared__ R4 s_us[kNMax];                     // shifted warm-start rates per step
    __shared__ Real s_vs[CONT ? kNMax : 1];        // shifted warm-start acceleration
    __shared__ R4 s_end[3][64];                    // p_N, v_N, q_N
    __shared__ Real s_gtab[GATE ? 8 * kGMax : 1];  // the gate table, staged once
    __shared__ uint8_t s_f8[GATE ? kNMax : 1];     // front flags of the nominal, steps 0..N-1
    __shared__ int s_cnt[PC_N + 64];               // progress counters; then a word per lane that nothing reads

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int m = blk * 64 + lane;
    const int K = a.K, N = a.N;
    const bool active = m <= K;
    const bool nominal = m == K;
    const bool sampled = m < K;
    const Real dt = (Real)a.dt;
    const Real h2 = Real(0.5) * dt;
    const Real dt6 = dt / Real(6);
    const Real h4 = Real(0.5) * h2, dt12 = Real(0.5) * dt6;

    if (GATE)
        for (int i = threadIdx.x; i < 8 * a.G; i += blockDim.x) s_gtab[i] = ((const Real *)a.gates_r)[i];
    for (int k = threadIdx.x; k < N; k += blockDim.x) {
        int src = k + h.shift;
        if (src > N - 1) src = N - 1;
        R4 o;
        o.x = h.warm ? (Real)a.wU[4 * src + 0] : (Real)a.hover;
        o.y = h.warm ? (Real)a.wU[4 * src + 1] : (Real)a.hover;
        o.z = h.warm ? (Real)a.wU[4 * src + 2] : (Real)a.hover;
        o.w = h.warm ? (Real)a.wU[4 * src + 3] : (Real)a.hover;
        s_us[k] = o;
        if (CONT) s_vs[k] = h.warm ? (Real)a.wV[src] : Real(0);
    }
    if (threadIdx.x < PC_N) s_cnt[threadIdx.x] = (int)threadIdx.x < kDrawWaves ? (int)threadIdx.x : 0;
    __syncthreads();

    auto counter = [&](const int c) { return lane == 0 ? &s_cnt[c] : &s_cnt[PC_N + lane]; };
    if (wave >= W_DRAW) {
        const Real rlo = (Real)a.rate_lim[0], rhi = (Real)a.rate_lim[1];
        const Real dlo = (Real)a.dv_lim[0], dhi = (Real)a.dv_lim[1];
        const Real sig0 = sampled ? (Real)a.sigma[0] : Real(0), sig1 = sampled ? (Real)a.sigma[1] : Real(0);
        const Real sig2 = sampled ? (Real)a.sigma[2] : Real(0), sig3 = sampled ? (Real)a.sigma[3] : Real(0);
        const Real sigv = sampled ? (Real)a.sigma_v : Real(0);
        const uint32_t s_solve = __builtin_amdgcn_readfirstlane(h.s);
        const PipeWatch watch = {&s_cnt[CONT && (lane & 1) ? PC_TERM : PC_CHAIN], RI};
        int *const mine = counter(PC_DRAW + wave - W_DRAW);
        for (int k = wave - W_DRAW; k < N; k += kDrawWaves) {
            const R4 us = s_us[k];
            const Normal4<Real> z = normals4<Real>((uint32_t)m, (uint32_t)k, s_solve, 0u, a.seed_lo, a.seed_hi);
            R4 u;
            u.x = clamp_finite(us.x + sig0 * z.z0, rlo, rhi);
            u.y = clamp_finite(us.y + sig1 * z.z1, rlo, rhi);
            u.z = clamp_finite(us.z + sig2 * z.z2, rlo, rhi);
            u.w = clamp_finite(us.w + sig3 * z.z3, rlo, rhi);
            Real V = Real(0);
            if (CONT) {
                const Real zv = normal1<Real>((uint32_t)m, (uint32_t)k, s_solve, 1u, a.seed_lo, a.seed_hi);
                V = clamp_finite(s_vs[k] + sigv * zv, dlo, dhi);
            }
            watch.wait<2>(k);
            s_r[k & (RI - 1)][lane] = u;
            if (CONT) s_v[k & (RI - 1)][lane] = V;
            pipe_publish(mine, k + kDrawWaves);
        }
    } else if (wave == 4) {
        // thrust chain, carried in binary64 in every precision (an
        // integrator: in binary32 its rounding over the horizon reaches the
        // attitude through the small inertia and the position through the attitude)
        double T[4];
        for (int i = 0; i < 4; ++i) T[i] = a.req[kReqThrust + i];
        const double inv_dt = 1.0 / a.dt, hh = 0.5 * a.dt, ddt = a.dt;
        const double t_min = a.t_min, t_max = a.t_max;
        R4 *rec = (R4 *)a.ctrl + m;
        const int reader = CONT ? PC_TERM : (TRACK ? PC_COST : PC_POS);
        const PipeWatch watch = {&s_cnt[lane < kDrawWaves ? PC_DRAW + lane : (lane & 1 ? PC_POS : reader)],
                                 lane < kDrawWaves ? 0 : RI};
        pipe_run<R4>(
            N, watch, counter(PC_CHAIN), [&](const int k, R4 &in) { in = s_r[k & (RI - 1)][lane]; },
            [&](const int k, const R4 &in, R4 &) {
                Real u[4] = {in.x, in.y, in.z, in.w}, tm[4], te[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // the clip to the range that keeps the thrust within its
                    // bounds over the step (multiplied by 1/dt: the bound can
                    // differ from the quotient in the last binary64 place)
                    u[i] = (Real)clamp_finite((double)u[i], (t_min - T[i]) * inv_dt, (t_max - T[i]) * inv_dt);
                    const double ur = (double)u[i];
                    tm[i] = (Real)(T[i] + hh * ur);
                    T[i] += ddt * ur;
                    te[i] = (Real)T[i];
                }
                R4 o;
                o.x = tm[0]; o.y = tm[1]; o.z = tm[2]; o.w = tm[3];
                s_T[k & (RI - 1)][0][lane] = o;
                o.x = te[0]; o.y = te[1]; o.z = te[2]; o.w = te[3];
                s_T[k & (RI - 1)][1][lane] = o;
                o.x = u[0]; o.y = u[1]; o.z = u[2]; o.w = u[3];
                if (!GATE) s_u[k & (RI - 1)][lane] = o;
                if (sampled) store_nt(rec, o);
                rec += K;
            });
    } else if (wave == 0) {
        // body rates
        const Model<Real> M(a);
        Real w[3];
        for (int i = 0; i < 3; ++i) w[i] = (Real)h.x0[10 + i];
        const double *const T0 = a.req + kReqThrust;
        StepInput<Real> in1 = step_input(M, (Real)T0[0], (Real)T0[1], (Real)T0[2], (Real)T0[3]);
        struct In { R4 tm, te; };
        const PipeWatch watch = {&s_cnt[lane == 0 ? PC_CHAIN : (lane & 1 ? PC_ATT : PC_COST)], lane == 0 ? 0 : RS};
        pipe_run<In>(
            N, watch, counter(PC_RATE),
            [&](const int k, In &in) {
                in.tm = s_T[k & (RI - 1)][0][lane];
                in.te = s_T[k & (RI - 1)][1][lane];
            },
            [&](const int k, const In &in, In &) {
                R4 (*slot)[64] = s_w[k & (RS - 1)];
                const StepInput<Real> in2 = step_input(M, in.tm.x, in.tm.y, in.tm.z, in.tm.w);
                const StepInput<Real> in4 = step_input(M, in.te.x, in.te.y, in.te.z, in.te.w);
                Real ws[3], kw[3], dw[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) ws[i] = w[i];
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const StepInput<Real> &si = st == 0 ? in1 : (st < 3 ? in2 : in4);
                    slot[st][lane].x = ws[0]; slot[st][lane].y = ws[1]; slot[st][lane].z = ws[2];
                    kw[0] = si.tx - M.gx * ws[1] * ws[2];
                    kw[1] = si.ty - M.gy * ws[2] * ws[0];
                    kw[2] = si.tz - M.gz * ws[0] * ws[1];
                    if (st == 0) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] = kw[i];
                    } else if (st < 3) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] += Real(2) * kw[i];
                    } else {
#pragma unroll
                        for (int i = 0; i < 3; ++i) dw[i] = dt6 * (dw[i] + kw[i]);
                    }
                    if (st < 3) {
                        const Real hs = st < 2 ? h2 : dt;
#pragma unroll
                        for (int i = 0; i < 3; ++i) ws[i] = w[i] + hs * kw[i];
                    }
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) w[i] += dw[i];
                // the thrusts at the end of a step are those at the start of the next
                in1 = in4;
            });
        // w_N, as the first stage of a step N
        const PipeWatch last = {&s_cnt[lane & 1 ? PC_ATT : PC_COST], RS};
        last.wait<0>(N);
        R4 *const o = s_w[N & (RS - 1)][0];
        o[lane].x = w[0]; o[lane].y = w[1]; o[lane].z = w[2];
        pipe_publish(counter(PC_RATE), N + 1);
    } else if (wave == 1) {
        // attitude
        Real q[4];
        for (int i = 0; i < 4; ++i) q[i] = (Real)h.x0[6 + i];
        struct In { R4 w[4]; };
        const PipeWatch watch = {&s_cnt[lane == 0 ? PC_RATE : (TRACK && (lane & 1) ? PC_COST : PC_POS)], lane == 0 ? 0 : RS};
        pipe_run<In>(
            N, watch, counter(PC_ATT),
            [&](const int k, In &in) {
#pragma unroll
                for (int st = 0; st < 4; ++st) in.w[st] = s_w[k & (RS - 1)][st][lane];
            },
            [&](const int k, const In &wst, In &) {
                R4 (*slot)[64] = s_q[k & (RS - 1)];
                Real qs[4], kq[4], dq[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) qs[i] = q[i];
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const R4 ws = wst.w[st];
                    R4 o;
                    o.x = qs[0]; o.y = qs[1]; o.z = qs[2]; o.w = qs[3];
                    slot[st][lane] = o;
                    // kq is twice the quaternion rate; the factor 1/2 is
                    // carried by the step sizes (exact: a power of two)
                    kq[0] = -qs[1] * ws.x - qs[2] * ws.y - qs[3] * ws.z;
                    kq[1] = qs[0] * ws.x + qs[2] * ws.z - qs[3] * ws.y;
                    kq[2] = qs[0] * ws.y - qs[1] * ws.z + qs[3] * ws.x;
                    kq[3] = qs[0] * ws.z + qs[1] * ws.y - qs[2] * ws.x;
                    if (st == 0) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) dq[i] = kq[i];
                    } else if (st < 3) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) dq[i] += Real(2) * kq[i];
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            dq[i] = dt12 * (dq[i] + kq[i]);
                            q[i] += dq[i];
                        }
                    }
                    if (st < 3) {
                        const Real hq = st < 2 ? h4 : h2;
#pragma unroll
                        for (int i = 0; i < 4; ++i) qs[i] = q[i] + hq * kq[i];
                    }
                }
                renormalize(q);
            });
        if (TRACK) {
            R4 o;
            o.x = q[0]; o.y = q[1]; o.z = q[2]; o.w = q[3];
            s_end[2][lane] = o;
        }
    } else if (wave == 2) {
        // position and velocity
        const Model<Real> M(a);
        Real p[3], v[3];
        for (int i = 0; i < 3; ++i) {
            p[i] = (Real)h.x0[i];
            v[i] = (Real)h.x0[3 + i];
        }
        const double *const T0 = a.req + kReqThrust;
        Real fm1 = step_input(M, (Real)T0[0], (Real)T0[1], (Real)T0[2], (Real)T0[3]).fm;
        struct In { R4 tm, te, q[4]; };
        const PipeWatch watch = {&s_cnt[lane == 0 ? PC_ATT : PC_COST], lane == 0 ? 0 : RS};
        auto pos_step = [&](const int k, const In &in, auto drag_tag) {
            constexpr bool DRAG = decltype(drag_tag)::value;
            const Real fm2 = step_input(M, in.tm.x, in.tm.y, in.tm.z, in.tm.w).fm;
            const Real fm4 = step_input(M, in.te.x, in.te.y, in.te.z, in.te.w).fm;
            Real vs[3], kv[3], dpv[3], dvv[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) vs[i] = v[i];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const Real q[4] = {in.q[st].x, in.q[st].y, in.q[st].z, in.q[st].w};
                stage_accel<DRAG>(M, st == 0 ? fm1 : (st < 3 ? fm2 : fm4), q, vs, kv);
                if (st == 0) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) { dpv[i] = vs[i]; dvv[i] = kv[i]; }
                } else if (st < 3) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) { dpv[i] += Real(2) * vs[i]; dvv[i] += Real(2) * kv[i]; }
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i) { dpv[i] = dt6 * (dpv[i] + vs[i]); dvv[i] = dt6 * (dvv[i] + kv[i]); }
                }
                if (st < 3) {
                    const Real hs = st < 2 ? h2 : dt;
#pragma unroll
                    for (int i = 0; i < 3; ++i) vs[i] = v[i] + hs * kv[i];
                }
            }
            R4 (*ps)[64] = s_p[k & (RS - 1)];
            ps[0][lane].x = p[0]; ps[0][lane].y = p[1]; ps[0][lane].z = p[2];
            if (!CONT) {
                const Real *const o2 = TRACK ? v : dpv;
                ps[CONT ? 0 : 1][lane].x = o2[0]; ps[CONT ? 0 : 1][lane].y = o2[1]; ps[CONT ? 0 : 1][lane].z = o2[2];
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                p[i] += dpv[i];
                v[i] += dvv[i];
            }
            fm1 = fm4;
        };
        auto load = [&](const int k, In &in) {
            in.tm = s_T[k & (RI - 1)][0][lane];
            in.te = s_T[k & (RI - 1)][1][lane];
#pragma unroll
            for (int st = 0; st < 4; ++st) in.q[st] = s_q[k & (RS - 1)][st][lane];
        };
        if (M.drag)
            pipe_run<In>(N, watch, counter(PC_POS), load,
                         [&](const int k, const In &in, In &) { pos_step(k, in, std::true_type{}); });
        else
            pipe_run<In>(N, watch, counter(PC_POS), load,
                         [&](const int k, const In &in, In &) { pos_step(k, in, std::false_type{}); });
        s_end[0][lane].x = p[0]; s_end[0][lane].y = p[1]; s_end[0][lane].z = p[2];
        s_end[1][lane].x = v[0]; s_end[1][lane].y = v[1]; s_end[1][lane].z = v[2];
    } else if (wave == 5 && CONT) {
        // the speed chain (binary64, as the thrusts), the path point and
        // tangent of every step, the input terms
        double vs = h.v_prev;
        const double inv_dt = 1.0 / a.dt, ddt = a.dt, hdt = 0.5 * a.dt, v_max = a.v_max;
        const Real rd0 = (Real)a.R_dT[0], rd1 = (Real)a.R_dT[1], rd2 = (Real)a.R_dT[2], rd3 = (Real)a.R_dT[3];
        const Real *path = (const Real *)a.path_r;
        Real *vrec = (Real *)a.vctrl + m;
        Real th_hi = (Real)h.theta0, th_lo = 0;
        if (sizeof(Real) == 4) th_lo = (Real)(h.theta0 - (double)th_hi);
        const Real L = (Real)a.path_len;
        const Real ds = (Real)(a.path_len / (double)a.P), inv_ds = (Real)((double)a.P / a.path_len);
        struct In { R4 u; Real V, f; R4 A0, A1, B0, B1; };
        auto rows = [&](In &in) {
            const Real fl = floor(th_hi * inv_ds);
            in.f = ((th_hi - fl * ds) + th_lo) * inv_ds;
            const int i = (fl >= Real(0) && fl < Real(1 << 30)) ? ((int)fl % a.P) : 0;
            const int i1 = (i + 1 == a.P) ? 0 : i + 1;
            const R4 *A = (const R4 *)(path + 8 * i), *B = (const R4 *)(path + 8 * i1);
            in.A0 = A[0]; in.A1 = A[1]; in.B0 = B[0]; in.B1 = B[1];
        };
        const PipeWatch watch = {&s_cnt[lane < kDrawWaves ? PC_DRAW + lane : (lane & 1 ? PC_CHAIN : PC_COST)],
                                 lane < kDrawWaves || (lane & 1) ? 0 : RS};
        pipe_run<In>(
            N, watch, counter(PC_TERM),
            [&](const int k, In &in) {
                in.u = s_u[k & (RI - 1)][lane];
                in.V = s_v[k & (RI - 1)][lane];
            },
            [&](const int k, const In &in, In &nxt) {
                const Real V = (Real)clamp_finite((double)in.V, (0.0 - vs) * inv_dt, (v_max - vs) * inv_dt);
                const Real speed = (Real)vs;
                {   // theta_{k+1}; its table rows are in flight while this step computes
                    const double vsn = vs + ddt * (double)V;
                    const Real adv = (Real)(hdt * (vs + vsn));
                    vs = vsn;
                    const Real y = adv + th_lo;
                    const Real t = th_hi + y;
                    th_lo = (sizeof(Real) == 4) ? y - (t - th_hi) : Real(0);
                    th_hi = t;
                    if (th_hi >= L) th_hi -= L;
                    rows(nxt);
                }
                if (sampled) store_nt(vrec, V);
                vrec += K;
                const R4 u = in.u;
                const Real ut = rd0 * u.x * u.x + rd1 * u.y * u.y + rd2 * u.z * u.z + rd3 * u.w * u.w;
                const Real f = in.f, g1 = Real(1) - f;
                const Real A[6] = {in.A0.x, in.A0.y, in.A0.z, in.A0.w, in.A1.x, in.A1.y};
                const Real B[6] = {in.B0.x, in.B0.y, in.B0.z, in.B0.w, in.B1.x, in.B1.y};
                const Real px = g1 * A[0] + f * B[0], py = g1 * A[1] + f * B[1], pz = g1 * A[2] + f * B[2];
                Real tx = g1 * A[3] + f * B[3], ty = g1 * A[4] + f * B[4], tz = g1 * A[5] + f * B[5];
                const Real tn = inv_sqrt(tx * tx + ty * ty + tz * tz);
                tx *= tn; ty *= tn; tz *= tn;
                R4 (*o)[64] = s_t[k & (RS - 1)];
                R4 c;
                c.x = px; c.y = py; c.z = pz; c.w = ut;
                o[0][lane] = c;
                c.x = tx; c.y = ty; c.z = tz; c.w = V;
                o[1][lane] = c;
                o[2][lane].x = speed;
            },
            rows);
    } else {
        // costs, all terms of a step in one sum
        KSum<Real> J;
        const Real w_max = (Real)a.w_max, w_lim = (Real)a.w_lim;
        R4 w;
        w.x = (Real)h.x0[10]; w.y = (Real)h.x0[11]; w.z = (Real)h.x0[12];
        auto rate_limit = [&](Real &term, const R4 &wn) {
            const Real ww[3] = {wn.x, wn.y, wn.z};
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const Real e = fmax(fabs(ww[i]) - w_max, Real(0));
                term += w_lim * e * e;
            }
        };
        GateRegs<Real> g0r;
        if constexpr (GATE) {
            const Real q_near = (Real)a.q_near, r_near2 = (Real)(a.r_near * a.r_near), half = (Real)a.gate_half;
            GateRegs<Real> gt;
            int g = h.g0, passes = 0;
            gt.load(s_gtab, g);
            g0r = gt;
            struct In { R4 p, d, w; };
            const PipeWatch watch = {&s_cnt[lane == 0 ? PC_RATE : PC_POS], lane == 0 ? -1 : 0};
            pipe_run<In>(
                N, watch, counter(PC_COST),
                [&](const int k, In &in) {
                    in.p = s_p[k & (RS - 1)][0][lane];
                    in.d = s_p[k & (RS - 1)][CONT ? 0 : 1][lane];
                    in.w = s_w[(k + 1) & (RS - 1)][0][lane];
                },
                [&](const int k, const In &in, In &) {
                    Real term = Real(0);
                    const Real dx[3] = {in.d.x, in.d.y, in.d.z};
                    const Real ax = in.p.x - gt.cx;
                    const Real ay = in.p.y - gt.cy;
                    const Real az = in.p.z - gt.cz;
                    const Real bx = in.p.x - g0r.cx;
                    const Real by = in.p.y - g0r.cy;
                    const Real bz = in.p.z - g0r.cz;
                    const Real d2 = bx * bx + by * by + bz * bz;
                    if (d2 < r_near2) term += q_near * d2;  // Eq. (7), current gate
                    if (nominal) s_f8[k] = (bx * g0r.nx + by * g0r.ny) < Real(0);
                    // |p_{k+1} - c|^2 - |p_k - c|^2 = dp . (2 (p_k - c) + dp)
                    term += dx[0] * (Real(2) * ax + dx[0]) + dx[1] * (Real(2) * ay + dx[1]) +
                            dx[2] * (Real(2) * az + dx[2]);
                    const Real sa = ax * gt.nx + ay * gt.ny;
                    const Real sb = (ax + dx[0]) * gt.nx + (ay + dx[1]) * gt.ny;
                    if (sa < Real(0) && sb >= Real(0)) {
                        const Real t = sa / (sa - sb);
                        const Real yx = ax + t * dx[0], yy = ay + t * dx[1], yz = az + t * dx[2];
                        const Real lat = yx * gt.hx + yy * gt.hy;
                        const bool inside = fabs(lat) <= half && fabs(yz) <= half;
                        const int j = k + 1;
                        const bool allowed = passes > 0 || ((h.allow[j >> 5] >> (j & 31)) & 1u);
                        if (inside && allowed) {
                            g = (g + 1 == a.G) ? 0 : g + 1;
                            ++passes;
                            gt.load(s_gtab, g);
                        }
                    }
                    rate_limit(term, in.w);
                    J.add(term);
                });
        } else if constexpr (TRACK) {
            const Real *xref = (const Real *)a.xref_r;
            const int i0 = h.i0;
            auto ref_row = [&](const int k) {
                int r = i0 + k;
                if (r > a.R - 1) r = a.R - 1;
                return xref + 16 * r;
            };
            struct In { R4 p, v, q, w, u; Real x[13]; };
            const PipeWatch watch = {&s_cnt[lane == 0 ? PC_RATE : PC_POS], lane == 0 ? -1 : 0};
            pipe_run<In>(
                N, watch, counter(PC_COST),
                [&](const int k, In &in) {
                    in.p = s_p[k & (RS - 1)][0][lane];
                    in.v = s_p[k & (RS - 1)][CONT ? 0 : 1][lane];
                    in.q = s_q[k & (RS - 1)][0][lane];
                    in.w = s_w[(k + 1) & (RS - 1)][0][lane];
                    in.u = s_u[k & (RI - 1)][lane];
                    const Real *xr = ref_row(k);
#pragma unroll
                    for (int i = 0; i < 13; ++i) in.x[i] = xr[i];
                },
                [&](const int, const In &in, In &) {
                    const Real x[13] = {in.p.x, in.p.y, in.p.z, in.v.x, in.v.y, in.v.z, in.q.x,
                                        in.q.y, in.q.z, in.q.w, w.x,    w.y,    w.z};
                    Real term = Real(0);
#pragma unroll
                    for (int i = 0; i < 13; ++i) {
                        const Real e = x[i] - in.x[i];
                        term += (Real)a.Q[i] * e * e;
                    }
                    const R4 u = in.u;
                    term += (Real)a.R_dT[0] * u.x * u.x + (Real)a.R_dT[1] * u.y * u.y + (Real)a.R_dT[2] * u.z * u.z +
                            (Real)a.R_dT[3] * u.w * u.w;
                    rate_limit(term, in.w);
                    J.add(term);
                    w = in.w;
                });
        } else {
            const Real q_l = (Real)a.q_l, q_c = (Real)a.q_c, r_dv = (Real)a.r_dv, mu = (Real)a.mu;
            const Real qw0 = (Real)a.Q_w[0], qw1 = (Real)a.Q_w[1], qw2 = (Real)a.Q_w[2];
            struct In { R4 p, c, t, w; Real vs; };
            const PipeWatch watch = {&s_cnt[lane == 0 ? PC_RATE : (lane & 1 ? PC_POS : PC_TERM)], lane == 0 ? -1 : 0};
            pipe_run<In>(
                N, watch, counter(PC_COST),
                [&](const int k, In &in) {
                    in.p = s_p[k & (RS - 1)][0][lane];
                    in.c = s_t[k & (RS - 1)][0][lane];
                    in.t = s_t[k & (RS - 1)][1][lane];
                    in.vs = s_t[k & (RS - 1)][2][lane].x;
                    in.w = s_w[(k + 1) & (RS - 1)][0][lane];
                },
                [&](const int, const In &in, In &) {
                    Real term = Real(0);
                    const Real tx = in.t.x, ty = in.t.y, tz = in.t.z, V = in.t.w;
                    const Real ex = in.p.x - in.c.x;
                    const Real ey = in.p.y - in.c.y;
                    const Real ez = in.p.z - in.c.z;
                    const Real et = ex * tx + ey * ty + ez * tz;
                    const Real lx = et * tx, ly = et * ty, lz = et * tz;
                    const Real cxe = ex - lx, cye = ey - ly, cze = ez - lz;
                    term += q_l * (lx * lx + ly * ly + lz * lz);
                    term += q_c * (cxe * cxe + cye * cye + cze * cze);
                    term += qw0 * w.x * w.x + qw1 * w.y * w.y + qw2 * w.z * w.z;
                    term += r_dv * V * V;
                    term += in.c.w;
                    term -= mu * in.vs;
                    rate_limit(term, in.w);
                    J.add(term);
                    w = in.w;
                });
        }
        __syncthreads();
        if (TRACK) {
            int r = h.i0 + N;
            if (r > a.R - 1) r = a.R - 1;
            const Real *xr = (const Real *)a.xref_r + 16 * r;
            const R4 pN = s_end[0][lane], vN = s_end[1][lane], qN = s_end[2][lane];
            const Real x[13] = {pN.x, pN.y, pN.z, vN.x, vN.y, vN.z, qN.x, qN.y, qN.z, qN.w, w.x, w.y, w.z};
            Real term = 0;
#pragma unroll
            for (int i = 0; i < 13; ++i) {
                const Real e = x[i] - xr[i];
                term += (Real)a.QN[i] * e * e;
            }
            J.add(term);
        }
        if (GATE && nominal) {
            const R4 ph = s_end[0][lane];
            const Real bx = ph.x - g0r.cx;
            const Real by = ph.y - g0r.cy;
            a.front8[N] = (bx * g0r.nx + by * g0r.ny) < Real(0);
        }
        if (GATE && blk == (K >> 6))
            for (int i = lane; i < N; i += 64) a.front8[i] = s_f8[i];
        Real Jfinal = Real(0);
        if (active) {
            Jfinal = J.value();
            if (nominal) a.cur->J_nom = (double)Jfinal;
            else ((Real *)a.J)[m] = Jfinal;
        }
        store_tile_min(Jfinal, active && !nominal && isfinite(Jfinal), a.tmin, blk);
    }
    if (wave != 3) __syncthreads();     // (the cost wave meets the others above)
}

template <int OBJ, typename Real, int R>
__global__ __launch_bounds__(64 * rate_pipe_waves(OBJ)) void k_rollout_rate(KArgs a)
{
    __shared__ HeadVals h;
    compute_head<OBJ == OBJ_CONTOUR>(a, h);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish_head(a, h);
    rollout_rate_body<OBJ, Real, R>(a, blockIdx.x, h);
}

template <int OBJ, typename Real> __global__ __launch_bounds__(192) void k_rollout3(KArgs a)
{
    __shared__ HeadVals h;
    compute_head<OBJ == OBJ_CONTOUR>(a, h);
    if (blockIdx.x == 0 && threadIdx.x == 0) publish_head(a, h);
    rollout3_body<OBJ, Real>(a, blockIdx.x, h);
}

// ---------------------------------------------------------------- control cost

// The control-cost term of information-theoretic MPPI added to every sample's
// cost: gamma * sum_k sum_i U*_k,i (U^m_k,i - U*_k,i) / sigma_i^2 over the
// channels with sigma_i > 0 (thrusts, then the contouring speed), U* the
// shifted warm start of the solve and U^m the stored clipped sample, summed in
// step order.  One wave per 64-sample tile reads its samples step by step
// (64 consecutive records per step) and rewrites the tile's smallest finite
// cost.
template <typename Real, bool HAS_V> __device__ __forceinline__ void ctrl_cost_body(const KArgs &a, int tile)
{
    typedef typename Vec4<Real>::T R4;
    const int m = tile * 64 + (int)threadIdx.x;
    const int K = a.K, N = a.N;
    const DevCur *cur = a.cur;
    const int shift = cur->shift;
    const bool warm = cur->warm != 0;
    const Real gam = (Real)a.ctrl_cost, hover = (Real)a.hover;
    const Real is0 = (Real)a.inv_sig2[0], is1 = (Real)a.inv_sig2[1], is2 = (Real)a.inv_sig2[2];
    const Real is3 = (Real)a.inv_sig2[3], isv = (Real)a.inv_sig2[4];
    Real Jm = Real(INFINITY);
    if (m < K) {
        const R4 *ctrl = (const R4 *)a.ctrl;
        const Real *vctrl = (const Real *)a.vctrl;
        Real C = Real(0);
        for (int k = 0; k < N; ++k) {
            const int src = k + shift < N ? k + shift : N - 1;
            const Real u0 = warm ? (Real)a.wU[4 * src + 0] : hover, u1 = warm ? (Real)a.wU[4 * src + 1] : hover;
            const Real u2 = warm ? (Real)a.wU[4 * src + 2] : hover, u3 = warm ? (Real)a.wU[4 * src + 3] : hover;
            const R4 u = ctrl[(size_t)k * (size_t)K + (size_t)m];
            C += gam * u0 * (u.x - u0) * is0;
            C += gam * u1 * (u.y - u1) * is1;
            C += gam * u2 * (u.z - u2) * is2;
            C += gam * u3 * (u.w - u3) * is3;
            if (HAS_V) {
                const Real vs = warm ? (Real)a.wV[src] : Real(0);
                C += gam * vs * (vctrl[(size_t)k * (size_t)K + (size_t)m] - vs) * isv;
            }
        }
        Jm = ((Real *)a.J)[m] + C;
        ((Real *)a.J)[m] = Jm;
    }
    store_tile_min(Jm, m < K && isfinite(Jm), a.tmin, tile);
}

template <typename Real, bool HAS_V> __global__ __launch_bounds__(64) void k_ctrl_cost(KArgs a)
{
    ctrl_cost_body<Real, HAS_V>(a, blockIdx.x);
}

// ---------------------------------------------------------------- weighted average

// Sum over the 64 lanes of a wave (all lanes active) by a fixed tree,
// returned to every lane: binary32 through the DPP moves of wave_min (a lane
// without a source adds 0; lane 63 ends with the sum), binary64 through lane
// shuffles.
template <int CTRL, int ROW_MASK = 0xf> __device__ __forceinline__ float dpp_or_zero(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}

__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_or_zero<0xb1>(v);
    v += dpp_or_zero<0x4e>(v);
    v += dpp_or_zero<0x114>(v);
    v += dpp_or_zero<0x118>(v);
    v += dpp_or_zero<0x142, 0xa>(v);
    v += dpp_or_zero<0x143, 0xc>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ __forceinline__ double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Eq. (4)-(5) for step k in one block of kFinalThreads threads:
//   J_min = min over the tile minima (each wave reduces them all),  w~_m = exp(-(J_m - J_min)/lambda)
//   (0 for non-finite J_m),  S = sum_m w~_m,  U_k = sum_m w~_m U^m_k / S.
// Thread t adds the samples t, t + kFinalThreads, ... in that order.  The
// thread sums go to LDS; lane l of wave i then adds value i of threads l,
// l + 64, ..., l + kFinalThreads - 64 in that order and the lanes are added
// by the fixed tree of wave_sum, one value per wave, all values at once.  S
// and sum_m w~_m^2 come out of the same loop in every block, bit for bit, so
// no block waits for another.  The block of step 0 also writes the first
// input, the report, the nominal's pass mask for the next solve and the
// warm-start hand-over.  The samples are loaded first, then the tile minima,
// so that one wait covers all of them.
//
// REGEN: the samples are not read from the sample tensor (which the rollout
// then does not write) but drawn again from the counter-based noise of this
// solve and the shifted warm start of step k that the rollout left in nomU /
// nomV, with the same operations as the rollout's draw, so the weighted sums
// are the same bit for bit: Philox and Box-Muller arithmetic in place of
// 16 B (20 B contouring) of HBM traffic per sample and step.
//
// SKIP: the weights of a round are formed before its samples are read, and a
// sample whose weight is exactly 0 (a cost more than kWeightCut temperatures
// above J_min) is neither read nor drawn: it adds nothing to any sum, so the
// result is the same bit for bit.  With sharp weights (lambda = 1 at the
// benchmark's noise) almost no sample is read: K = 262144, N = 200, binary64
// sums: 157 -> 48 us.  Used wherever a thread has several rounds of samples
// (where a part of them weighs something it costs a little: rate input,
// K = 33000, N = 20 37.7 -> 39 us a solve; reading all costs up to 18 us more
// there with sharp weights); with one round the samples are loaded at once
// with the costs, which saves a round trip to memory.
// A round is final_loads samples a thread (binary64: four spill, K = 8192,
// N = 100: 59.3 us a solve against 54.2).
template <typename Real> constexpr int final_loads = sizeof(Real) == 8 ? 2 : 4;
// A block of whose first round at least one sample in sixteen weighs something
// (the samples of a solve are alike, so all blocks find the same) reads all its
// samples: the conditional loads of skipping are waited for one by one.
// Binary32 samples with binary64 sums, skipping -> reading all: contouring with
// all weights alive K = 131072, N = 20 111 -> 98 us a solve, K = 500000
// 330 -> 279 (107 and 310 before samples were skipped); gate, one in ten
// alive, K = 500000 249 -> 240.  Fewer samples (binary32 sums) and binary64
// samples lose nothing worth it by skipping.
constexpr int kDenseLanes = 4;
template <typename Real> constexpr Real kWeightCut = sizeof(Real) == 4 ? Real(105) : Real(750);

// S: horizon steps k .. k + S - 1 in one block.  The weights depend on the
// costs only, so a block of several steps forms them once: batches, whose
// average otherwise spends itself on them (256 uneven instances, lambda = 1:
// 457 -> 218 us), give each block final_steps() of them.
template <typename Acc, bool HAS_V, int S> struct FinalLds {
    static constexpr int NV = S * (HAS_V ? 5 : 4) + 2;  // step s: values s C ..; then the two weight sums
    Acc part[NV][kFinalThreads], tot[NV];
};

template <typename Real, typename Acc, bool HAS_V, bool REGEN, int UR = 4, bool SKIP = false, int S = 1>
__device__ __forceinline__ void final_body(const KArgs &a, int k, FinalLds<Acc, HAS_V, S> &lds)
{
    constexpr int C = HAS_V ? 5 : 4;
    constexpr int NV = FinalLds<Acc, HAS_V, S>::NV;
    constexpr int NT = kFinalThreads, NWV = NT / 64;
    typedef typename Vec4<Real>::T R4;
    static_assert(SKIP || S == 1, "several steps share the weights of a round");
    constexpr bool DENSE = SKIP && !REGEN && sizeof(Real) < sizeof(Acc);
    __shared__ int s_live[DENSE ? NWV : 1];
    auto &s_part = lds.part;
    auto &s_tot = lds.tot;

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int K = a.K, N = a.N;
    const Real *J = (const Real *)a.J;
    const R4 *ctrl = (const R4 *)a.ctrl + (size_t)k * (size_t)K;
    const Real *vctrl = HAS_V ? (const Real *)a.vctrl + (size_t)k * (size_t)K : nullptr;
    const Real inv_lambda = (Real)(1.0 / a.lambda);
    DevCur *cur = a.cur;
    DevWarm *w = a.warm;
    const bool head = k == 0;
    const bool gate = a.objective == OBJ_GATE;
    // regenerated draws: the shifted warm start of step k and the noise key
    const int ns = S == 1 ? 1 : min(S, N - k);
    R4 us[S] = {};
    Real vs[S] = {};
    uint32_t s_solve = 0;
    if (REGEN) {
        for (int s = 0; s < S; ++s) {
            if (s >= ns) break;
            us[s] = ((const R4 *)a.nomU)[k + s];
            if (HAS_V) vs[s] = ((const Real *)a.nomV)[k + s];
        }
        s_solve = cur->s;
    }
    const Real tmin = (Real)a.t_min, tmax = (Real)a.t_max, vmax = (Real)a.v_max;
    const Real sig0 = (Real)a.sigma[0], sig1 = (Real)a.sigma[1], sig2 = (Real)a.sigma[2], sig3 = (Real)a.sigma[3];
    const Real sigv = (Real)a.sigma_v;
    auto redraw = [&](const int m, const int st, R4 &u, Real &V) {
        const Normal4<Real> z = normals4<Real>((uint32_t)m, (uint32_t)(k + st), s_solve, 0u, a.seed_lo, a.seed_hi);
        u.x = clamp_finite(us[st].x + sig0 * z.z0, tmin, tmax);
        u.y = clamp_finite(us[st].y + sig1 * z.z1, tmin, tmax);
        u.z = clamp_finite(us[st].z + sig2 * z.z2, tmin, tmax);
        u.w = clamp_finite(us[st].w + sig3 * z.z3, tmin, tmax);
        if (HAS_V) {
            const Real zv = normal1<Real>((uint32_t)m, (uint32_t)(k + st), s_solve, 1u, a.seed_lo, a.seed_hi);
            V = clamp_finite(vs[st] + sigv * zv, Real(0), vmax);
        }
    };

    // loads: the first UR samples of this thread, then the tile minima (every
    // wave reads all of them), four per lane before the first comparison, so
    // that one round trip to memory covers all of them
    Real Jm[UR], vm[UR];
    R4 u[UR];
#pragma unroll
    for (int i = 0; i < UR; ++i) {
        const int m = tid + NT * i;
        if (SKIP) Jm[i] = Real(INFINITY);
        if (m < K) {
            Jm[i] = J[m];
            if (!REGEN && !SKIP) {
                u[i] = ctrl[m];
                if (HAS_V) vm[i] = vctrl[m];
            }
        }
    }
    Real mn = Real(INFINITY);
    for (int t0 = lane; t0 < a.n_tiles; t0 += 4 * 64) {
        Real tv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = t0 + 64 * j;
            tv[j] = t < a.n_tiles ? ((const Real *)a.tmin)[t] : Real(INFINITY);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) mn = tv[j] < mn ? tv[j] : mn;
    }
    // head values for the report and the hand-over (block of step 0)
    const bool fr = head && gate && tid <= N && tid < 256 && a.front8[tid] != 0;
    const bool fr_last = head && gate && tid == 0 && N >= 256 && a.front8[256] != 0;
    // (spread over the lanes of wave 0: lane 5 the report's head fields,
    // lane 6 the warm-start fields, lanes 7..19 one state component each)
    double rep_Jnom = 0.0, rep_theta0 = 0.0, rep_t = 0.0, rep_x = 0.0, rep_v = 0.0;
    int32_t rep_g0 = 0, rep_i0 = 0, rep_shift = 0;
    uint32_t rep_s = 0;
    if (head && (tid == 5 || tid == 6)) {
        rep_Jnom = cur->J_nom;
        rep_theta0 = cur->theta0;
        rep_t = cur->t_now;
        rep_g0 = cur->g0;
        rep_i0 = cur->i0;
        rep_shift = cur->shift;
        rep_s = cur->s;
        rep_v = cur->v_prev;
    }
    if (head && tid >= 7 && tid < 20) rep_x = cur->x0[tid - 7];
    // J_min within each wave (a minimum does not depend on the grouping, so
    // every wave of every block finds the same value without a block barrier)
    const Real jmin = wave_min(mn);

    // weighted sums, UR samples per round in sample order; the next round's
    // loads are issued before this round's arithmetic
    Acc v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = Acc(0);
    if constexpr (SKIP) {
        // the weights of a round of samples; the samples of one step of it,
        // of the lanes that weigh something (the others 0)
        struct Weights { Real w[UR]; bool any[UR], live[UR]; };
        struct Samples { R4 u[UR]; Real v[UR]; };
        auto costs = [&](const int m0, Real *Jr) {
#pragma unroll
            for (int i = 0; i < UR; ++i) {
                const int m = m0 + NT * i;
                Jr[i] = Real(INFINITY);
                if (m < K) Jr[i] = J[m];
            }
        };
        // which samples of a round weigh something; their weights are formed
        // with the fetch of the first step, while its samples are on their way
        auto sort_out = [&](const Real *Jr, Weights &r) {
#pragma unroll
            for (int i = 0; i < UR; ++i) {
                r.w[i] = -(Jr[i] - jmin) * inv_lambda;
                r.live[i] = isfinite(Jr[i]) && r.w[i] > -kWeightCut<Real>;
                r.any[i] = __builtin_amdgcn_ballot_w64(r.live[i]) != 0;
            }
        };
        auto fetch = [&](const int m0, const int st, Weights &r, Samples &x) {
#pragma unroll
            for (int i = 0; i < UR; ++i) {
                const int m = m0 + NT * i;
                const Real arg = r.w[i];
                if (st == 0) r.w[i] = Real(0);
                x.u[i] = R4{};
                x.v[i] = Real(0);
                if (r.any[i] && st < ns) {
                    if (r.live[i]) {
                        if (REGEN) {
                            redraw(m, st, x.u[i], x.v[i]);
                        } else {
                            x.u[i] = ctrl[(size_t)st * (size_t)K + (size_t)m];
                            if (HAS_V) x.v[i] = vctrl[(size_t)st * (size_t)K + (size_t)m];
                        }
                        if (st == 0) r.w[i] = exp(arg);
                    }
                }
            }
        };
        auto sum = [&](const int st, const Weights &r, const Samples &x) {
#pragma unroll
            for (int i = 0; i < UR; ++i) {
                if (r.any[i]) {
                    const Acc wa = (Acc)r.w[i];
                    Acc *const vv = v + st * C;
                    vv[0] += wa * (Acc)x.u[i].x;
                    vv[1] += wa * (Acc)x.u[i].y;
                    vv[2] += wa * (Acc)x.u[i].z;
                    vv[3] += wa * (Acc)x.u[i].w;
                    if (HAS_V) vv[C - 1] += wa * (Acc)x.v[i];
                    if (st == 0) {
                        v[S * C] += wa;
                        v[S * C + 1] += wa * wa;
                    }
                }
            }
        };
        // All samples, two a round: no load depends on a weight, so
        // the next round's are in flight while this one is summed.
        auto dense_rounds = [&] {
            constexpr int D = 2;
            struct Round { R4 u[D]; Real v[D]; };
            auto load_costs = [&](const int m0, Real *Jr) {
#pragma unroll
                for (int i = 0; i < D; ++i) Jr[i] = J[min(m0 + NT * i, K - 1)];
            };
            auto weigh = [&](const int m0, Real *Jr) {
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    const Real wr = exp(-(Jr[i] - jmin) * inv_lambda);
                    Jr[i] = m0 + NT * i < K && isfinite(Jr[i]) ? wr : Real(0);
                }
            };
            auto load = [&](const int m0, Round &r) {
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    const int m = min(m0 + NT * i, K - 1);
                    r.u[i] = ctrl[m];
                    if (HAS_V) r.v[i] = vctrl[m];
                }
            };
            auto add = [&](const Real *wr, const Round &r) {
#pragma unroll
                for (int i = 0; i < D; ++i) {
                    const Acc wa = (Acc)wr[i];
                    v[0] += wa * (Acc)r.u[i].x;
                    v[1] += wa * (Acc)r.u[i].y;
                    v[2] += wa * (Acc)r.u[i].z;
                    v[3] += wa * (Acc)r.u[i].w;
                    if (HAS_V) v[C - 1] += wa * (Acc)r.v[i];
                    v[C] += wa;
                    v[C + 1] += wa * wa;
                }
            };
            constexpr int step = NT * D;
            Real w0[D], w1[D];
            Round r0, r1;
            load_costs(tid, w0);
            load_costs(tid + step, w1);
            load(tid, r0);
            for (int r = 0; r < K; r += 2 * step) {     // (the same for every thread)
                const int m0 = tid + r, m1 = m0 + step, m2 = m1 + step;
                weigh(m0, w0);
                load(m1, r1);
                add(w0, r0);
                load_costs(m2, w0);
                weigh(m1, w1);
                load(m2, r0);
                add(w1, r1);
                load_costs(m2 + step, w1);
            }
        };
        // the costs two rounds ahead, the samples one step or round ahead of
        // the sums; two rounds unrolled so that both buffers stay in registers
        Weights wa, wb;
        Samples x[2];
        Real Jb[UR];
        const int step = NT * UR;
        const int rounds = (K + step - 1) / step;   // the same for every thread
        costs(tid + step, Jb);
        sort_out(Jm, wa);
        bool dense = false;
        if constexpr (DENSE) {
            int n_live = 0;
#pragma unroll
            for (int i = 0; i < UR; ++i) n_live += __builtin_popcountll(__builtin_amdgcn_ballot_w64(wa.live[i]));
            if (lane == 0) s_live[wv] = n_live;
            __syncthreads();
            n_live = 0;
#pragma unroll
            for (int i = 0; i < NWV; ++i) n_live += s_live[i];
            dense = n_live >= kDenseLanes * UR * NWV;
            if (dense) dense_rounds();
        }
        if (!dense) fetch(tid, 0, wa, x[0]);
        for (int r = 0; r < rounds && !dense; r += 2) {
            const int m0 = tid + r * step, m1 = m0 + step, m2 = m1 + step;
            costs(m2, Jm);
#pragma unroll
            for (int st = 0; st < S; ++st) {
                if (st + 1 < S) fetch(m0, st + 1, wa, x[(st + 1) & 1]);
                else { sort_out(Jb, wb); fetch(m1, 0, wb, x[S & 1]); }
                sum(st, wa, x[st & 1]);
            }
            costs(m2 + step, Jb);
#pragma unroll
            for (int st = 0; st < S; ++st) {
                if (st + 1 < S) fetch(m1, st + 1, wb, x[(S + st + 1) & 1]);
                else { sort_out(Jm, wa); fetch(m2, 0, wa, x[0]); }
                sum(st, wb, x[(S + st) & 1]);
            }
        }
    } else
    for (int m0 = tid; m0 < K; m0 += NT * UR) {
        Real Jn[UR], vn[UR];
        R4 un[UR];
        const int m1 = m0 + NT * UR;
        if (m1 < K) {
#pragma unroll
            for (int i = 0; i < UR; ++i) {
                const int m = m1 + NT * i;
                if (m < K) {
                    Jn[i] = J[m];
                    if (!REGEN) {
                        un[i] = ctrl[m];
                        if (HAS_V) vn[i] = vctrl[m];
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < UR; ++i) {
            if (m0 + NT * i < K) {
                if (REGEN) redraw(m0 + NT * i, 0, u[i], vm[i]);
                const Real wr = isfinite(Jm[i]) ? exp(-(Jm[i] - jmin) * inv_lambda) : Real(0);
                const Acc wa = (Acc)wr;
                v[0] += wa * (Acc)u[i].x;
                v[1] += wa * (Acc)u[i].y;
                v[2] += wa * (Acc)u[i].z;
                v[3] += wa * (Acc)u[i].w;
                if (HAS_V) v[4] += wa * (Acc)vm[i];
                v[C] += wa;
                v[C + 1] += wa * wa;
            }
        }
        if (m1 < K) {
#pragma unroll
            for (int i = 0; i < UR; ++i) {
                Jm[i] = Jn[i];
                if (!REGEN) {
                    u[i] = un[i];
                    if (HAS_V) vm[i] = vn[i];
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) s_part[i][tid] = v[i];
    __syncthreads();
    for (int i = wv; i < NV; i += NWV) {
        Acc t = s_part[i][lane];
#pragma unroll
        for (int j = 1; j < NWV; ++j) t += s_part[i][64 * j + lane];
        t = wave_sum(t);
        if (lane == 0) s_tot[i] = t;
    }
    __syncthreads();
    const Acc den = s_tot[S * C], den2 = s_tot[S * C + 1];
    const bool ok = isfinite(jmin) && den > Acc(0);
    if (ok && tid < C * ns) {
        const double uk = (double)(s_tot[tid] / den);
        const int st = tid / C, c = tid % C;
        if (c < 4) {
            a.wU[4 * (k + st) + c] = uk;
            if (a.U_host) a.U_host[4 * (k + st) + c] = uk;
        } else {
            a.wV[k + st] = uk;
        }
    }
    if (!HAS_V && ok && tid < ns) a.wV[k + tid] = 0.0;
    if (!head) return;

    // pass mask of the next solve: bit j = front flag of the nominal at step j
    if (gate) {
        if (tid < 256) {
            const unsigned long long bal = __ballot(fr);
            if ((tid & 63) == 0 && ok) {
                w->allow[tid >> 5] = (uint32_t)bal;
                w->allow[(tid >> 5) + 1] = (uint32_t)(bal >> 32);
            }
        }
        if (tid == 0 && ok) w->allow[8] = fr_last ? 1u : 0u;
    } else if (tid < kMaskWords && ok) {
        w->allow[tid] = 0xffffffffu;
    }
    // the report and the warm-start hand-over, one group of fields per lane
    auto report = [&](DevResult *r) {
        if (tid < 4) {
            r->u0[tid] = ok ? (double)(s_tot[tid] / den) : (double)NAN;
        } else if (tid == 4) {
            r->J_min = (double)jmin;
            r->S = (double)den;
            r->S2 = (double)den2;
            r->ess = ok ? (double)den * (double)den / (double)den2 : 0.0;
        } else if (tid == 5) {
            r->J_nom = rep_Jnom;
            r->theta0 = rep_theta0;
            r->status = ok ? ST_OK : ST_NONFINITE;
            r->g0 = rep_g0;
            r->i0 = rep_i0;
            r->shift = rep_shift;
            r->s = rep_s;
        }
    };
    report(a.res);
    if (a.res_host) report(a.res_host);
    if (tid < 4) {
        if (a.u0_out) a.u0_out[tid] = ok ? (double)(s_tot[tid] / den) : (double)NAN;
    } else if (tid == 6 && ok) {
        w->warm = 1;
        w->g0 = rep_g0;
        w->s = rep_s + 1u;
        w->N = N;
        w->t_prev = rep_t;
        w->theta0 = rep_theta0;
        // rate model: the progress speed state of this solve
        w->vtheta = a.input_model == INPUT_RATE ? rep_v : 0.0;
    } else if (tid >= 7 && tid < 20 && ok) {
        w->x_prev[tid - 7] = rep_x;
    }
}

template <typename Real, typename Acc, bool HAS_V, bool REGEN, int UR, bool SKIP>
__global__ __launch_bounds__(kFinalThreads) void k_final(KArgs a)
{
    __shared__ FinalLds<Acc, HAS_V, 1> lds;
    final_body<Real, Acc, HAS_V, REGEN, UR, SKIP>(a, blockIdx.x, lds);
}

// ---------------------------------------------------------------- batched (persistent)

// The item of unit u: the largest i in [0, n) with prefix[i] <= u (prefix[0]
// = 0, prefix[n] = total).  Every persistent kernel takes its units in
// increasing order, so the item only moves forward from the block's previous
// one: usually one load per unit instead of a binary search.
__device__ __forceinline__ int advance_item(const int32_t *prefix, int n, int u, int item)
{
    while (item + 1 < n && prefix[item + 1] <= u) ++item;
    return item;
}

// Stage the kernel arguments of an item's context in LDS, with the item's
// request and output pointers.
__device__ __forceinline__ void stage_args(StagedArgs &s_a, int &s_ctx, const BArgs &b, int item)
{
    const BatchItem it = b.items[item];
    if (it.ctx != s_ctx) {
        const uint32_t *src = (const uint32_t *)(b.table + it.ctx);
        uint32_t *dst = (uint32_t *)&s_a;
        for (int t = threadIdx.x; t < (int)(sizeof(KArgs) / 4); t += blockDim.x) dst[t] = src[t];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        s_a.req = it.req;
        s_a.u0_out = it.u0_out;
        if (it.ws) {
            const WsLayout l = ws_layout(s_a.K, s_a.N, s_a.C, s_a.real_bytes);
            s_a.ctrl = it.ws + l.ctrl;
            s_a.vctrl = s_a.C == 5 ? it.ws + l.vctrl : nullptr;
            s_a.nomU = it.ws + l.nomU;
            s_a.nomV = it.ws + l.nomV;
            s_a.J = it.ws + l.J;
            s_a.tmin = it.ws + l.tmin;
            s_a.front8 = (uint8_t *)(it.ws + l.front8);
        }
        // a workspace is bound per item: restage the next item in any case
        s_ctx = it.ws ? -1 : it.ctx;
    }
    __syncthreads();
}

// One unit per (item, block of 256 samples), all steps of the item; units
// are taken from a device queue in order (longest horizons first).
template <typename Real, bool HAS_V> __global__ __launch_bounds__(256) void kb_sample(BArgs b)
{
    __shared__ StagedArgs s_a;
    __shared__ int s_ctx, s_unit;
    if (threadIdx.x == 0) s_ctx = -1;
    if (blockIdx.x == 0 && threadIdx.x == 0) b.desc->queue = 0u;
    const int n = b.desc->n, total = b.desc->n_sample_units;
    int item = 0;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_unit = (int)atomicAdd(&b.desc->sample_queue, 1u);
        __syncthreads();
        const int u = s_unit;
        if (u >= total) break;
        item = advance_item(b.sample_prefix, n, u, item);
        stage_args(s_a, s_ctx, b, item);
        sample_body<Real, HAS_V>(s_a, u - b.sample_prefix[item], 0, s_a.N);
    }
}

template <int OBJ, typename Real, int WAVES> __global__ __launch_bounds__(64 * WAVES) void kb_rollout(BArgs b)
{
    __shared__ DrawLds<OBJ, Real, false> lds;
    __shared__ StagedArgs s_a;
    __shared__ int s_ctx, s_unit;
    if (threadIdx.x == 0) s_ctx = -1;
    const int n = b.desc->n, total = b.desc->n_tiles;
    int item = 0;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_unit = (int)atomicAdd(&b.desc->queue, 1u);
        __syncthreads();
        const int u = s_unit;
        if (u >= total) break;
        item = advance_item(b.tile_prefix, n, u, item);
        stage_args(s_a, s_ctx, b, item);
        const int blk = u - b.tile_prefix[item];
        if (WAVES == 2) rollout2_body<OBJ, Real>(s_a, blk);
        else if (s_a.input_model == INPUT_RATE)
            rollout1_body<OBJ, Real, false, false, true>(s_a, blk, *(const DevCur *)s_a.cur, lds);
        else
            rollout1_body<OBJ, Real, false, false, false>(s_a, blk, *(const DevCur *)s_a.cur, lds);
    }
}

template <int OBJ, typename Real> __global__ __launch_bounds__(192) void kb_rollout3(BArgs b)
{
    __shared__ StagedArgs s_a;
    __shared__ HeadVals h;
    __shared__ int s_ctx, s_unit;
    if (threadIdx.x == 0) s_ctx = -1;
    const int n = b.desc->n, total = b.desc->n_tiles;
    int item = 0;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_unit = (int)atomicAdd(&b.desc->queue, 1u);
        __syncthreads();
        const int u = s_unit;
        if (u >= total) break;
        item = advance_item(b.tile_prefix, n, u, item);
        stage_args(s_a, s_ctx, b, item);
        const int blk = u - b.tile_prefix[item];
        compute_head<OBJ == OBJ_CONTOUR>(s_a, h);
        if (blk == 0 && threadIdx.x == 0) publish_head(s_a, h);
        rollout3_body<OBJ, Real>(s_a, blk, h);
    }
}

// Rings of 4 steps in binary32 leave LDS for two workgroups on a CU, the bound
// of four waves per SIMD the registers too (without it 168 and 165 for
// contouring and tracking: one workgroup.  One context in a batch, K = 20000,
// N = 50: contouring 96 -> 75 us a step, tracking 82 -> 70).
template <int OBJ, typename Real, int R>
__global__ __launch_bounds__(64 * pipe_waves(OBJ, sizeof(Real)), sizeof(Real) == 4 && R == 4 ? 4 : 1) void kb_rollout4(BArgs b)
{
    __shared__ StagedArgs s_a;
    __shared__ HeadVals h;
    __shared__ int s_ctx, s_unit;
    if (threadIdx.x == 0) s_ctx = -1;
    const int n = b.desc->n, total = b.desc->n_tiles;
    int item = 0;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_unit = (int)atomicAdd(&b.desc->queue, 1u);
        __syncthreads();
        const int u = s_unit;
        if (u >= total) break;
        item = advance_item(b.tile_prefix, n, u, item);
        stage_args(s_a, s_ctx, b, item);
        const int blk = u - b.tile_prefix[item];
        compute_head<OBJ == OBJ_CONTOUR>(s_a, h);
        if (blk == 0 && threadIdx.x == 0) publish_head(s_a, h);
        rollout4_body<OBJ, Real, R>(s_a, blk, h);
    }
}

// One-wave rollouts that draw their samples (binary32): no
// sample kernel.  PIPE: with the pipelined rollout's arithmetic, for launches
// whose tiles fill the chip several times over: a tile then costs the issue
// of one wave's operations instead of the pipeline's latency and handoffs.
// RATE: the launch holds contexts of the rate input; MIXED: beside those of the
// thrust input (12 contexts of K = 4096, N = 50 and three objectives, half of
// them on rates: 575 us a step with a launch per input model, 297 together; a
// launch of rates alone does without the branch: 64 contouring contexts of
// K = 8192 509 -> 489).
// As many waves per SIMD as spill no register (a spilled value is read behind
// the sample's store and waits for it, in every step): two where the
// pipeline's sums or the thrust chain need the registers, else three.  Against
// four, with flat accesses: 256 uneven instances 1231 -> 1201 us; where a SIMD
// has one tile or two and nothing hides the wait: 12 contexts of K = 4096,
// N = 100, tracking 246 -> 190, gate 228 -> 175 (235 by a sample kernel and a
// rollout that reads its samples); 32 contouring contexts of K = 4096, N = 100
// 404 -> 304.
template <int OBJ, typename Real, bool PIPE, bool RATE, bool MIXED = false>
__global__ __launch_bounds__(64, draw_waves(RATE || PIPE)) void kb_rollout_draw(BArgs b)
{
    __shared__ DrawLds<OBJ, Real, true> lds;
    __shared__ StagedArgs s_a;
    __shared__ HeadVals h;
    __shared__ int s_ctx, s_unit;
    if (threadIdx.x == 0) s_ctx = -1;
    const int n = b.desc->n, total = b.desc->n_tiles;
    int item = 0;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_unit = (int)atomicAdd(&b.desc->queue, 1u);
        __syncthreads();
        const int u = s_unit;
        if (u >= total) break;
        item = advance_item(b.tile_prefix, n, u, item);
        stage_args(s_a, s_ctx, b, item);
        const int blk = u - b.tile_prefix[item];
        compute_head<OBJ == OBJ_CONTOUR>(s_a, h);
        if (blk == 0 && threadIdx.x == 0) publish_head(s_a, h);
        if (RATE && (!MIXED || s_a.input_model == INPUT_RATE)) rollout1_body<OBJ, Real, true, PIPE, RATE>(s_a, blk, h, lds);
        else rollout1_body<OBJ, Real, true, PIPE, false>(s_a, blk, h, lds);
    }
}

// One unit per (item, 64-sample tile) of the control-cost term; items
// without the term are skipped.
template <typename Real, bool HAS_V> __global__ __launch_bounds__(64) void kb_ctrl_cost(BArgs b)
{
    __shared__ StagedArgs s_a;
    __shared__ int s_ctx;
    if (threadIdx.x == 0) s_ctx = -1;
    __syncthreads();
    const int n = b.desc->n, total = b.desc->n_tiles;
    int item = 0;
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        item = advance_item(b.tile_prefix, n, u, item);
        stage_args(s_a, s_ctx, b, item);
        if (s_a.ctrl_cost != 0.0) ctrl_cost_body<Real, HAS_V>(s_a, u - b.tile_prefix[item]);
        __syncthreads();
    }
}

// One unit per (item, S steps) of the weighted average.  The sample and rollout
// kernels of this step have finished, so their work queues are reset here
// for the next iteration of the step.
// S = final_steps() where the steps outnumber the CUs, else 1: blocks of several
// steps would then leave CUs without one (4 contexts of K = 16384, N = 50, all
// weights alive: 35 us in 52 blocks, 12 in 200; 3 of K = 8192, N = 100, sharp
// weights: 5 us more in 300 blocks than in 75).  With so few blocks binary32
// sums read all samples, without waiting for their weights (samples that are
// drawn again cost only where they weigh something).
// (With both averages in one kernel its registers spill: 12 us a launch -> 17.)
template <typename Real, typename Acc, bool HAS_V, int S, bool REGEN>
__global__ __launch_bounds__(kFinalThreads) void kb_final(BArgs b)
{
    // loads in flight: of several steps one (two spill: 256 uneven instances
    // 1223 -> 1213 us), else final_loads()
    constexpr int UR = S > 1 ? 1 : final_loads<Real>;
    constexpr bool SKIP = REGEN || S > 1 || sizeof(Acc) == 8;
    __shared__ FinalLds<Acc, HAS_V, S> lds;
    __shared__ StagedArgs s_a;
    __shared__ int s_ctx;
    if (threadIdx.x == 0) s_ctx = -1;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        b.desc->queue = 0u;
        b.desc->sample_queue = 0u;
    }
    // every thread reads s_ctx in stage_args before its first barrier
    __syncthreads();
    const int n = b.desc->n, total = b.desc->n_steps;
    int item = 0;
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        item = advance_item(b.step_prefix, n, u, item);
        stage_args(s_a, s_ctx, b, item);
        final_body<Real, Acc, HAS_V, REGEN, UR, SKIP, S>(s_a, S * (u - b.step_prefix[item]), lds);
        __syncthreads();
    }
}

// REGEN: the rollouts left no sample tensor, draw the samples again.
template <typename Real, typename Acc, bool HAS_V, int S>
static void launch_batch_average(const BArgs &b, const BatchLaunch &L, hipStream_t st)
{
    if (L.regen) hipLaunchKernelGGL((kb_final<Real, Acc, HAS_V, S, true>), dim3(L.final_groups), dim3(kFinalThreads), 0, st, b);
    else hipLaunchKernelGGL((kb_final<Real, Acc, HAS_V, S, false>), dim3(L.final_groups), dim3(kFinalThreads), 0, st, b);
}

template <typename Real, int OBJ>
static hipError_t launch_batch_t(const BArgs &b, const BatchLaunch &L, hipStream_t st, int32_t *ran)
{
    constexpr bool HAS_V = OBJ == OBJ_CONTOUR;
    if constexpr (sizeof(Real) == 4) {
        if (L.draw) {
            if (L.rollout_waves == 4) {
                *ran |= MPPI_RAN_WIDE;
                hipLaunchKernelGGL((kb_rollout_draw<OBJ, Real, true, false>), dim3(L.draw_groups), dim3(64), 0, st, b);
            } else if (L.rate && L.thrust) {
                *ran |= MPPI_RAN_MIXED;
                hipLaunchKernelGGL((kb_rollout_draw<OBJ, Real, false, true, true>), dim3(L.draw_groups), dim3(64), 0, st, b);
            } else if (L.rate)
                hipLaunchKernelGGL((kb_rollout_draw<OBJ, Real, false, true>), dim3(L.draw_groups), dim3(64), 0, st, b);
            else
                hipLaunchKernelGGL((kb_rollout_draw<OBJ, Real, false, false>), dim3(L.draw_groups), dim3(64), 0, st, b);
        }
    }
    if (!L.draw && L.rollout_waves < 3)
        hipLaunchKernelGGL((kb_sample<Real, HAS_V>), dim3(L.sample_groups), dim3(256), 0, st, b);
    if (L.draw) {
    } else if (L.rollout_waves == 4) {
        if constexpr (sizeof(Real) == 4) {
            if (L.ring_steps == 8)
                hipLaunchKernelGGL((kb_rollout4<OBJ, Real, 8>), dim3(L.rollout_groups), dim3(64 * pipe_waves(OBJ, sizeof(Real))), 0, st, b);
            else
                hipLaunchKernelGGL((kb_rollout4<OBJ, Real, 4>), dim3(L.rollout_groups), dim3(64 * pipe_waves(OBJ, sizeof(Real))), 0, st, b);
        } else {
            hipLaunchKernelGGL((kb_rollout4<OBJ, Real, 4>), dim3(L.rollout_groups), dim3(64 * pipe_waves(OBJ, sizeof(Real))), 0, st, b);
        }
    } else if (L.rollout_waves == 3)
        hipLaunchKernelGGL((kb_rollout3<OBJ, Real>), dim3(L.rollout_groups), dim3(192), 0, st, b);
    else if (L.rollout_waves == 2)
        hipLaunchKernelGGL((kb_rollout<OBJ, Real, 2>), dim3(L.rollout_groups), dim3(128), 0, st, b);
    else if constexpr (sizeof(Real) == 8)   // (binary32 draws)
        hipLaunchKernelGGL((kb_rollout<OBJ, Real, 1>), dim3(L.rollout_groups), dim3(64), 0, st, b);
    if (L.ctrl_groups > 0)
        hipLaunchKernelGGL((kb_ctrl_cost<Real, HAS_V>), dim3(L.ctrl_groups), dim3(64), 0, st, b);
    if (L.acc64 || sizeof(Real) == 8) {
        launch_batch_average<Real, double, HAS_V, final_steps(HAS_V, 8)>(b, L, st);
    } else if constexpr (sizeof(Real) == 4) {
        if (L.single) {
            *ran |= MPPI_RAN_SINGLE;
            launch_batch_average<Real, float, HAS_V, 1>(b, L, st);
        } else {
            launch_batch_average<Real, float, HAS_V, final_steps(HAS_V, 4)>(b, L, st);
        }
    }
    return hipGetLastError();
}

hipError_t launch_batch(const BArgs &b, const BatchLaunch &L, hipStream_t st, int32_t *ran)
{
    if (L.fp64) {
        switch (L.objective) {
        case OBJ_CONTOUR: return launch_batch_t<double, OBJ_CONTOUR>(b, L, st, ran);
        case OBJ_TRACK: return launch_batch_t<double, OBJ_TRACK>(b, L, st, ran);
        default: return launch_batch_t<double, OBJ_GATE>(b, L, st, ran);
        }
    }
    switch (L.objective) {
    case OBJ_CONTOUR: return launch_batch_t<float, OBJ_CONTOUR>(b, L, st, ran);
    case OBJ_TRACK: return launch_batch_t<float, OBJ_TRACK>(b, L, st, ran);
    default: return launch_batch_t<float, OBJ_GATE>(b, L, st, ran);
    }
}

// ---------------------------------------------------------------- launches

template <typename Real> static hipError_t launch_setup_t(const KArgs &a, hipStream_t st)
{
    int n = a.G > a.P ? a.G : a.P;
    if (a.R > n) n = a.R;
    if (n < 1) n = 1;
    hipLaunchKernelGGL(k_setup<Real>, dim3((n + 255) / 256), dim3(256), 0, st, a);
    return hipGetLastError();
}

struct Request { double v[kReqDoubles]; };

__global__ __launch_bounds__(64) void k_request(Request r, double *d_req)
{
    if (threadIdx.x < kReqDoubles) d_req[threadIdx.x] = r.v[threadIdx.x];
}

hipError_t launch_request(const double *values, double *d_req, hipStream_t st)
{
    Request r;
    for (int i = 0; i < kReqDoubles; ++i) r.v[i] = values[i];
    hipLaunchKernelGGL(k_request, dim3(1), dim3(64), 0, st, r, d_req);
    return hipGetLastError();
}

hipError_t launch_setup(const KArgs &a, bool fp64, hipStream_t st)
{
    return fp64 ? launch_setup_t<double>(a, st) : launch_setup_t<float>(a, st);
}

template <typename Real, typename Acc, bool HAS_V>
static hipError_t launch_average_t(const KArgs &a, hipStream_t st)
{
    // binary32: all of a thread's samples in one round of loads when they are
    // at most eight, else (and in binary64, whose registers hold half as
    // many) rounds of final_loads with the next round's loads in flight; the
    // accumulation order, and so the result, is the same either way
    if constexpr (sizeof(Real) == 4) {
        if (a.K <= 8 * kFinalThreads) {
            // (K < 65536 takes binary32 sums)
            if (a.regen) hipLaunchKernelGGL((k_final<Real, Real, HAS_V, true, 8, false>), dim3(a.N), dim3(kFinalThreads), 0, st, a);
            else hipLaunchKernelGGL((k_final<Real, Real, HAS_V, false, 8, false>), dim3(a.N), dim3(kFinalThreads), 0, st, a);
            return hipGetLastError();
        }
    }
    if (a.regen)
        hipLaunchKernelGGL((k_final<Real, Acc, HAS_V, true, final_loads<Real>, true>), dim3(a.N), dim3(kFinalThreads), 0, st, a);
    else
        hipLaunchKernelGGL((k_final<Real, Acc, HAS_V, false, final_loads<Real>, true>), dim3(a.N), dim3(kFinalThreads), 0, st, a);
    return hipGetLastError();
}

template <typename Real, int OBJ>
static hipError_t launch_solve_t(const KArgs &a, bool acc64, hipStream_t st, hipEvent_t *ev, int32_t *ran)
{
    constexpr bool HAS_V = OBJ == OBJ_CONTOUR;
    const dim3 gs((a.K + 1 + 255) / 256, (a.N + kSampleSteps - 1) / kSampleSteps);
    if (ev) (void)hipEventRecord(ev[0], st);
    // a one-wave rollout that draws its samples (binary32) needs only the head first
    const bool draw = sizeof(Real) == 4 && a.rollout_draw && !a.rollout_pair;
    if (draw) {
        if constexpr (sizeof(Real) == 4) hipLaunchKernelGGL(k_head<HAS_V>, dim3(1), dim3(256), 0, st, a);
    } else if (a.rollout_waves < 3 && !a.rate_pipe && !a.rollout_pair) {
        hipLaunchKernelGGL((k_sample<Real, HAS_V>), gs, dim3(256), 0, st, a);
    }
    if (ev) (void)hipEventRecord(ev[1], st);
    const dim3 gt((a.K + 1 + 63) / 64);
    *ran = 0;
    if (a.rate_pipe) {
        // (rings of 4 where 8 would not fit the LDS; binary64 contouring not at all)
        constexpr int R = sizeof(Real) == 8 || OBJ == OBJ_CONTOUR ? 4 : 8;
        if constexpr (rate_pipe_fits(OBJ, sizeof(Real))) {
            *ran = MPPI_RAN_RATE_PIPE;
            hipLaunchKernelGGL((k_rollout_rate<OBJ, Real, R>), gt, dim3(64 * rate_pipe_waves(OBJ)), 0, st, a);
        }
    } else if (a.rollout_waves == 4) {
        if constexpr (sizeof(Real) == 4) {
            if (a.ring_steps == 8)
                hipLaunchKernelGGL((k_rollout4<OBJ, Real, 8>), gt, dim3(64 * pipe_waves(OBJ, sizeof(Real))), 0, st, a);
            else
                hipLaunchKernelGGL((k_rollout4<OBJ, Real, 4>), gt, dim3(64 * pipe_waves(OBJ, sizeof(Real))), 0, st, a);
        } else {
            hipLaunchKernelGGL((k_rollout4<OBJ, Real, 4>), gt, dim3(64 * pipe_waves(OBJ, sizeof(Real))), 0, st, a);
        }
    } else if (a.rollout_waves == 3) {
        hipLaunchKernelGGL((k_rollout3<OBJ, Real>), gt, dim3(192), 0, st, a);
    } else if (a.rollout_waves == 2) {
        hipLaunchKernelGGL((k_rollout_split<OBJ, Real>), gt, dim3(128), 0, st, a);
    } else if (a.rollout_pair) {
        if constexpr (sizeof(Real) == 4) {
            *ran = MPPI_RAN_PAIR;
            hipLaunchKernelGGL((k_rollout_pair<OBJ, Real>), gt, dim3(128), 0, st, a);
        }
    } else if (draw) {
        if constexpr (sizeof(Real) == 4) hipLaunchKernelGGL((k_rollout<OBJ, Real, true>), gt, dim3(64), 0, st, a);
    } else {
        hipLaunchKernelGGL((k_rollout<OBJ, Real, false>), gt, dim3(64), 0, st, a);
    }
    if (a.ctrl_cost != 0.0)
        hipLaunchKernelGGL((k_ctrl_cost<Real, HAS_V>), dim3(a.n_tiles), dim3(64), 0, st, a);
    if (ev) (void)hipEventRecord(ev[2], st);
    hipError_t e;
    if constexpr (sizeof(Real) == 8) e = launch_average_t<Real, double, HAS_V>(a, st);
    else e = acc64 ? launch_average_t<Real, double, HAS_V>(a, st) : launch_average_t<Real, float, HAS_V>(a, st);
    if (ev) (void)hipEventRecord(ev[3], st);
    return e;
}

hipError_t launch_solve(const KArgs &a, bool fp64, bool acc64, hipStream_t st, hipEvent_t *ev, int32_t *ran)
{
    if (fp64) {
        switch (a.objective) {
        case OBJ_CONTOUR: return launch_solve_t<double, OBJ_CONTOUR>(a, true, st, ev, ran);
        case OBJ_TRACK: return launch_solve_t<double, OBJ_TRACK>(a, true, st, ev, ran);
        default: return launch_solve_t<double, OBJ_GATE>(a, true, st, ev, ran);
        }
    }
    switch (a.objective) {
    case OBJ_CONTOUR: return launch_solve_t<float, OBJ_CONTOUR>(a, acc64, st, ev, ran);
    case OBJ_TRACK: return launch_solve_t<float, OBJ_TRACK>(a, acc64, st, ev, ran);
    default: return launch_solve_t<float, OBJ_GATE>(a, acc64, st, ev, ran);
    }
}

// ------------------------------------------------------- fixed workspace

// Workspace of the allocation-free solve: one array per GPU, held by the
// library's code object until the process ends.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the symbol):
// it resolves the device address per device and passes that.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_lock;
void *g_scratch_ptr[kScratchDevices] = {};
}  // namespace

hipError_t scratch_address(void **ptr)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace mppi
