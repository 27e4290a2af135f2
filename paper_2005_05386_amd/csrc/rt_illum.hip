// Riemannian illumination, direct part (Sec. 4, "Riemannian illumination"):
// a point q of a surface is lit by a point light L through the geodesics
// that connect q to L, and its radiant intensity is Lambertian, measured
// in the metric.  For every traced pixel that hit an object this pass
//   - finds a geodesic from q to L by shooting: the g-unit direction v at q
//     and the arc length T with gamma_{q,v}(T) = L, solved by Newton's
//     method on two direction angles and T (finite-difference columns for
//     the angles, the end velocity for T), starting from the straight
//     segment;
//   - marches that geodesic (RK4, each step's chord tested against the
//     objects its culling window reaches, hits within 1e-3 of q ignored) to
//     decide whether it reaches L;
//   - takes the Lambert term cos = g(N, v) / |N|_g with N the metric normal
//     of the surface, g^-1 grad F, so that g(N, v) = grad F . v and
//     |N|_g^2 = grad F^T g^-1 grad F.
// Several geodesics may join q and L; this finds the one reached from the
// straight segment.  The paper gives no method for this step.
#include <algorithm>

#include "rt_device.hpp"
#include "rt_internal.hpp"
#include "rt_step.hpp"

using namespace rtd;

namespace {

// Outward gradient of the implicit function of object id at x (sphere
// |x - c|^2 - r^2, plane n.x - d, torus signed distance).
__device__ __forceinline__ V3<float> obj_grad(int id, V3<float> x, int ns, int np, const float4 *__restrict__ SPH,
                                              const float4 *__restrict__ PLN, const float *__restrict__ TOR) {
    if (id < ns) {
        const float4 s = SPH[id];
        return mk(2.f * (x.x - s.x), 2.f * (x.y - s.y), 2.f * (x.z - s.z));
    }
    id -= ns;
    if (id < np) {
        const float4 p = PLN[id];
        return mk(p.x, p.y, p.z);
    }
    const float *tp = TOR + 8 * (id - np);
    const V3<float> q = mk(x.x - tp[0], x.y - tp[1], x.z - tp[2]);
    const V3<float> a = mk(tp[3], tp[4], tp[5]);
    const float ax = dot(q, a);
    const V3<float> rad = axpy(-ax, a, q);
    const float rn = sqrt_(dot(rad, rad));
    const float e = rn - tp[6];
    const V3<float> g = axpy(ax, a, (rn > 1e-20f ? e / rn : 0.f) * rad);
    return rsqrt_(e * e + ax * ax) * g;
}

// Culling windows of the shots and the visibility march: every
// ILLUM_CULL_EVERY steps a lane's window is the box of half-width
// A.cull_margin about its position (the distance it can cover before the
// next window, from the metric's speed bound); the bumps and objects that
// some active lane's window reaches are OR-ed over the wave by ballots.
// Isotropic and anisotropic graph bumps are culled this way; the other
// kinds walk every record of the table and skip, wave by wave, a record no
// lane is inside.
template <int KIND> constexpr bool bump_cull = KIND == KIND_GRAPH || KIND == KIND_GANISO;
template <int KIND> using IAcc = Acc32<KIND, false, false, !bump_cull<KIND>>;

struct Box {
    float lo[3], hi[3];
};
__device__ __forceinline__ Box lane_box(V3<float> p, float m) {
    return {{p.x - m, p.y - m, p.z - m}, {p.x + m, p.y + m, p.z + m}};
}

template <int KIND>
__device__ __forceinline__ uint64_t bump_window(const float4 *__restrict__ Bs, int n, const Box &w) {
    uint64_t mask = 0;
    for (int b = 0; b < n; ++b) {
        const float4 b0 = Bs[2 * b], b1 = Bs[2 * b + 1];
        bool need;
        if constexpr (KIND == KIND_GRAPH) {
            need = box_dist2(b0.x, b0.y, b0.z, w.lo, w.hi) <= b1.z;
        } else {
            const float rho = aniso_box_rho(b0, b1, w.lo, w.hi);
            need = rho * rho <= b1.w * 1.00001f;
        }
        if (ballot(need)) mask |= 1ull << b;
    }
    return mask;
}

// Steps of length h that every lane of the wave can take at constant velocity
// before the first lane's gap (1e6: none) is used up by the fastest lane (the
// shots' own speed, which coarse steps take away from that of a g-unit velocity).
__device__ __forceinline__ int steps_within(float gap, V3<float> y, bool on, float h) {
    const float v = sqrt_(wave_max(on ? dot(y, y) : 0.f)) * 1.0001f;
    const float q = (wave_min(on ? gap : 1e6f) * 0.999f - 2e-4f) * rcp_(fmaxf(v, 1e-3f) * h) - 2.0f;
    return (int)fminf(fmaxf(q, 0.f), 1e6f);
}
// The same from p to the next cut region (an anisotropic one taken as a ball),
// for the lanes with `on`; called by the whole wave.
template <int KIND>
__device__ __forceinline__ int free_steps(const float4 *__restrict__ Bs, int n, V3<float> p, V3<float> y, bool on, float h) {
    float gap = 1e6f;
    for (int b = 0; b < n; ++b) {
        const float4 b0 = Bs[2 * b], b1 = Bs[2 * b + 1];
        const V3<float> d = mk(p.x - b0.x, p.y - b0.y, p.z - b0.z);
        float R;
        if constexpr (KIND == KIND_GRAPH) R = sqrt_(b1.z);
        else R = sqrt_(b1.w) * rsqrt_(fminf(fminf(b1.x, b1.y), b1.z));
        gap = fminf(gap, sqrt_(dot(d, d)) - R * 1.0001f);
    }
    return steps_within(gap, y, on, h);
}

// Integrate the geodesic from (q, v) over arc length T: n = ceil(T / h)
// RK4 steps, the last one shortened; two-float position.  False on a
// non-finite state or a step budget overrun (and for lanes not active, which
// only take part in the wave's questions: called by the whole wave).  Where
// the window reaches no bump the lanes fly free, a constant increment per
// step, until the nearest cut region: the long shots of the last iterations
// spend most of their length outside the bumps.
template <int KIND>
__device__ __forceinline__ bool shoot(IAcc<KIND> &acc, const rti::IllumArgs &A, bool active, V3<float> q, V3<float> v,
                                      float T, V3<float> &X, V3<float> &Y) {
    const float h = A.h;
    int n = active ? max(1, (int)ceilf(T / h)) : 0;
    bool ok = active && n <= A.max_steps;
    if (!ok) n = 0;
    V3<float> xh = q, xl = mk(0.f, 0.f, 0.f), y = v;
    int wend = 0;
    for (int i = 0; ballot(i < n) != 0;) {
        if constexpr (bump_cull<KIND>) {
            if (i >= wend && A.cull_margin >= 0.f) {
                wend = i + rti::ILLUM_CULL_EVERY;
                const bool on = i < n;
                uint64_t mask = 0;
                if (on) mask = bump_window<KIND>(acc.B, A.n_bumps, lane_box(xh + xl, A.cull_margin));
                // (the same for every lane with on)
                const int src = __builtin_ctzll(ballot(on));
                acc.mask = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mask, src) |
                           ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mask >> 32), src) << 32);
                if (acc.mask == 0) {
                    const V3<float> dx = free_step<STEP_RK4>(y, h);
                    const int m = free_steps<KIND>(acc.B, A.n_bumps, xh + xl, y, on, h);
                    if (m > 0 && ballot(on && !finite6(dx, mk(0.f, 0.f, 0.f))) == 0) {
                        if (on) {
                            y = y + mk(0.f, 0.f, 0.f);
                            const int c = min(m, n - 1 - i);
                            for (int j = 0; j < c; ++j) {
                                two_sum_add(xh.x, xl.x, dx.x);
                                two_sum_add(xh.y, xl.y, dx.y);
                                two_sum_add(xh.z, xl.z, dx.z);
                            }
                            if (c < m) {
                                // the lane's last, shortened step
                                const V3<float> dl = free_step<STEP_RK4>(y, T - (float)(n - 1) * h);
                                two_sum_add(xh.x, xl.x, dl.x);
                                two_sum_add(xh.y, xl.y, dl.y);
                                two_sum_add(xh.z, xl.z, dl.z);
                                n = 0;
                            }
                        }
                        i += m;
                        wend = i;
                        continue;
                    }
                }
            }
        }
        if (i < n) {
            const float hs = i == n - 1 ? T - (float)(n - 1) * h : h;
            V3<float> dx, dv;
            if (!step_rk4<float>(acc, xh + xl, y, hs, dx, dv) || !finite6(dx, dv)) {
                ok = false;
                n = 0;
            } else {
                two_sum_add(xh.x, xl.x, dx.x);
                two_sum_add(xh.y, xl.y, dx.y);
                two_sum_add(xh.z, xl.z, dx.z);
                y = y + dv;
            }
        }
        ++i;
    }
    X = xh + xl;
    Y = y;
    return ok;
}

// Isotropic bumps spread over the 16 lanes of a DPP row: lane l holds the
// bumps l, l + 16, ... of a table of up to 16 NB (the others have weight
// zero), every lane of the row the same state.  A stage computes the terms of
// 16 bumps at once, each lane its own, and then every lane adds them up in
// increasing index order, the terms broadcast along the row: the values of the
// walk, without its chain of loads and exponentials.  Groups of four bumps
// that act on no lane of the wave are left out (their terms are zero).  Needs
// all 64 lanes.
template <int NB> struct RowBumps {
    float4 b0[NB], b1[NB];
    bool two;    // some lane's second bump may act
    bool &seen;  // some bump acted since cleared
    // The terms of the bumps of lanes N..N+3 of each row, in this order: one
    // move and four multiply-adds per bump, their first factor read along the
    // row (from the compiler, a move for each of the five).
    template <int N>
    static __device__ __forceinline__ void add4(GraphAccum &A, float w, V3<float> d, float t) {
        float w0, w1;
#define RT_ROW_TERM(W, L) \
    "v_mov_b32_dpp " W ", %6 row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp %0, %7, " W " row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp %1, %8, " W " row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp %2, %9, " W " row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp %3, %10, " W " row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t"
        __asm__("s_nop 1\n\t" RT_ROW_TERM("%4", "%c11") RT_ROW_TERM("%5", "%c12") RT_ROW_TERM("%4", "%c13")
                    RT_ROW_TERM("%5", "%c14")
                : "+v"(A.gx), "+v"(A.gy), "+v"(A.gz), "+v"(A.q), "=&v"(w0), "=&v"(w1)
                : "v"(w), "v"(d.x), "v"(d.y), "v"(d.z), "v"(t), "n"(N), "n"(N + 1), "n"(N + 2), "n"(N + 3));
#undef RT_ROW_TERM
    }
    __device__ __forceinline__ bool operator()(V3<float> p, V3<float> y, V3<float> &a) const {
        GraphAccum A{0.f, 0.f, 0.f, 0.f};
        const float yy = dot(y, y);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (k > 0 && !two) break;
            const V3<float> d = mk(p.x - b0[k].x, p.y - b0[k].y, p.z - b0[k].z);
            const float r2 = fmaf(d.z, d.z, fmaf(d.y, d.y, d.x * d.x));
            const float e = exp2_(b0[k].w * r2);
            const float w = r2 <= b1[k].z ? -(b1[k].x * e) : 0.0f;  // (both factors of q negated)
            const float dv = fmaf(d.z, y.z, fmaf(d.y, y.y, d.x * y.x));
            const float t = -fmaf(b1[k].y, dv * dv, -yy);
            const uint64_t in = ballot(w != 0.0f);
            const uint32_t m = (uint32_t)in | (uint32_t)(in >> 32);
            if (m & 0x000F000Fu) add4<0>(A, w, d, t);
            if (m & 0x00F000F0u) add4<4>(A, w, d, t);
            if (m & 0x0F000F00u) add4<8>(A, w, d, t);
            if (m & 0xF000F000u) add4<12>(A, w, d, t);
            seen |= m != 0;
        }
        a = graph_finish(A);
        return true;
    }
};

// shoot of one geodesic per row, T the same in every lane (the whole wave
// takes the same steps; a row that failed is left to run on).  At each culling
// window the bumps that some row's window reaches are moved to the first
// lanes, in their order, so that whole groups of four are left out of the sums
// (frames of 63x47 with 18 bumps 31.6 ms in place, 23.5 moved; 677x342 with 20
// bumps 103 and 83; 1080p with 16 bumps 236 and 235).
template <int NB>
__device__ __forceinline__ bool shoot_rows(const float4 (&b0)[NB], const float4 (&b1)[NB], const rti::IllumArgs &A,
                                           V3<float> q, V3<float> v, float T, V3<float> &X, V3<float> &Y) {
    const float h = A.h;
    const int n = uniform_i(max(1, (int)ceilf(T / h)));
    bool ok = n <= A.max_steps, seen = false;
    V3<float> xh = q, xl = mk(0.f, 0.f, 0.f), y = v;
    RowBumps<NB> acc{{}, {}, false, seen};
    __shared__ float4 tab[32 * NB];
    const int l = lane_id() & 15;
    float R[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) R[k] = b1[k].z >= 0.f ? sqrt_(b1[k].z) * 1.0001f : -1e6f;
    int fly = 0;   // first step to look for free flight again
    int wend = 0;  // first step of the next window
    for (int i = 0; i < n && ballot(ok);) {
        if (i >= wend) {
            wend = i + rti::ILLUM_CULL_EVERY;
            const Box w = lane_box(xh + xl, A.cull_margin);
            uint32_t need = 0;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                uint64_t m = ballot(ok && box_dist2(b0[k].x, b0[k].y, b0[k].z, w.lo, w.hi) <= b1[k].z);
                m |= m >> 32;
                need |= ((uint32_t)(m | m >> 16) & 0xFFFFu) << (16 * k);
            }
            const int count = __popc(need);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                // needed ones first; the others keep their places behind them
                const int j = l + 16 * k, rank = __popc(need & ((1u << j) - 1u));
                const int pos = (need >> j) & 1u ? rank : count + j - rank;
                tab[2 * pos] = b0[k];
                tab[2 * pos + 1] = b1[k];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                acc.b0[k] = tab[2 * (l + 16 * k)];
                acc.b1[k] = tab[2 * (l + 16 * k) + 1];
            }
            acc.two = count > 16;
        }
        seen = false;
        const float hs = i == n - 1 ? T - (float)(n - 1) * h : h;
        V3<float> dx, dv;
        step_rk4<float>(acc, xh + xl, y, hs, dx, dv);
        ok = ok && finite6(dx, dv);
        two_sum_add(xh.x, xl.x, dx.x);
        two_sum_add(xh.y, xl.y, dx.y);
        two_sum_add(xh.z, xl.z, dx.z);
        y = y + dv;
        ++i;
        if (!seen && i >= fly) {
            // steps free of every cut region for every row, as free_steps
            const V3<float> p = xh + xl;
            float gap = 1e6f;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const V3<float> d = mk(p.x - b0[k].x, p.y - b0[k].y, p.z - b0[k].z);
                gap = fminf(gap, sqrt_(dot(d, d)) - R[k]);
            }
            const int m = uniform_i(min(steps_within(gap, y, ok, h), n - 1 - i));
            fly = i + 4;
            if (m > 0) {
                const V3<float> dx1 = free_step<STEP_RK4>(y, h);
                for (int j = 0; j < m; ++j) {
                    two_sum_add(xh.x, xl.x, dx1.x);
                    two_sum_add(xh.y, xl.y, dx1.y);
                    two_sum_add(xh.z, xl.z, dx1.z);
                }
                i += m;
            }
        }
    }
    X = xh + xl;
    Y = y;
    return ok;
}

// March the same geodesic with the chord of every step tested against the
// objects of the window; true when nothing is crossed between t = skip and
// t = T.
template <int KIND>
__device__ __forceinline__ bool reaches(IAcc<KIND> &acc, V3<float> q, V3<float> v, float T, float skip,
                                        const rti::IllumArgs &A, const float4 *__restrict__ SPH,
                                        const float4 *__restrict__ PLN, const float *__restrict__ TOR) {
    const float h = A.h;
    const int n = max(1, (int)ceilf(T / h));
    const int no = A.n_planes + A.n_tori;
    V3<float> xh = q, xl = mk(0.f, 0.f, 0.f), y = v;
    float t = 0.f;
    uint64_t sm[4] = {0ull, 0ull, 0ull, 0ull};
    uint32_t om = 0;
    for (int i = 0; i < n; ++i) {
        const V3<float> p = xh + xl;
        if (i % rti::ILLUM_CULL_EVERY == 0) {
            if (A.cull_margin >= 0.f) {
                const Box w = lane_box(p, A.cull_margin);
                if constexpr (bump_cull<KIND>) acc.mask = bump_window<KIND>(acc.B, A.n_bumps, w);
#pragma unroll
                for (int c = 0; c < 4; ++c) sm[c] = 0ull;
                for (int k = 0; k < A.n_spheres; ++k) {
                    const float4 s = SPH[k];
                    if (ballot(box_dist2(s.x, s.y, s.z, w.lo, w.hi) <= s.w * s.w)) sm[k >> 6] |= 1ull << (k & 63);
                }
                om = 0;
                for (int k = 0; k < no; ++k) {
                    bool on;
                    if (k < A.n_planes) {
                        const float4 pl = PLN[k];
                        const float c = pl.x * p.x + pl.y * p.y + pl.z * p.z - pl.w;
                        on = fabsf(c) <= A.cull_margin * (fabsf(pl.x) + fabsf(pl.y) + fabsf(pl.z));
                    } else {
                        const float *tp = TOR + 8 * (k - A.n_planes);
                        const float rr = tp[6] + tp[7];
                        on = box_dist2(tp[0], tp[1], tp[2], w.lo, w.hi) <= rr * rr;
                    }
                    if (ballot(on)) om |= 1u << k;
                }
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int rem = A.n_spheres - 64 * c;
                    sm[c] = rem >= 64 ? ~0ull : (rem > 0 ? (1ull << rem) - 1ull : 0ull);
                }
                om = (1u << no) - 1u;
            }
        }
        const float hs = i == n - 1 ? T - (float)(n - 1) * h : h;
        V3<float> dx, dv;
        if (!step_rk4<float>(acc, p, y, hs, dx, dv)) return false;
        const float DD = dot(dx, dx);
        float first = 2.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            for (uint64_t m = sm[c]; m; m &= m - 1ull) {
                const float4 s = SPH[64 * c + __builtin_ctzll(m)];
                const V3<float> o = mk((xh.x - s.x) + xl.x, (xh.y - s.y) + xl.y, (xh.z - s.z) + xl.z);
                // both roots: a chord that starts on a sphere (s ~ 0) may still cross it later
                const float B = dot(dx, o), C = fmaf(-s.w, s.w, dot(o, o));
                const float disc = fmaf(B, B, -DD * C);
                if (disc >= 0.f) {
                    const float qd = sqrt_(disc), inv = rcp_(DD);
                    const float s1 = (-B - qd) * inv, s2 = (-B + qd) * inv;
                    if (s1 >= 0.f && s1 <= 1.f && t + s1 * hs > skip) first = fminf(first, s1);
                    else if (s2 >= 0.f && s2 <= 1.f && t + s2 * hs > skip) first = fminf(first, s2);
                }
            }
        }
        for (uint32_t m = om; m; m &= m - 1u) {
            const int k = __builtin_ctz(m);
            float F0, F1;
            if (k < A.n_planes) {
                const float4 pl = PLN[k];
                F0 = pl.x * p.x + pl.y * p.y + pl.z * p.z - pl.w;
                F1 = F0 + (pl.x * dx.x + pl.y * dx.y + pl.z * dx.z);
            } else {
                const float *tp = TOR + 8 * (k - A.n_planes);
                F0 = torus_sdf<float>(tp, p);
                F1 = torus_sdf<float>(tp, p + dx);
            }
            if ((F0 > 0.f) != (F1 > 0.f)) {
                const float sc = fminf(fmaxf(F0 / (F0 - F1), 0.f), 1.f);
                if (t + sc * hs > skip) first = fminf(first, sc);
            }
        }
        if (first <= 1.f) return false;
        two_sum_add(xh.x, xl.x, dx.x);
        two_sum_add(xh.y, xl.y, dx.y);
        two_sum_add(xh.z, xl.z, dx.z);
        y = y + dv;
        t += hs;
    }
    return true;
}

// Per-pixel frame about the straight direction to the light and the
// direction for the angles (al, be), normalised to g-unit at q.
struct Frame {
    V3<float> e0, e1, e2;
};
__device__ __forceinline__ Frame light_frame(V3<float> q, V3<float> L) {
    const V3<float> dl = L - q;
    Frame f;
    f.e0 = rsqrt_(dot(dl, dl)) * dl;
    const V3<float> t0 = fabsf(f.e0.x) < 0.9f ? mk(1.f, 0.f, 0.f) : mk(0.f, 1.f, 0.f);
    f.e1 = axpy(-dot(t0, f.e0), f.e0, t0);
    f.e1 = rsqrt_(dot(f.e1, f.e1)) * f.e1;
    f.e2 = mk(f.e0.y * f.e1.z - f.e0.z * f.e1.y, f.e0.z * f.e1.x - f.e0.x * f.e1.z, f.e0.x * f.e1.y - f.e0.y * f.e1.x);
    return f;
}

// Everything a lane needs for one pixel.
template <int KIND> struct Pixel {
    const float4 *Bs;
    V3<float> q;
    Frame F;
    __device__ __forceinline__ float gdd(const rti::IllumArgs &A, V3<float> d) const {
        return metric_gdd<KIND>(Bs, A.n_bumps, A.twist_amp, A.twist_theta0, q, d);
    }
    __device__ __forceinline__ V3<float> dir(const rti::IllumArgs &A, float al, float be) const {
        const V3<float> u = axpy(be, F.e2, axpy(al, F.e1, F.e0));
        return rsqrt_(gdd(A, u)) * u;
    }
};
// ONE: a single parameter set, so the table pointer is the same for every
// lane and the bump records are read with scalar loads.
template <int KIND, bool ONE = false>
__device__ __forceinline__ Pixel<KIND> pixel(const rti::IllumArgs &A, const float4 *__restrict__ BF, int pix) {
    Pixel<KIND> P;
    if constexpr (ONE) {
        P.Bs = BF;
    } else {
        const int set = pix / (A.width * A.height);
        P.Bs = BF + (int64_t)set * A.n_bumps * (is_deform(KIND) ? DEFORM_F4 : 2);
    }
    P.q = mk(A.hit[3 * pix], A.hit[3 * pix + 1], A.hit[3 * pix + 2]);
    P.F = light_frame(P.q, mk(A.light[0], A.light[1], A.light[2]));
    return P;
}
__device__ __forceinline__ uint64_t all_bumps(int n) { return n >= 64 ? ~0ull : ((1ull << n) - 1ull); }

// Wave-aggregated append of pix to list (count at *ctr).
__device__ __forceinline__ void append(int *list, int *ctr, int pix, bool take) {
    const uint64_t m = ballot(take);
    if (!m) return;
    const int lane = lane_id();
    const int leader = __builtin_ctzll(m);
    int base = 0;
    if (lane == leader) base = atomicAdd(ctr, __popcll(m));
    base = __shfl(base, leader);
    if (take) list[base + __popcll(m & ((1ull << lane) - 1ull))] = pix;
}

// Status codes of the API; 3 marks a converged pixel awaiting the finish,
// 4 one converged at an intermediate target of the continuation.
enum { ST_LIT = 1, ST_BLOCKED = 0, ST_AWAY = 2, ST_NONE = -1, ST_NOHIT = -3, ST_CONV = 3, ST_CONT = 4 };

// The target of the shots of pixel P: the light, or during the
// continuation the point q + cont (L - q) of the straight segment.
template <class P> __device__ __forceinline__ V3<float> target(float cont, const P &Px, V3<float> L) {
    return cont < 1.f ? axpy(cont, L - Px.q, Px.q) : L;
}

// Pixels per wave when the three shots of an iteration run on three lanes.
constexpr int PAR_PIX = 21;
// The lines below count waves of the whole device, here per CU (sizes quoted are
// those of 256 CUs).  A list is short while 32 waves per CU hold it at three lanes
// per pixel (172032 pixels).
__device__ __host__ __forceinline__ int short_list(const rti::IllumArgs &A) { return A.n_cu * 32 * PAR_PIX; }

// Pixel t of the frames, in the order of the lists, and the count of such t.
// Frames of more than short_list pixels go in 8x8 tiles, one per wave (-1
// beyond the edge): the windows of the full-grid launches then cover a tile
// instead of a strip of 64 pixels and reach fewer bumps (1080p with 16 bumps
// 236 ms in strips, 224 in tiles; 818x557 with 4 bumps 18.5 and 18.3).  Smaller
// frames, whose lists are solved pixel by pixel, keep the strips (127x75 with 3
// bumps 3.97 ms, in tiles 4.45: the finish reaches more objects at once).
__device__ __forceinline__ bool in_tiles(const rti::IllumArgs &A) {
    return (int64_t)A.n_sets * A.width * A.height > short_list(A);
}
__device__ __forceinline__ int64_t pixel_count(const rti::IllumArgs &A) {
    return in_tiles(A) ? (int64_t)A.n_sets * ((A.width + 7) / 8) * ((A.height + 7) / 8) * 64
                       : (int64_t)A.n_sets * A.width * A.height;
}
__device__ __forceinline__ int nth_pixel(const rti::IllumArgs &A, int64_t t) {
    if (!in_tiles(A)) return t < (int64_t)A.n_sets * A.width * A.height ? (int)t : -1;
    const int tx = (A.width + 7) / 8, ty = (A.height + 7) / 8;
    const int w = (int)(t >> 6), set = w / (tx * ty), r = w - set * (tx * ty), j = r / tx, i = r - j * tx;
    const int x = 8 * i + (int)(t & 7), y = 8 * j + (int)((t >> 3) & 7);
    return set < A.n_sets && x < A.width && y < A.height ? (set * A.height + y) * A.width + x : -1;
}

// Initial state: pixels that hit start from the straight segment.
template <int KIND>
__global__ __launch_bounds__(256) void k_illum_init(rti::IllumArgs A, const float4 *__restrict__ BF) {
    const int64_t n = pixel_count(A);
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
        const int pix = nth_pixel(A, base + threadIdx.x);
        const bool hit = pix >= 0 && A.id[pix] >= 0;
        if (pix >= 0) {
            float T = 0.f;
            if (hit) {
                const Pixel<KIND> P = pixel<KIND>(A, BF, pix);
                const V3<float> L = mk(A.light[0], A.light[1], A.light[2]);
                T = sqrtf(P.gdd(A, L - P.q));
            }
            A.w_al[pix] = 0.f;
            A.w_be[pix] = 0.f;
            A.w_T[pix] = T;
            A.w_F[pix] = __builtin_huge_valf();
            A.status[pix] = hit ? ST_NONE : ST_NOHIT;
            A.shade[pix] = 0.f;
        }
        append(A.list[0], A.ctr + 0, pix, hit);
    }
}

// Residual F of the base shot in iteration it: a Newton step is to be taken,
// or the pixel leaves the list, converged or stalled (from the fifth iteration
// on, a residual that did not halve).  last: the previous residual, updated.
enum { J_STEP, J_CONV, J_STALL };
__device__ __forceinline__ int assess(const rti::IllumArgs &A, int it, V3<float> F, float &last) {
    const float fn = fmaxf(fabsf(F.x), fmaxf(fabsf(F.y), fabsf(F.z)));
    const bool stalled = it >= 4 && fn > 0.5f * last;
    last = fn;
    return fn < A.tol ? J_CONV : (stalled ? J_STALL : J_STEP);
}

// Damped Newton step on (al, be, T) from the residual F = X - L, the end
// velocity Y (the T column) and the shots Xa, Xb at al + eps, be + eps;
// true when the pixel stays on the list.
template <int KIND>
__device__ __forceinline__ bool newton(const rti::IllumArgs &A, const Pixel<KIND> &P, V3<float> L, float eps,
                                      float &al, float &be, float &T, V3<float> F, V3<float> X, V3<float> Y,
                                      V3<float> Xa, V3<float> Xb) {
    const V3<float> ca = (1.f / eps) * (Xa - X), cb = (1.f / eps) * (Xb - X);
    const float M[9] = {ca.x, cb.x, Y.x, ca.y, cb.y, Y.y, ca.z, cb.z, Y.z};
    const float c0 = M[4] * M[8] - M[5] * M[7], c1 = M[2] * M[7] - M[1] * M[8], c2 = M[1] * M[5] - M[2] * M[4];
    const float c3 = M[5] * M[6] - M[3] * M[8], c4 = M[0] * M[8] - M[2] * M[6], c5 = M[2] * M[3] - M[0] * M[5];
    const float c6 = M[3] * M[7] - M[4] * M[6], c7 = M[1] * M[6] - M[0] * M[7], c8 = M[0] * M[4] - M[1] * M[3];
    const float det = M[0] * c0 + M[1] * c3 + M[2] * c6;
    if (!(fabsf(det) > 1e-20f)) return false;
    const float idet = -1.f / det;
    const float da = idet * (c0 * F.x + c1 * F.y + c2 * F.z);
    const float db = idet * (c3 * F.x + c4 * F.y + c5 * F.z);
    const float dT = idet * (c6 * F.x + c7 * F.y + c8 * F.z);
    // damping: at most 0.3 in the angles and half the length per step
    const float m = fmaxf(fabsf(da), fabsf(db));
    const float sa = m > 0.3f ? 0.3f / m : 1.f;
    const float sT = fabsf(dT) > 0.5f * T ? 0.5f * T / fabsf(dT) : 1.f;
    const float sc = fminf(sa, sT);
    al = al + sc * da;
    be = be + sc * db;
    T = T + sc * dT;
    // geodesics much longer than the straight segment are not pursued
    return T <= 4.f * sqrtf(P.gdd(A, L - P.q)) + 1.f;
}

// Angle displacement of the finite-difference shots.
constexpr float ILLUM_EPS = 1e-3f;

// Kinds whose shots walk no list of bumps: a step is one instruction stream, and
// waves that share a SIMD slow each other.
template <int KIND> constexpr bool cheap_steps = !bump_cull<KIND> && !is_deform(KIND);

// Waves per CU that a short list is spread over: two per SIMD, one for the kinds of cheap
// steps.  With a bump walk the line is flat: a 1080p frame takes 283, 281, 280,
// 272, 272 and 278 ms at 512, 768, 1024, 1536, 2048 and 4096 (before
// k_illum_rows), for its time is the longest chain.  The 160x104 quadric takes 58,
// 65 and 95 ms at 1024, 2048 and 4096, the twist 10.1, 12.3 and 17.7.
constexpr int SOLVE_WAVES = 8;
template <int KIND> __device__ __forceinline__ int solve_waves(const rti::IllumArgs &A) {
    return A.n_cu * (cheap_steps<KIND> ? SOLVE_WAVES / 2 : SOLVE_WAVES);
}

// Lists of the kinds of cheap steps longer than this are bound by issue, not by
// their longest chain: k_illum_solve then takes one iteration and packs the pixels
// that go on into the next list, and the continuation stops at each target, so
// that waves stay full (the 420x405 quadric: 81 ms, and 94 with each pixel solved
// to its end; 77 before there was such a launch).  Kinds with a bump walk are
// faster solved to the end at any length (431x401: 16 anisotropic bumps 143 ms, 189
// packed; 16 isotropic ones 56 and 75; 16 deformations 53 and 66).
constexpr int PACK_ABOVE = 64;
template <int KIND> __device__ __host__ __forceinline__ bool packs(const rti::IllumArgs &A, int64_t n) {
    return cheap_steps<KIND> && n > A.n_cu * PACK_ABOVE;
}

// Pixels per CU that k_illum_rows takes, one per wave: four waves per SIMD.  1080p with
// 16 bumps takes 245, 240, 235 and 248 ms at 1024, 2048, 4096 and 8192; frames
// of 3 to 90 thousand pixels change by 1% to 15% in the same order.
constexpr int ROWS_MAX = 16;
__device__ __host__ __forceinline__ int rows_max(const rti::IllumArgs &A) { return A.n_cu * ROWS_MAX; }

// Blocks of four waves that hold any short list of a frame of n pixels, and
// SOLVE_WAVES waves per CU.
inline int solve_blocks(const rti::IllumArgs &A, int64_t n) {
    return (int)std::max<int64_t>(A.n_cu * SOLVE_WAVES / 4,
                                  (std::min<int64_t>(n, short_list(A)) + 4 * PAR_PIX - 1) / (4 * PAR_PIX));
}

// What the shots of iteration it of a pixel lead to: the iterations done if it
// goes on (-1: none, at the next target of the continuation), else 0.  through:
// a pixel that converges at a target of the continuation goes on to the next.
template <int KIND>
__device__ __forceinline__ int advance(const rti::IllumArgs &A, const Pixel<KIND> &P, V3<float> L, int it, bool okab,
                                       V3<float> X, V3<float> Y, V3<float> Xa, V3<float> Xb, float &al, float &be,
                                       float &T, float &last, float &cont, int &code, int *status, bool through = true) {
    const V3<float> Lp = target(cont, P, L);
    const V3<float> F = X - Lp;
    const int j = assess(A, it, F, last);
    if (j == J_STEP) {
        if (okab && newton<KIND>(A, P, Lp, ILLUM_EPS, al, be, T, F, X, Y, Xa, Xb) && it + 1 < A.max_iters) return it + 1;
    } else if (j == J_CONV && code == ST_CONT && through) {
        // the next stage of the continuation starts from here
        const int st = (int)(cont * rti::ILLUM_CONT_STAGES + 0.5f);
        const float lam0 = (float)st / rti::ILLUM_CONT_STAGES, lam1 = (float)(st + 1) / rti::ILLUM_CONT_STAGES;
        T *= lam1 / lam0;
        last = __builtin_huge_valf();
        cont = lam1;
        code = st + 1 < rti::ILLUM_CONT_STAGES ? ST_CONT : ST_CONV;
        return -1;
    } else if (j == J_CONV) {
        *status = code;
    }
    return 0;
}

// A short list[it & 1]: the pixels' remaining iterations, each pixel on its
// own (one iteration where packs(n_in)); the launches that follow find their lists
// empty.  Lanes 3j, 3j+1, 3j+2
// of a wave shoot the base and the two displaced directions of pixel j side by
// side; lane 3j tests the residual, takes the Newton step and hands the new state to its
// neighbours.  During the continuation a pixel that converges goes on to the
// next stage's target at once.  A shot is a serial chain of up to thousands of
// steps, so a launch per iteration lasted as long as its longest shot, and the
// sum of those maxima was most of the time; here a pixel's time is the sum of
// its own shots.  Same values as the launches one by one.
// rows: k_illum_rows follows; lists of up to rows_max pixels are left to it
// whole, and of a longer list the last rows_max pixels to be solved (their
// state in w_X and the arrays of the state).
template <int KIND, bool ONE>
__global__ __launch_bounds__(256) void k_illum_solve(rti::IllumArgs A, const float4 *__restrict__ BF, int it, bool rows) {
    const int *in = A.list[it & 1];
    const int n_in = A.ctr[it];
    if (n_in > short_list(A) || (rows && n_in <= rows_max(A))) return;
    int *done = A.ctr + 2 * (A.max_iters + 1) + it, *handed = A.ctr + 3 * (A.max_iters + 1) + it;
    const uint64_t all = all_bumps(A.n_bumps);
    const V3<float> L = mk(A.light[0], A.light[1], A.light[2]);
    const float eps = ILLUM_EPS;
    const int lane = lane_id(), role = lane % 3, src = lane - role;
    const int per_wave = min(PAR_PIX, max(1, (n_in + solve_waves<KIND>(A) - 1) / solve_waves<KIND>(A)));
    const bool through = !packs<KIND>(A, (int64_t)A.n_sets * A.width * A.height);
    const int base = (blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6)) * per_wave;
    if (base >= n_in) return;
    const int k = base + lane / 3;
    bool live = lane < 3 * per_wave && k < n_in;
    int pix = 0;
    float al = 0.f, be = 0.f, T = 0.f, last = 0.f, cont = A.cont;
    int code = A.conv_code;
    Pixel<KIND> P{};
    P.Bs = BF;  // (idle lanes: any table)
    if (live) {
        pix = in[k];
        P = pixel<KIND, ONE>(A, BF, pix);
        al = A.w_al[pix];
        be = A.w_be[pix];
        T = A.w_T[pix];
        last = A.w_F[pix];
    }
    while (ballot(live)) {
        bool ok = false;
        V3<float> X = mk(0.f, 0.f, 0.f), Y = X;
        V3<float> v = X;
        if (live) v = P.dir(A, role == 1 ? al + eps : al, role == 2 ? be + eps : be);
        IAcc<KIND> acc{P.Bs, all, A.twist_amp, A.twist_theta0, nullptr, nullptr};
        ok = shoot<KIND>(acc, A, live, P.q, v, T, X, Y);
        // the displaced shots to lane 3j
        const int s1 = min(lane + 1, 63), s2 = min(lane + 2, 63);
        const V3<float> Xa = mk(__shfl(X.x, s1), __shfl(X.y, s1), __shfl(X.z, s1));
        const V3<float> Xb = mk(__shfl(X.x, s2), __shfl(X.y, s2), __shfl(X.z, s2));
        const int oka = __shfl((int)ok, s1), okb = __shfl((int)ok, s2);
        int next = 0;  // iterations done if the pixel goes on, else 0
        if (live && role == 0) {
            if (ok) next = advance<KIND>(A, P, L, it, oka && okb, X, Y, Xa, Xb, al, be, T, last, cont, code, A.status + pix, through);
            // a pixel that ends, also by a failed shot, leaves the state of its last step
            if (next == 0) {
                A.w_al[pix] = al;
                A.w_be[pix] = be;
                A.w_T[pix] = T;
                A.w_F[pix] = last;
            }
        }
        next = __shfl(next, src);
        al = __shfl(al, src);
        be = __shfl(be, src);
        T = __shfl(T, src);
        const int ended = __popcll(ballot(live && role == 0 && next == 0));
        live = live && next != 0;
        if (packs<KIND>(A, n_in)) {
            if (live && role == 0) {
                A.w_al[pix] = al;
                A.w_be[pix] = be;
                A.w_T[pix] = T;
                A.w_F[pix] = last;
            }
            append(A.list[(it + 1) & 1], A.ctr + it + 1, pix, live && role == 0);
            return;
        }
        it = max(next, 0);
        if (rows) {
            int left = 0;
            if (lane == 0) {
                left = n_in - ended -
                       (ended ? atomicAdd(done, ended) : __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
            if (uniform_i(left) <= rows_max(A)) {
                if (live && role == 0) {
                    A.w_al[pix] = al;
                    A.w_be[pix] = be;
                    A.w_T[pix] = T;
                    A.w_F[pix] = last;
                    A.w_X[3 * pix] = __int_as_float(it);
                    A.w_X[3 * pix + 1] = cont;
                    A.w_X[3 * pix + 2] = __int_as_float(code);
                }
                append(A.list[2], handed, pix, live && role == 0);
                return;
            }
        }
    }
}

// The pixels of a list of up to rows_max, or those that k_illum_solve handed
// over, to their end: one wave per pixel, its three shots on three rows of 16
// lanes (the fourth repeats the base), the bumps spread over the lanes of each
// row.  What is left there are serial chains of up to 50 shots of hundreds of
// steps, whose latency is the time: with the walk of the bumps in every lane
// 2.4 to 5 us a step even on an idle GPU, spread over the lanes about 1 us.
// 1080p with 16 bumps 270 ms without these launches, 235 with them; 72x48 with
// 13 bumps 90 and 36.  Same values as the other launches.
template <int NB, bool ONE>
__global__ __launch_bounds__(64) void k_illum_rows(rti::IllumArgs A, const float4 *__restrict__ BF, int it) {
    const int n_in = A.ctr[it];
    if (n_in > short_list(A)) return;
    const bool whole = n_in <= rows_max(A);
    const int n = whole ? n_in : min(A.ctr[3 * (A.max_iters + 1) + it], rows_max(A));
    const int k = blockIdx.x;
    if (k >= n) return;
    const int lane = lane_id(), role = lane >> 4;
    const V3<float> L = mk(A.light[0], A.light[1], A.light[2]);
    const int pix = uniform_i(whole ? A.list[it & 1][k] : A.list[2][k]);
    const Pixel<KIND_GRAPH> P = pixel<KIND_GRAPH, ONE>(A, BF, pix);
    float4 b0[NB], b1[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int b = (lane & 15) + 16 * j;
        b0[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        b1[j] = make_float4(0.f, 0.f, -1.f, 1.f);
        if (b < A.n_bumps) b0[j] = P.Bs[2 * b], b1[j] = P.Bs[2 * b + 1];
    }
    float al = A.w_al[pix], be = A.w_be[pix], T = A.w_T[pix], last = A.w_F[pix], cont = A.cont;
    int code = A.conv_code;
    if (!whole) {
        it = __float_as_int(A.w_X[3 * pix]);
        cont = A.w_X[3 * pix + 1];
        code = __float_as_int(A.w_X[3 * pix + 2]);
    }
    for (;;) {
        V3<float> X, Y;
        const V3<float> v = P.dir(A, role == 1 ? al + ILLUM_EPS : al, role == 2 ? be + ILLUM_EPS : be);
        const uint64_t ok = ballot(shoot_rows<NB>(b0, b1, A, P.q, v, T, X, Y));
        if (!(ok & 1ull)) break;
        const V3<float> Xa = mk(__shfl(X.x, 16), __shfl(X.y, 16), __shfl(X.z, 16));
        const V3<float> Xb = mk(__shfl(X.x, 32), __shfl(X.y, 32), __shfl(X.z, 32));
        X = mk(__shfl(X.x, 0), __shfl(X.y, 0), __shfl(X.z, 0));
        Y = mk(__shfl(Y.x, 0), __shfl(Y.y, 0), __shfl(Y.z, 0));
        const bool okab = ((ok >> 16) & (ok >> 32) & 1ull) != 0;
        const int next = uniform_i(
            advance<KIND_GRAPH>(A, P, L, it, okab, X, Y, Xa, Xb, al, be, T, last, cont, code, A.status + pix));
        if (next == 0) break;
        it = max(next, 0);
    }
    if (lane == 0) {
        A.w_al[pix] = al;
        A.w_be[pix] = be;
        A.w_T[pix] = T;
        A.w_F[pix] = last;
    }
}

// One Newton iteration for every pixel of list[it & 1]: shoot; converged
// pixels are marked, the others take a damped step and move to the next list.
// While the list fills the grid, the iteration runs in two launches: here a
// lane shoots the base direction of one pixel, and a pixel that is due a
// step keeps its end point and velocity and goes to the step list, whose
// displaced shots k_illum_step takes two lanes per pixel; so lanes whose
// pixel converged do not wait on the displaced shots of their neighbours.
// A short list may have been solved by k_illum_solve before (solved: leave it).
// Both ways compute the same values.
template <int KIND, bool ONE>
__global__ __launch_bounds__(256) void k_illum_iter(rti::IllumArgs A, const float4 *__restrict__ BF, int it, bool solved) {
    const int *in = A.list[it & 1];
    const int n_in = A.ctr[it];
    const uint64_t all = all_bumps(A.n_bumps);
    const V3<float> L = mk(A.light[0], A.light[1], A.light[2]);
    if (solved && n_in <= short_list(A)) return;
    int *steps = A.list[2];
    for (int base = blockIdx.x * blockDim.x; base < n_in; base += gridDim.x * blockDim.x) {
        const int k = base + threadIdx.x;
        const bool act = k < n_in;
        bool due = false;
        int pix = 0;
        Pixel<KIND> P{};
        P.Bs = BF;
        V3<float> X = mk(0.f, 0.f, 0.f), Y = X, v = X;
        float T = 0.f;
        if (act) {
            pix = in[k];
            P = pixel<KIND, ONE>(A, BF, pix);
            T = A.w_T[pix];
            v = P.dir(A, A.w_al[pix], A.w_be[pix]);
        }
        IAcc<KIND> acc{P.Bs, all, A.twist_amp, A.twist_theta0, nullptr, nullptr};
        const bool ok = shoot<KIND>(acc, A, act, P.q, v, T, X, Y);
        if (act) {
            int j = J_STALL;
            if (ok) {
                float last = A.w_F[pix];
                j = assess(A, it, X - target(A.cont, P, L), last);
                A.w_F[pix] = last;
                if (j == J_CONV) A.status[pix] = A.conv_code;
            }
            if (j == J_STEP) {
                A.w_X[3 * pix] = X.x;
                A.w_X[3 * pix + 1] = X.y;
                A.w_X[3 * pix + 2] = X.z;
                A.w_Y[3 * pix] = Y.x;
                A.w_Y[3 * pix + 1] = Y.y;
                A.w_Y[3 * pix + 2] = Y.z;
                due = true;
            }
        }
        append(steps, A.ctr + A.max_iters + 1 + it, pix, due);
    }
}

// Second launch of a full-grid iteration: for every pixel of the step list,
// lanes 2j and 2j+1 shoot the two displaced directions of pixel j, and lane
// 2j takes the Newton step from them and the stored base shot.
template <int KIND, bool ONE>
__global__ __launch_bounds__(256) void k_illum_step(rti::IllumArgs A, const float4 *__restrict__ BF, int it) {
    const int *steps = A.list[2];
    int *out = A.list[(it + 1) & 1];
    const int n_st = A.ctr[A.max_iters + 1 + it];
    const uint64_t all = all_bumps(A.n_bumps);
    const V3<float> L = mk(A.light[0], A.light[1], A.light[2]);
    const float eps = ILLUM_EPS;
    const int lane = lane_id(), role = lane & 1;
    const int per_block = blockDim.x / 2;
    for (int base = blockIdx.x * per_block; base < n_st; base += gridDim.x * per_block) {
        const int k = base + (threadIdx.x >> 1);
        const bool act = k < n_st;
        bool again = false;
        int pix = 0;
        V3<float> Xs = mk(0.f, 0.f, 0.f), Ys = Xs, v = Xs;
        float al = 0.f, be = 0.f, T = 0.f;
        Pixel<KIND> P{};
        P.Bs = BF;
        if (act) {
            pix = steps[k];
            P = pixel<KIND, ONE>(A, BF, pix);
            al = A.w_al[pix];
            be = A.w_be[pix];
            T = A.w_T[pix];
            v = P.dir(A, role == 0 ? al + eps : al, role == 1 ? be + eps : be);
        }
        IAcc<KIND> acc{P.Bs, all, A.twist_amp, A.twist_theta0, nullptr, nullptr};
        const bool ok = shoot<KIND>(acc, A, act, P.q, v, T, Xs, Ys);
        // the beta shot of lane 2j+1 to lane 2j
        const int src = lane | 1;
        const V3<float> Xb = mk(__shfl(Xs.x, src), __shfl(Xs.y, src), __shfl(Xs.z, src));
        const int okb = __shfl((int)ok, src);
        if (act && role == 0 && ok && okb) {
            const V3<float> X = mk(A.w_X[3 * pix], A.w_X[3 * pix + 1], A.w_X[3 * pix + 2]);
            const V3<float> Y = mk(A.w_Y[3 * pix], A.w_Y[3 * pix + 1], A.w_Y[3 * pix + 2]);
            const V3<float> Lp = target(A.cont, P, L);
            again = newton<KIND>(A, P, Lp, eps, al, be, T, X - Lp, X, Y, Xs, Xb);
            A.w_al[pix] = al;
            A.w_be[pix] = be;
            A.w_T[pix] = T;
        }
        append(out, A.ctr + it + 1, pix, again);
    }
}

// Lambert term and visibility for the converged pixels; every hit pixel
// gets its direction and length.
template <int KIND, bool ONE>
__global__ __launch_bounds__(256) void k_illum_finish(rti::IllumArgs A, const float4 *__restrict__ BF,
                                                      const float4 *__restrict__ SPH, const float4 *__restrict__ PLN,
                                                      const float *__restrict__ TOR) {
    const int64_t n = pixel_count(A);
    const uint64_t all = all_bumps(A.n_bumps);
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        const int pix = nth_pixel(A, t);
        if (pix < 0) continue;
        int status = A.status[pix];
        if (status == ST_NOHIT) {
            if (A.dir) A.dir[3 * pix] = A.dir[3 * pix + 1] = A.dir[3 * pix + 2] = 0.f;
            if (A.len) A.len[pix] = 0.f;
            continue;
        }
        const Pixel<KIND> P = pixel<KIND, ONE>(A, BF, pix);
        const float T = A.w_T[pix];
        const V3<float> v = P.dir(A, A.w_al[pix], A.w_be[pix]);
        float shade = 0.f;
        if (status == ST_CONV) {
            // Lambert term in the metric: grad F . v / sqrt(grad F^T g^-1 grad F)
            const V3<float> gF = obj_grad(A.id[pix], P.q, A.n_spheres, A.n_planes, SPH, PLN, TOR);
            float G[9];
            const V3<float> E[3] = {mk(1.f, 0.f, 0.f), mk(0.f, 1.f, 0.f), mk(0.f, 0.f, 1.f)};
            for (int i = 0; i < 3; ++i) G[4 * i] = P.gdd(A, E[i]);
            for (int i = 0; i < 3; ++i)
                for (int j = i + 1; j < 3; ++j)
                    G[3 * i + j] = G[3 * j + i] = 0.5f * (P.gdd(A, E[i] + E[j]) - G[4 * i] - G[4 * j]);
            const float a0 = G[4] * G[8] - G[5] * G[7], a1 = G[2] * G[7] - G[1] * G[8], a2 = G[1] * G[5] - G[2] * G[4];
            const float a4 = G[0] * G[8] - G[2] * G[6], a5 = G[2] * G[3] - G[0] * G[5], a8 = G[0] * G[4] - G[1] * G[3];
            const float gdet = G[0] * a0 + G[1] * (G[5] * G[6] - G[3] * G[8]) + G[2] * (G[3] * G[7] - G[4] * G[6]);
            // grad F^T adj(G) grad F / det (adj(G) is symmetric for symmetric G)
            const float qf = (gF.x * (a0 * gF.x + a1 * gF.y + a2 * gF.z) + gF.y * (a1 * gF.x + a4 * gF.y + a5 * gF.z) +
                              gF.z * (a2 * gF.x + a5 * gF.y + a8 * gF.z)) / gdet;
            const float c = dot(gF, v) * rsqrt_(qf);
            IAcc<KIND> acc{P.Bs, all, A.twist_amp, A.twist_theta0, nullptr, nullptr};
            if (!(c > 0.f)) {
                status = ST_AWAY;
            } else if (reaches<KIND>(acc, P.q, v, T, 1e-3f, A, SPH, PLN, TOR)) {
                status = ST_LIT;
                shade = fminf(c, 1.f);
            } else {
                status = ST_BLOCKED;
            }
        }
        A.status[pix] = status;
        A.shade[pix] = shade;
        if (A.dir) {
            A.dir[3 * pix] = v.x;
            A.dir[3 * pix + 1] = v.y;
            A.dir[3 * pix + 2] = v.z;
        }
        if (A.len) A.len[pix] = T;
    }
}

__global__ void k_illum_zero(int *ctr, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) ctr[i] = 0;
}

// Retry seeds.  A hit pixel left without a geodesic (its Newton iteration
// from the straight segment stalled, failed or ran out of iterations)
// starts again from the converged direction of a neighbour: of the 8
// neighbouring pixels of the same parameter set that have converged, the
// one whose hit point is nearest, its direction written in this pixel's
// frame (angles about the straight direction to the light) and its length.
// Reads only converged pixels and writes only unconverged ones.
template <int KIND, bool ONE>
__global__ __launch_bounds__(256) void k_illum_seed(rti::IllumArgs A, const float4 *__restrict__ BF, int *ctr) {
    const int HW = A.width * A.height;
    const int64_t n = pixel_count(A);
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
        const int pix = nth_pixel(A, base + threadIdx.x);
        bool take = false;
        if (pix >= 0 && A.status[pix] == ST_NONE) {
            const int set = pix / HW, r = pix - set * HW, j = r / A.width, i = r - j * A.width;
            const V3<float> q = mk(A.hit[3 * pix], A.hit[3 * pix + 1], A.hit[3 * pix + 2]);
            int best = -1;
            float bestd = __builtin_huge_valf();
            for (int dj = -1; dj <= 1; ++dj)
                for (int di = -1; di <= 1; ++di) {
                    const int ii = i + di, jj = j + dj;
                    if ((di == 0 && dj == 0) || ii < 0 || jj < 0 || ii >= A.width || jj >= A.height) continue;
                    const int nb = set * HW + jj * A.width + ii;
                    if (A.status[nb] != ST_CONV) continue;
                    const V3<float> d = mk(A.hit[3 * nb], A.hit[3 * nb + 1], A.hit[3 * nb + 2]) - q;
                    const float d2 = dot(d, d);
                    if (d2 < bestd) {
                        bestd = d2;
                        best = nb;
                    }
                }
            if (best >= 0) {
                const Pixel<KIND> P = pixel<KIND, ONE>(A, BF, pix), Q = pixel<KIND, ONE>(A, BF, best);
                const V3<float> v = Q.dir(A, A.w_al[best], A.w_be[best]);
                const float c = dot(v, P.F.e0);
                if (c > 1e-2f * sqrt_(dot(v, v))) {
                    const float ic = 1.f / c;
                    A.w_al[pix] = dot(v, P.F.e1) * ic;
                    A.w_be[pix] = dot(v, P.F.e2) * ic;
                    A.w_T[pix] = A.w_T[best];
                    A.w_F[pix] = __builtin_huge_valf();
                    take = true;
                }
            }
        }
        append(A.list[0], ctr, pix, take);
    }
}

// Continuation stage: targets move from q + lam0 (L - q) to q + lam1 (L - q).
// lam0 = 0: every hit pixel still without a geodesic starts from the
// straight segment to the first target; otherwise the pixels that converged
// at lam0 (ST_CONT) start from that solution, the length scaled.
template <int KIND, bool ONE>
__global__ __launch_bounds__(256) void k_illum_cont(rti::IllumArgs A, const float4 *__restrict__ BF, int *ctr,
                                                    float lam0, float lam1) {
    const int64_t n = pixel_count(A);
    const V3<float> L = mk(A.light[0], A.light[1], A.light[2]);
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += gridDim.x * blockDim.x) {
        const int pix = nth_pixel(A, base + threadIdx.x);
        bool take = false;
        if (pix >= 0) {
            const int st = A.status[pix];
            if (lam0 == 0.f && st == ST_NONE) {
                const Pixel<KIND> P = pixel<KIND, ONE>(A, BF, pix);
                A.w_al[pix] = 0.f;
                A.w_be[pix] = 0.f;
                A.w_T[pix] = lam1 * sqrtf(P.gdd(A, L - P.q));
                take = true;
            } else if (lam0 > 0.f && st == ST_CONT) {
                A.w_T[pix] *= lam1 / lam0;
                take = true;
            }
            if (take) {
                A.status[pix] = ST_NONE;
                A.w_F[pix] = __builtin_huge_valf();
            }
        }
        append(A.list[0], ctr, pix, take);
    }
}

template <int KIND, bool ONE>
void illum_rounds(const rti::IllumArgs &a, const rti::DeviceData &d, int grid, hipStream_t s) {
    const int sgrid = solve_blocks(a, (int64_t)a.n_sets * a.width * a.height);
    const int rgrid = (int)std::min<int64_t>((int64_t)a.n_sets * a.width * a.height, rows_max(a));
    const bool rows = KIND == KIND_GRAPH && a.n_bumps > 0 && a.n_bumps <= 32;
    const bool packed = packs<KIND>(a, (int64_t)a.n_sets * a.width * a.height);
    // one iteration's launches; solve: the pixels of a short list go to their end
    auto iteration = [&](const rti::IllumArgs &q, int it, bool solve) {
        if (solve) hipLaunchKernelGGL((k_illum_solve<KIND, ONE>), dim3(sgrid), dim3(256), 0, s, q, d.bump_f, it, rows);
        if constexpr (KIND == KIND_GRAPH) {
            if (solve && rows && a.n_bumps <= 16)
                hipLaunchKernelGGL((k_illum_rows<1, ONE>), dim3(rgrid), dim3(64), 0, s, q, d.bump_f, it);
            else if (solve && rows)
                hipLaunchKernelGGL((k_illum_rows<2, ONE>), dim3(rgrid), dim3(64), 0, s, q, d.bump_f, it);
        }
        hipLaunchKernelGGL((k_illum_iter<KIND, ONE>), dim3(grid), dim3(256), 0, s, q, d.bump_f, it, solve);
        hipLaunchKernelGGL((k_illum_step<KIND, ONE>), dim3(grid), dim3(256), 0, s, q, d.bump_f, it);
    };
    for (int it = 0; it < a.max_iters; ++it) iteration(a, it, true);
    // retries from converged neighbours, a quarter of the iterations each (a
    // seed from a neighbour is close: 1080p 432 -> 390 ms for 99.88 -> 99.83%
    // of the hits found, the quadric unchanged); each round has its own
    // counters
    rti::IllumArgs r = a;
    r.max_iters = std::max(a.max_iters / 4, 1);
    for (int round = 1; round <= rti::ILLUM_RETRY_ROUNDS; ++round) {
        r.ctr = a.ctr + round * rti::illum_ctr_words(a.max_iters);
        hipLaunchKernelGGL((k_illum_seed<KIND, ONE>), dim3(grid), dim3(256), 0, s, r, d.bump_f, r.ctr);
        for (int it = 0; it < r.max_iters; ++it) iteration(r, it, it == 0 || packed);
    }
    // continuation in the light position for the pixels still unsolved, half
    // the iterations per stage (a quarter loses 15% of the quadric's hits)
    r.max_iters = std::max(a.max_iters / 2, 1);
    for (int st = 0; st < rti::ILLUM_CONT_STAGES; ++st) {
        const float lam0 = (float)st / rti::ILLUM_CONT_STAGES, lam1 = (float)(st + 1) / rti::ILLUM_CONT_STAGES;
        r.ctr = a.ctr + (1 + rti::ILLUM_RETRY_ROUNDS + st) * rti::illum_ctr_words(a.max_iters);
        r.cont = lam1;
        r.conv_code = st + 1 < rti::ILLUM_CONT_STAGES ? ST_CONT : ST_CONV;
        hipLaunchKernelGGL((k_illum_cont<KIND, ONE>), dim3(grid), dim3(256), 0, s, r, d.bump_f, r.ctr, lam0, lam1);
        for (int it = 0; it < r.max_iters; ++it) iteration(r, it, it == 0 || packed);
    }
    hipLaunchKernelGGL((k_illum_finish<KIND, ONE>), dim3(grid), dim3(256), 0, s, a, d.bump_f, d.sph_f, d.pln_f,
                       d.tor_f);
}

template <int KIND>
hipError_t illum_kind(const rti::IllumArgs &a, const rti::DeviceData &d, int grid, hipStream_t s) {
    hipLaunchKernelGGL(k_illum_zero, dim3(1), dim3(256), 0, s, a.ctr,
                       (1 + rti::ILLUM_RETRY_ROUNDS + rti::ILLUM_CONT_STAGES) * rti::illum_ctr_words(a.max_iters));
    hipLaunchKernelGGL((k_illum_init<KIND>), dim3(grid), dim3(256), 0, s, a, d.bump_f);
    if (a.n_sets == 1)
        illum_rounds<KIND, true>(a, d, grid, s);
    else
        illum_rounds<KIND, false>(a, d, grid, s);
    return hipGetLastError();
}

}  // namespace

namespace rti {

hipError_t launch_illum(const IllumArgs &a, const DeviceData &d, int grid, hipStream_t s) {
    switch (a.kind) {
#define RT_ILLUM(K) \
    case K: return illum_kind<K>(a, d, grid, s);
        RT_ILLUM(KIND_EUCLID)
        RT_ILLUM(KIND_GRAPH)
        RT_ILLUM(KIND_TWIST)
        RT_ILLUM(KIND_ZTWIST)
        RT_ILLUM(KIND_DEFORM)
        RT_ILLUM(KIND_DEFORM_ROT)
        RT_ILLUM(KIND_GANISO)
        RT_ILLUM(KIND_GQUAD)
#undef RT_ILLUM
    default: return hipErrorInvalidValue;
    }
}

}  // namespace rti
