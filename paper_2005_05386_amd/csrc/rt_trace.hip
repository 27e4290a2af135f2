// Geodesic trace kernels for gfx950.
//
// A trace is a short sequence of launches on one stream:
//   reset    zero the counter block and statistics (a fill kernel, so the
//            sequence stays valid inside a captured graph);
//   pass p   persistent waves pull 64-ray chunks from per-XCD atomic
//            counters and integrate each lane's ray for at most S accepted
//            steps; rays that neither hit nor terminated are compacted into
//            the other ray queue (per parameter set) for pass p+1, so every
//            pass starts with full waves;
//            A window that reaches no bump and no object is flown in closed
//            form (free flight), the others are marched in a loop of their
//            own that stops where some lane hits or fails;
//   refine   one lane per chord hit, in double precision: bisection of the
//            step fraction on the sign of the hit object's implicit function
//            along the partial step of the same integrator, then the output.
//
// Inside a pass, every K steps each wave computes the bounding box of its
// lanes' positions, grows it by the distance a unit-speed ray can cover in
// K+1 steps (g >= I for the graph metric and the 4K twist, so the Euclidean
// speed of a g-unit velocity is at most 1), and culls bumps (cut sphere
// cull_sigmas*sigma) and objects against it: lane i tests bump i / sphere
// 64w+i and a ballot turns the answers into wave-uniform masks.  Bump
// parameters for the masked bumps are then read with scalar loads.
#include <algorithm>
#include <mutex>

#include "rt.h"
#include "rt_device.hpp"
#include "rt_internal.hpp"
#include "rt_step.hpp"

using namespace rtd;
using rti::TraceArgs;

static_assert(rtd::DEFORM_F4 == rti::DEFORM_F4 && rtd::DEFORM_D == rti::DEFORM_D,
              "device and host deformation table strides differ");
static_assert(rtd::KIND_DEFORM_ROT == rti::KERNEL_KIND_DEFORM_ROT, "rotating deformation kind differs");

namespace {

// The output index is made opaque where it is used: otherwise the compiler
// hoists the nine per-lane output addresses (18 registers, loop invariant)
// out of the step loop, where they stay live through every step for a
// store that happens once per ray.
__device__ __forceinline__ void write_out(const TraceArgs &A, unsigned oi, V3<float> x, float t, V3<float> y, int id,
                                          int steps) {
    __asm__ volatile("" : "+v"(oi));
    A.out_hit[3 * oi + 0] = x.x;
    A.out_hit[3 * oi + 1] = x.y;
    A.out_hit[3 * oi + 2] = x.z;
    A.out_t[oi] = t;
    A.out_id[oi] = id;
    float n = rsqrt_(dot(y, y));
    A.out_dir[3 * oi + 0] = y.x * n;
    A.out_dir[3 * oi + 1] = y.y * n;
    A.out_dir[3 * oi + 2] = y.z * n;
    if (A.out_steps) A.out_steps[oi] = steps;
}

// Checkpoint c of ray id on the adjoint tape.
__device__ __forceinline__ void write_ckpt(const TraceArgs &A, int id, int c, V3<float> xh, V3<float> xl,
                                           V3<float> y) {
    float *ck = A.tape_ck + ((((int64_t)(id >> 6) * A.n_ckpt + c) * 9) * 64 + (id & 63));
    ck[0 * 64] = xh.x;
    ck[1 * 64] = xh.y;
    ck[2 * 64] = xh.z;
    ck[3 * 64] = xl.x;
    ck[4 * 64] = xl.y;
    ck[5 * 64] = xl.z;
    ck[6 * 64] = y.x;
    ck[7 * 64] = y.y;
    ck[8 * 64] = y.z;
}

// Refine record of a chord hit: 4 float4 (64 B) where t is steps * h and
// the hit step is h (RK4 and Euler without learned crossings), else 5
// (80 B: also t as two floats and the step size).
constexpr bool compact_record(int step, bool surr) { return step != STEP_RK45 && !surr; }

// Kinds and integrators with a small-launch variant of the pass kernel.
constexpr bool has_small_variant(int kind, int step) {
    return step != STEP_RK45 && kind != KIND_EUCLID && kind != KIND_ZTWIST;
}

// ========================================================= ray generation
// Initial state of a ray: x = eye, y = the pixel direction d scaled to unit
// length in the metric at the eye (y = d / sqrt(g(d, d))).  Computed by the
// first pass in registers, so the state makes no trip through memory.
template <int KIND>
__device__ __forceinline__ V3<float> initial_velocity(const TraceArgs &A, const float4 *__restrict__ Bs, int pi,
                                                      int pj) {
    float su = (2.0f * ((float)pi + 0.5f) / (float)A.width - 1.0f) * A.tan_half * A.aspect;
    float sv = (1.0f - 2.0f * ((float)pj + 0.5f) / (float)A.height) * A.tan_half;
    V3<float> d = mk(su * A.right[0] + sv * A.up[0] + A.fwd[0], su * A.right[1] + sv * A.up[1] + A.fwd[1],
                     su * A.right[2] + sv * A.up[2] + A.fwd[2]);
    d = rsqrt_(dot(d, d)) * d;
    const V3<float> e = mk(A.eye[0], A.eye[1], A.eye[2]);
    const float gdd = metric_gdd<KIND>(Bs, A.n_bumps, A.twist_amp, A.twist_theta0, e, d);
    return rsqrt_(gdd) * d;
}

// Batched segments: each lane's state at the start of a culling window, in
// LDS (read back only when the lane marches the window again).
__device__ __forceinline__ float4 *batch_save() {
    __shared__ float4 save[3 * 256];
    return save;
}

// ============================================================ free flight
// Kinds whose acceleration is exactly zero outside the bumps or deformations
// the wave has listed (the graph of a sum of bumps and a composition of local
// deformations are flat there).
constexpr bool flat_outside(int kind) {
    return kind == KIND_EUCLID || kind == KIND_GRAPH || kind == KIND_GANISO || is_deform(kind);
}
// The twist's acceleration vanishes in the computed arithmetic once
// rho >= TWIST_FREE: exp(-2 rho) < 2^-25 there, so tanh rho rounds to 1 and
// the sech^2 terms are exact zeros; what is left carries exp(-rho^2) < 2e-33
// times at most rho^3, |theta0| <= 1.5 and amp <= 1, and the z component is
// zero.  With |a| < 1e-27, a velocity component of at least TWIST_MIN_V is the
// same float after adding h a for any h < 1e4.
constexpr float TWIST_FREE = 8.7f, TWIST_MIN_V = 1e-15f;
// Distance from the box [mn, mx] of the wave's positions to the nearest cut
// region (twist: to the ball of radius TWIST_FREE) or object, rounded down; called by the whole wave.  Cut regions and
// tori are taken as balls about their centres.
template <int KIND>
__device__ __forceinline__ float free_distance(const TraceArgs &A, const float4 *__restrict__ Bs,
                                               const float4 *__restrict__ SPH, const float4 *__restrict__ PLN,
                                               const float *__restrict__ TOR, int lane, const float mn[3],
                                               const float mx[3]) {
    float gap = __builtin_huge_valf();
    if constexpr (KIND == KIND_TWIST) gap = sqrt_(box_dist2(0.f, 0.f, 0.f, mn, mx)) - TWIST_FREE;
    if (KIND != KIND_EUCLID && KIND != KIND_TWIST && lane < A.n_bumps) {
        const float4 *__restrict__ q = Bs + (is_deform(KIND) ? DEFORM_F4 : 2) * lane;
        const float4 b0 = q[0], b1 = q[1];
        float R;
        if constexpr (KIND == KIND_GRAPH) {
            R = sqrt_(b1.z);
        } else {
            // spread-scaled cut radius times the largest spread
            const float cut2 = is_deform(KIND) ? q[2].w : b1.w;
            R = sqrt_(cut2) * rsqrt_(fminf(fminf(b1.x, b1.y), b1.z));
        }
        gap = sqrt_(box_dist2(b0.x, b0.y, b0.z, mn, mx)) - R * 1.0001f;
    }
    for (int i = lane; i < A.n_spheres; i += 64) {
        const float4 s = SPH[i];
        gap = fminf(gap, sqrt_(box_dist2(s.x, s.y, s.z, mn, mx)) - s.w);
    }
    if (lane < A.n_planes) {
        const float4 pl = PLN[lane];
        const float c = pl.x * (mn[0] + mx[0]) + pl.y * (mn[1] + mx[1]) + pl.z * (mn[2] + mx[2]) - 2.f * pl.w;
        const float r = fabsf(pl.x) * (mx[0] - mn[0]) + fabsf(pl.y) * (mx[1] - mn[1]) + fabsf(pl.z) * (mx[2] - mn[2]);
        gap = fminf(gap, 0.5f * (fabsf(c) - r));
    }
    if (lane < A.n_tori) {
        const float *tp = TOR + 8 * lane;
        gap = fminf(gap, sqrt_(box_dist2(tp[0], tp[1], tp[2], mn, mx)) - (tp[6] + tp[7]));
    }
    return wave_min(gap) * 0.999f;
}

// ===================================================== segment versus scene
// First crossing of the chord [x, x + dx] with the listed objects (spheres
// sm, planes and tori om); p = xh + xl.  Updates (hit_s, hit_id) where a
// crossing comes before hit_s.
__device__ __forceinline__ void chord_scan(const uint64_t sm[4], uint64_t om, int ns, int np,
                                           const float4 *__restrict__ SPH, const float4 *__restrict__ PLN,
                                           const float *__restrict__ TOR, V3<float> xh, V3<float> xl, V3<float> p,
                                           V3<float> dx, float &hit_s, int &hit_id) {
    const float DD = dot(dx, dx);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint64_t m = sm[w];
        while (m) {
            int b = __builtin_ctzll(m);
            m &= m - 1;
            int idx = 64 * w + b;
            float4 s = SPH[idx];
            V3<float> o = mk((xh.x - s.x) + xl.x, (xh.y - s.y) + xl.y, (xh.z - s.z) + xl.z);
            float sc = sphere_chord(s, o, dx, DD);
            if (sc < hit_s) {
                hit_s = sc;
                hit_id = idx;
            }
        }
    }
    uint64_t m = om;
    while (m) {
        int b = __builtin_ctzll(m);
        m &= m - 1;
        float F0, F1;
        int oid;
        if (b < 8) {
            float4 pl = PLN[b];
            F0 = pl.x * p.x + pl.y * p.y + pl.z * p.z - pl.w;
            F1 = F0 + (pl.x * dx.x + pl.y * dx.y + pl.z * dx.z);
            oid = ns + b;
        } else {
            const float *tp = TOR + 8 * (b - 8);
            F0 = torus_sdf<float>(tp, p);
            F1 = torus_sdf<float>(tp, p + dx);
            oid = ns + np + (b - 8);
        }
        if ((F0 > 0.f) != (F1 > 0.f)) {
            float sc = fminf(fmaxf(F0 / (F0 - F1), 0.f), 1.f);
            if (sc < hit_s) {
                hit_s = sc;
                hit_id = oid;
            }
        }
    }
}

// ================================================================ the pass
// Occupancy: 7 waves per SIMD (at most 72 VGPRs) measured fastest for the
// RK4 graph and twist kernels, 6 for DP5(4) and for rotating deformations
// (77.5 -> 72.2 ms per 1080p frame), although long-lived values spill (the
// spills are a small share of the instructions).
// SURR: learned crossings (graph metric, RK4, one parameter set): a ray whose
// step chord enters the support sphere of an eligible bump stops on the
// sphere (the partial step is committed, its fraction of h added to t) and
// is queued for the crossing stage that runs after the pass.
// TAPE: differentiation forward (graph metric, RK4): checkpoints of the
// state every ckpt_every steps; a separate instantiation, so that the plain
// trace carries no per-step checkpoint test.
#ifndef RT_PASS_WAVES
#define RT_PASS_WAVES 7  // waves per SIMD the RK4 and Euler pass kernels are compiled for
#endif
#ifndef RT_GRAPH_WAVES
#define RT_GRAPH_WAVES 8  // the same for the isotropic graph metric, plain and taped (64 registers, no spill in the step loop)
#endif
#ifndef RT_TWIST_WAVES
#define RT_TWIST_WAVES 6  // the twist (4K frame 198.2 / 197.7 / 205.3 / 203.2 ms at 7 / 6 / 5 / 4)
#endif
#ifndef RT_BATCH_WAVES
#define RT_BATCH_WAVES 6  // the same for the batched-segment variant
#endif
#ifndef RT_LAT_WAVES
#define RT_LAT_WAVES 4  // the same for the small-launch variant
#endif
// LAT: the variant for passes of few chunks (fixed steps; at most
// lat_chunks, see the line's rule where it is set).  A wave alone on its SIMD
// issues a vector instruction every 5 to 6 cycles and waits out every scalar
// load, so what counts is the length of its own instruction stream: one or two
// listed bumps stay in registers for the whole window, more are read from the
// wave's list in LDS four at a time.  128 registers, no spills.  Against the
// walk (start of this design, then with free flight and the march below, then
// this): 64x64, one bump 1.25 / 1.09 / 0.91 ms; 86x84, 61 bumps 16.1 / 17.4 /
// 11.3 ms; 721x403, 12 anisotropic bumps 20.3 / 19.2 / 18.2 ms.  The other
// kinds only gain the registers (473x458 twist 8.0 / 6.7 / 6.1 ms, 206x192
// deformations 2.7 / 1.03 / 0.99 ms).  In launches
// that fill the SIMDs the walk is faster (the list's padding and register
// copies are issue slots), so those keep it.
// BATCH: batched multi-segment intersection (Sec. 4.1 proposes testing many
// segments of the polygon at once).  A culling window's K steps are first
// marched with no scene test while each lane keeps the bounding box of its
// polygon; the boxes, grown by a rounding margin, are then tested against
// the window's object lists.  If no lane's box meets an object the K steps
// stand; otherwise the lanes whose box does return to the window's start and
// march it again with the per-step chord tests, while the other lanes wait.
// A lane that ends by a miss or a failure while marching writes its output
// only once its box is cleared.  Windows and object lists only bound the
// work, so the outputs equal the plain kernel's bit for bit.
// FLY: free flight.  Adaptive traces of more than FLY_DEFORMS deformations do
// without: there its block keeps some 35 more scalars alive, which spill to vector
// registers inside the step loop, and few windows are empty (1280x720, RK45, with and
// without: 16 deformations 14.6-19.5 and 13.5-18.0 ms, 12 7.3-12.8 and 7.3-11.5, 8
// 5.1-6.5 and 5.9-6.8, 2 2.5-3.0 and 4.6-4.9).
constexpr int FLY_DEFORMS = 8;
constexpr bool few_fly(int kind, int step) { return is_deform(kind) && step == STEP_RK45; }
// Waves per SIMD a pass kernel is compiled for (adaptive steps: 6; flying between
// deformations 7.2 and 7.6 ms at 5 and 6 for nine of them, rotating ones 8.3 and 9.0
// flying, 15.7 and 17.4 for sixteen not flying).
constexpr int rk45_waves(int kind, bool fly) { return few_fly(kind, STEP_RK45) && (fly || kind == KIND_DEFORM_ROT) ? 5 : 6; }
// DENSE: isotropic tables of more than SPARSE_BUMPS.  Their windows list many
// bumps, of which few hold the window in their cut: the walk that tests every cut
// without asking (a select, no branch) is then faster from DENSE_WALK listed bumps
// on (48 bumps 1280x720 16.8-20.5 and 15.6-18.8 ms, 25 bumps 9.1-10.4 and 8.2-9.4, 20
// bumps 1000x700 4.1-8.3 and 4.1-7.6), while tables that seldom list so many pay for
// two loops (16 bumps 1920x1080 6.2-6.6 and 6.6-6.8, 17 bumps 7.2-8.8 and 7.5-8.8).
constexpr int SPARSE_BUMPS = 19, DENSE_WALK = 8;
constexpr bool has_dense(int kind, int step) { return kind == KIND_GRAPH && step != STEP_RK45; }
template <int KIND, int STEP, bool COUNT, bool SURR = false, bool TAPE = false, bool BATCH = false, bool LAT = false,
          bool FLY = true, bool DENSE = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LAT ? RT_LAT_WAVES : STEP == STEP_RK45 ? rk45_waves(KIND, FLY && !COUNT) : KIND == KIND_DEFORM_ROT ? 6 : (BATCH ? RT_BATCH_WAVES : (KIND == KIND_GRAPH && !SURR ? RT_GRAPH_WAVES : (KIND == KIND_TWIST ? RT_TWIST_WAVES : RT_PASS_WAVES))), 8))) void k_trace_pass(TraceArgs A, int pass, const float4 *__restrict__ BF,
                                                    const float4 *__restrict__ SPH,
                                                    const float4 *__restrict__ PLN,
                                                    const float *__restrict__ TOR) {
    static_assert(!BATCH || (STEP != STEP_RK45 && !COUNT && !SURR && !TAPE),
                  "batched segments: fixed-step integrators, plain trace");
    // t as two floats, the trial step and the attempt count change only
    // under DP5(4) and learned crossings; fixed-step traces derive t from the
    // step count and neither read nor keep them
    constexpr bool CARRY_T = STEP == STEP_RK45 || SURR;
    static_assert(!LAT || (has_small_variant(KIND, STEP) && !COUNT && !SURR && !BATCH),
                  "small-launch variant: fixed steps, plain and taped");
    constexpr bool LIST = LAT && (KIND == KIND_GRAPH || KIND == KIND_GANISO);
    float4 *list = nullptr;  // LIST: this wave's bump list
    if constexpr (LIST) {
        __shared__ float4 lists[4 * LIST_F4];
        list = lists + (threadIdx.x >> 6) * LIST_F4;
    }
    int groups = 0;  // LIST: its groups
    constexpr bool TIGHT = STEP != STEP_RK45 && !COUNT && !SURR && !BATCH;
    constexpr bool FLAT = FLY && flat_outside(KIND) && !COUNT && !SURR && !BATCH;
    constexpr bool FREE = FLAT || (KIND == KIND_TWIST && STEP != STEP_RK45 && !COUNT && !SURR && !BATCH);
    const int lane = lane_id();
    const int xcd0 = blockIdx.x % N_XCD;
    int *pass_ctr = A.ctr + rti::CTR_PASS0 + pass * rti::CTR_PASS_WORDS;
    const int HW = A.width * A.height;
    const int tiles = A.tiles_x * A.tiles_y;
    const int n_bumps = A.n_bumps, ns = A.n_spheres, np = A.n_planes, nt = A.n_tori;
    const int nsw = (ns + 63) >> 6;

    // chunk table of this pass: pass 0 walks every tile of every set; pass
    // p > 0 walks the sorted survivor list, each set padded to whole chunks
    int total_chunks, pre = 0, cnt = 0;
    if (pass == 0) {
        total_chunks = A.n_sets * tiles;
    } else {
        const int *surv = A.ctr + rti::CTR_PASS0 + (pass - 1) * rti::CTR_PASS_WORDS + rti::CTR_SURV;
        cnt = lane < A.n_sets ? surv[lane] : 0;
        pre = wave_incl_scan((cnt + 63) >> 6);
        total_chunks = uniform_i(__shfl(pre, 63));
    }
    // of the two variants of a later pass one takes it, by its chunk count
    if (A.lat_chunks > 0 && pass > 0 && (total_chunks <= A.lat_chunks) != LAT) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) pass_ctr[rti::CTR_NCH] = total_chunks;
    // no survivors (the late passes of a surrogate trace): nothing to pull,
    // count or write
    if (total_chunks == 0) return;
    const int *__restrict__ ids_in = A.ids[pass & 1];
    float *__restrict__ st = A.st;
    const int64_t cap = A.cap;

    unsigned long long st_wave = 0, st_lane = 0, st_bl = 0, st_ol = 0, st_steps = 0, st_rays = 0;
    unsigned long long st_ev = 0, st_be = 0, st_ot = 0;  // COUNT only
    unsigned long long st_bw = 0, st_br = 0;             // BATCH only: windows, replayed windows

    for (int xi = 0; xi < N_XCD; ++xi) {
        const int xp = (xcd0 + xi) & (N_XCD - 1);
        int *ctr = pass_ctr + xp * rti::CTR_CHUNK_STRIDE;
        for (;;) {
            int k = 0;
            if (lane == 0) k = atomicAdd(ctr, 1);
            k = uniform_i(__shfl(k, 0));
            const int chunk = k * N_XCD + xp;
            if (chunk >= total_chunks) break;

            // ---- resolve the set and this lane's ray id
            int set, id;
            bool valid;
            if (pass == 0) {
                set = chunk / tiles;
                id = chunk * 64 + lane;
                valid = true;
            } else {
                set = __popcll(ballot(pre <= chunk));
                int base_chunk = set > 0 ? __shfl(pre, set - 1) : 0;
                int cnt_s = __shfl(cnt, set);
                valid = (chunk - base_chunk) * 64 + lane < cnt_s;
                id = valid ? ids_in[chunk * 64 + lane] : 0;
            }
            set = uniform_i(set);
            // pixel of the ray: id = (set * tiles + tile) * 64 + lane-in-tile
            const int r = id - set * A.T;
            const int tile = r >> 6, tl_lane = r & 63;
            const int ty = tile / A.tiles_x, tx = tile - ty * A.tiles_x;
            const int pi = tx * 8 + (tl_lane & 7), pj = ty * 8 + (tl_lane >> 3);
            if (pass == 0) valid = pi < A.width && pj < A.height;
            const int pix = pj * A.width + pi;
            const float4 *__restrict__ Bs = BF + (int64_t)set * n_bumps * (is_deform(KIND) ? DEFORM_F4 : 2);
            const unsigned qbase = (unsigned)set * (unsigned)HW;

            V3<float> xh, xl, y;
            float th = 0.f, tl = 0.f, hc = A.h;
            int steps = 0, att = 0;
            int skip = -1;  // SURR only
            if (valid && pass == 0) {
                xh = mk(A.eye[0], A.eye[1], A.eye[2]);
                xl = mk(0.f, 0.f, 0.f);
                y = initial_velocity<KIND>(A, Bs, pi, pj);
            } else if (valid) {
                const float *__restrict__ src = st + ((int64_t)(id >> 6) * rti::Q_NFIELDS * 64 + (id & 63));
                auto F = [&](int f) { return src[f * 64]; };
                xh = mk(F(rti::Q_XH), F(rti::Q_XH + 1), F(rti::Q_XH + 2));
                xl = mk(F(rti::Q_XL), F(rti::Q_XL + 1), F(rti::Q_XL + 2));
                y = mk(F(rti::Q_Y), F(rti::Q_Y + 1), F(rti::Q_Y + 2));
                if constexpr (CARRY_T) {
                    th = F(rti::Q_TH);
                    tl = F(rti::Q_TL);
                    hc = F(rti::Q_H);
                    att = __float_as_int(F(rti::Q_ATT));
                }
                steps = __float_as_int(F(rti::Q_STEPS));
                if constexpr (SURR) skip = __float_as_int(F(rti::Q_SKIP));
            } else {
                xh = xl = y = mk(0.f, 0.f, 0.f);
            }
            if (pass == 0) st_rays += __popcll(ballot(valid));

            bool alive = valid;
            bool parked = false;  // SURR only
            int acc_pass = 0;
            int it = 0;
            uint64_t bmask = 0, omask = 0, emask = 0;
            uint64_t cutm = ~0ull;  // TIGHT: listed bumps whose cut some point of the window may be beyond
            int wend = 0;           // TIGHT: the iteration at which the window ends
            uint64_t sm[4] = {0, 0, 0, 0};
            V3<float> A0 = mk(0.f, 0.f, 0.f);
            bool need_a0 = true;
            unsigned c_eval = 0, c_bump = 0, c_obj = 0, lane_objs = 0;  // COUNT only
            // BATCH only: the window's marching or replaying state (wave-uniform
            // replay, wi, wlen), the lane's state at the window start, its
            // polygon box, and whether it waits or has an output pending
            bool replay = false, hold = false, inb = false;
            int wi = 0, wlen = 0, fin = 0, it_m = 0;
            V3<float> bmin = mk(0.f, 0.f, 0.f), bmax = bmin;

            // push chord hits to the refine queue (wave-aggregated); the lane's
            // registers still hold the state before the step
            auto push_hits = [&](bool hit, float hit_s, int hit_id, float hstep) {
                uint64_t hm = ballot(hit);
                if (hm) {
                    int base = 0;
                    if (lane == 0) base = atomicAdd(A.ctr + rti::CTR_REFINE, __popcll(hm));
                    base = uniform_i(__shfl(base, 0));
                    if (hit) {
                        int64_t r = base + mbcnt64(hm);
                        if constexpr (compact_record(STEP, SURR)) {
                            // t = steps h and the step is h: 4 float4
                            float4 *rec = A.rec + 4 * r;
                            rec[0] = make_float4(xh.x, xh.y, xh.z, xl.x);
                            rec[1] = make_float4(xl.y, xl.z, y.x, y.y);
                            rec[2] = make_float4(y.z, hit_s, __int_as_float(hit_id), __int_as_float((int)(qbase + pix)));
                            rec[3] = make_float4(__int_as_float(steps), __int_as_float((int)(uint32_t)bmask),
                                                 __int_as_float((int)(bmask >> 32)), 0.f);
                        } else {
                            float4 *rec = A.rec + rti::REC_F4 * r;
                            rec[0] = make_float4(xh.x, xh.y, xh.z, xl.x);
                            rec[1] = make_float4(xl.y, xl.z, y.x, y.y);
                            rec[2] = make_float4(y.z, th, hstep, hit_s);
                            rec[3] = make_float4(__int_as_float(hit_id), __int_as_float((int)(qbase + pix)),
                                                 __int_as_float(steps), tl);
                            rec[4] = make_float4(__int_as_float((int)(uint32_t)bmask),
                                                 __int_as_float((int)(bmask >> 32)), 0.f, 0.f);
                        }
                    }
                }
            };

            for (;;) {
                bool act = alive && (STEP == STEP_RK45 ? acc_pass < A.S : it < A.S) && !(SURR && parked);
                // batched: the pass length counts first marches only
                if constexpr (BATCH) act = alive && (replay ? (!hold && wi < wlen) : it_m < A.S);
                uint64_t am = ballot(act);
                if (am == 0) {
                    if constexpr (BATCH) {
                        // every replaying lane ended before the window did
                        if (replay) {
                            replay = false;
                            hold = false;
                            wi = 0;
                            continue;
                        }
                    }
                    break;
                }

                // ---- per-wave culling window
                int n_free = 0;  // steps that can be flown free from here
                if (BATCH ? (!replay && wi == 0) : (TIGHT ? it >= wend : it % A.K == 0)) {
                    if constexpr (TIGHT) wend = it + A.K;
                    // the lane id taken afresh: the table offsets derived from it
                    // are then formed in this block, once per window, instead of
                    // being hoisted out of the step loop and spilled (not in the
                    // batched variant, whose twist kernel then spilled inside its
                    // step loop and ran 1.6x slower)
                    int lane = lane_id();
                    if constexpr (!BATCH) __asm__ volatile("" : "+v"(lane));
                    V3<float> p = xh + xl;
                    if (A.cull_margin < 0.f) {
                        bmask = n_bumps >= 64 ? ~0ull : ((1ull << n_bumps) - 1ull);
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            int rem = ns - 64 * w;
                            sm[w] = rem >= 64 ? ~0ull : (rem > 0 ? ((1ull << rem) - 1ull) : 0ull);
                        }
                        omask = ((1ull << np) - 1ull) | (((1ull << nt) - 1ull) << 8);
                        if constexpr (SURR)
                            emask = ballot(lane < n_bumps && __float_as_int(A.surr_sb[2 * lane + 1].y) >= 0);
                    } else {
                        const float inf = __builtin_huge_valf();
                        const float pmn[3] = {wave_min(act ? p.x : inf), wave_min(act ? p.y : inf),
                                              wave_min(act ? p.z : inf)};
                        const float pmx[3] = {wave_max(act ? p.x : -inf), wave_max(act ? p.y : -inf),
                                              wave_max(act ? p.z : -inf)};
                        float m = A.cull_margin;
                        float disp = A.cull_disp;  // DEFORM: bound on |Phi(x) - x| in the window
                        if constexpr (is_deform(KIND)) {
                            // A geodesic is the preimage of a unit-speed line, so in the
                            // window it moves at most T + 2 max |Phi(x) - x|.  Deformation i
                            // moves a point q by |f_i(q)| |v_i| <= |a_i| |v_i| exp(-rho^2 / 2),
                            // rho the spread-scaled distance from q to c_i, and q is within
                            // the chain's displacement of the ray's point.  So a margin and
                            // a displacement bound that hold give, through the deformations
                            // near the box, a displacement bound and a margin that hold too;
                            // two rounds tighten both.
#pragma unroll
                            for (int round = 0; round < 2; ++round) {
                                const float lo0[3] = {pmn[0] - m, pmn[1] - m, pmn[2] - m};
                                const float hi0[3] = {pmx[0] + m, pmx[1] + m, pmx[2] + m};
                                float dl = 0.f;
                                if (lane < n_bumps) {
                                    const float rho = deform_box_rho(Bs + DEFORM_F4 * lane, lo0, hi0, disp);
                                    if (rho * rho <= Bs[DEFORM_F4 * lane + 2].w * 1.00001f) {
                                        // |f V| <= (|a||v| + |a||om| s_max max(rho, 1)) exp(-rho^2 / 2)
                                        // beyond spread-scaled distance rho
                                        const float4 d3 = Bs[DEFORM_F4 * lane + 3];
                                        dl = fmaf(d3.w, fmaxf(rho, 1.0f), d3.y) *
                                             exp2_(-0.5f * 1.44269504f * rho * rho);
                                    }
                                }
#pragma unroll
                                for (int o = 32; o >= 1; o >>= 1) dl += __shfl_xor(dl, o);
                                dl = __builtin_bit_cast(float, uniform_i(__builtin_bit_cast(int, dl))) * 1.001f;
                                disp = fminf(disp, dl);
                                m = fminf(m, A.cull_base + 2.0f * disp);
                            }
                        }
                        float lo[3], hi[3];
                        lo[0] = pmn[0] - m;
                        lo[1] = pmn[1] - m;
                        lo[2] = pmn[2] - m;
                        hi[0] = pmx[0] + m;
                        hi[1] = pmx[1] + m;
                        hi[2] = pmx[2] + m;
                        bool need = false, beyond = true;
                        float4 b0 = make_float4(0.f, 0.f, 0.f, 0.f), b1 = b0;
                        if (KIND == KIND_GRAPH && lane < n_bumps) {
                            b0 = Bs[2 * lane], b1 = Bs[2 * lane + 1];
                            need = box_dist2(b0.x, b0.y, b0.z, lo, hi) <= b1.z;
                            if constexpr (TIGHT) beyond = box_far2(b0.x, b0.y, b0.z, lo, hi) > b1.z * 0.9999f;
                        } else if (KIND == KIND_GANISO && lane < n_bumps) {
                            b0 = Bs[2 * lane], b1 = Bs[2 * lane + 1];
                            const float rho = aniso_box_rho(b0, b1, lo, hi);
                            need = rho * rho <= b1.w * 1.00001f;
                        } else if (is_deform(KIND) && lane < n_bumps) {
                            // the ball (in ray coordinates) where the deformation can act
                            const float rho = deform_box_rho(Bs + DEFORM_F4 * lane, lo, hi, disp);
                            need = rho * rho <= Bs[DEFORM_F4 * lane + 2].w * 1.00001f;
                        }
                        bmask = ballot(need);
                        if constexpr (LIST) groups = list_fill<KIND == KIND_GANISO>(list, bmask, need, b0, b1);
                        else if constexpr (TIGHT && KIND == KIND_GRAPH) cutm = ballot(beyond);
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            bool ns_need = false;
                            int idx = 64 * w + lane;
                            if (w < nsw && idx < ns) {
                                float4 s = SPH[idx];
                                ns_need = box_dist2(s.x, s.y, s.z, lo, hi) <= s.w * s.w;
                            }
                            sm[w] = w < nsw ? ballot(ns_need) : 0ull;
                        }
                        bool on = false;
                        if (lane < np) {
                            float4 pl = PLN[lane];
                            float cx = 0.5f * (lo[0] + hi[0]), cy = 0.5f * (lo[1] + hi[1]), cz = 0.5f * (lo[2] + hi[2]);
                            float ex = 0.5f * (hi[0] - lo[0]), ey = 0.5f * (hi[1] - lo[1]), ez = 0.5f * (hi[2] - lo[2]);
                            float c = pl.x * cx + pl.y * cy + pl.z * cz - pl.w;
                            float r = fabsf(pl.x) * ex + fabsf(pl.y) * ey + fabsf(pl.z) * ez;
                            on = fabsf(c) <= r;
                        } else if (lane >= 8 && lane < 8 + nt) {
                            const float *tp = TOR + 8 * (lane - 8);
                            float rr = tp[6] + tp[7];
                            on = box_dist2(tp[0], tp[1], tp[2], lo, hi) <= rr * rr;
                        }
                        omask = ballot(on);
                        if constexpr (SURR) {
                            // eligible support spheres this wave can reach in the window
                            bool en = false;
                            if (lane < n_bumps) {
                                const float4 c0 = A.surr_sb[2 * lane];
                                en = __float_as_int(A.surr_sb[2 * lane + 1].y) >= 0 &&
                                     box_dist2(c0.x, c0.y, c0.z, lo, hi) <= c0.w;
                            }
                            emask = ballot(en);
                        }
                        if constexpr (FREE) {
                            // Nothing in reach of this window: the steps are free flight,
                            // and so are those of the further windows that end before the
                            // nearest cut region or object.  The velocity is constant in
                            // flight, so that end follows from the wave's largest Euclidean
                            // speed (not from 1, the speed of a g-unit velocity there, which
                            // coarse steps do not keep: Euler steps through a sharp bump
                            // leave it up to a third faster).
                            // The twist is free only beyond its ball, and only if no
                            // velocity component is too small to absorb its acceleration.
                            const bool empty = ((FLAT && KIND != KIND_EUCLID ? bmask : 0ull) | sm[0] | sm[1] | sm[2] | sm[3] | omask) == 0;
                            if (empty && (FLAT || (box_dist2(0.f, 0.f, 0.f, pmn, pmx) > TWIST_FREE * TWIST_FREE &&
                                                   ballot(act && !(fminf(fabsf(y.x), fabsf(y.y)) >= TWIST_MIN_V)) == 0))) {
                                const float D = free_distance<KIND>(A, Bs, SPH, PLN, TOR, lane, pmn, pmx);
                                const float v2 = act ? dot(y, y) : 0.f;
                                float v = 1.001f;
                                if (ballot(v2 > 1.0f)) v = sqrt_(wave_max(v2)) * 1.0001f;
                                const float q = (D - 2e-4f) * rcp_(v * A.h_max) - 2.0f;
                                n_free = (int)fminf(fmaxf(q, 0.f), 1e6f);
                                // (an empty window was found empty by its own bound)
                                if constexpr (FLAT) n_free = max(n_free, A.K);
                                // (adaptive steps cull at multiples of the window)
                                if constexpr (!TIGHT) n_free = n_free / A.K * A.K;
                            }
                        }
                    }
                    if (COUNT && act) {
                        // objects inside this lane's own window (what one ray alone would need)
                        float m = A.cull_margin < 0.f ? 1e30f : A.cull_margin;
                        float llo[3] = {p.x - m, p.y - m, p.z - m}, lhi[3] = {p.x + m, p.y + m, p.z + m};
                        lane_objs = 0;
                        for (int i = 0; i < ns; ++i) {
                            float4 s = SPH[i];
                            lane_objs += box_dist2(s.x, s.y, s.z, llo, lhi) <= s.w * s.w ? 1u : 0u;
                        }
                        for (int i = 0; i < np; ++i) {
                            float4 pl = PLN[i];
                            float c = pl.x * p.x + pl.y * p.y + pl.z * p.z - pl.w;
                            lane_objs += fabsf(c) <= m * (fabsf(pl.x) + fabsf(pl.y) + fabsf(pl.z)) ? 1u : 0u;
                        }
                        for (int i = 0; i < nt; ++i) {
                            const float *tp = TOR + 8 * i;
                            float rr = tp[6] + tp[7];
                            lane_objs += box_dist2(tp[0], tp[1], tp[2], llo, lhi) <= rr * rr ? 1u : 0u;
                        }
                    }
                    if constexpr (BATCH) {
                        inb = act;
                        if (act) {
                            float4 *sv = batch_save();
                            sv[threadIdx.x] = make_float4(xh.x, xh.y, xh.z, xl.x);
                            sv[256 + threadIdx.x] = make_float4(xl.y, xl.z, y.x, y.y);
                            sv[512 + threadIdx.x] = make_float4(y.z, __int_as_float(steps), __int_as_float(acc_pass), 0.f);
                            bmin = bmax = p;
                        }
                        st_bw++;
                    }
                }
                if constexpr (FREE) {
                    // Free flight: a constant velocity, so a step is the three
                    // two-float additions of a constant increment (fixed steps; 12
                    // instructions) and its bookkeeping; no acceleration, no chord
                    // test, no culling until the flight ends.  The bits are those of
                    // the full steps.
                    if (n_free > 0) {
                        y = y + mk(0.f, 0.f, 0.f);
                        if constexpr (STEP != STEP_RK45) {
                            const V3<float> dx = free_step<STEP>(y, A.h);
                            // every active ray of a pass has taken the same number of steps
                            const int k0 = pass * A.S + it;
                            if (ballot(act && !finite6(dx, mk(0.f, 0.f, 0.f))) == 0) {
                                const int n = min(n_free, min(A.S - it, A.n_end - k0));
                                if (act) {
                                    for (int j = 0; j < n;) {
                                        int m = n - j;
                                        if constexpr (TAPE) {
                                            const int c = (k0 + j) / A.ckpt_every, o = (k0 + j) - c * A.ckpt_every;
                                            if (o == 0) write_ckpt(A, id, c, xh, xl, y);
                                            m = min(m, A.ckpt_every - o);
                                        }
                                        j += m;
#pragma unroll 4
                                        for (; m > 0; --m) {
                                            two_sum_add(xh.x, xl.x, dx.x);
                                            two_sum_add(xh.y, xl.y, dx.y);
                                            two_sum_add(xh.z, xl.z, dx.z);
                                        }
                                    }
                                    steps += n;
                                    acc_pass += n;
                                    if (k0 + n >= A.n_end) {
                                        write_out(A, qbase + pix, xh + xl, (float)steps * A.h, y, -1, steps);
                                        if (TAPE) A.tape_hit[(int64_t)(qbase + pix) * rti::TAPE_REC + 11] = __int_as_float(-1);
                                        alive = false;
                                    }
                                }
                                it += n;
                                continue;
                            }
                        } else {
                            // adaptive steps: a zero error estimate, so every trial is
                            // accepted and the step grows by the largest factor
                            A0 = mk(0.f, 0.f, 0.f);
                            need_a0 = false;
                            if (ballot(act && !finite6(A.h_max * y, mk(0.f, 0.f, 0.f))) == 0) {
                                for (int j = 0; j < n_free; ++j) {
                                    const bool on = alive && acc_pass < A.S;
                                    const uint64_t om = ballot(on);
                                    if (om == 0) break;
                                    st_lane += __popcll(om);
                                    if (on) {
                                        const float hs = fminf(hc, A.t_max - (th + tl));
                                        att++;
                                        hc = fminf(hs * 5.0f, A.h_max);
                                        two_sum_add(xh.x, xl.x, hs * y.x);
                                        two_sum_add(xh.y, xl.y, hs * y.y);
                                        two_sum_add(xh.z, xl.z, hs * y.z);
                                        two_sum_add(th, tl, hs);
                                        steps++;
                                        acc_pass++;
                                        if (steps >= A.max_steps || th + tl >= A.t_max * (1.0f - 1e-6f)) {
                                            write_out(A, qbase + pix, xh + xl, th + tl, y, -1, steps);
                                            alive = false;
                                        }
                                    }
                                }
                                it += n_free;
                                continue;
                            }
                        }
                    }
                }
                if constexpr (TIGHT) {
                    // ---- the march: steps of this window are computed, tested against the listed
                    // objects and committed in a loop with one wave-wide question per
                    // step, until some lane's step is an event (a chord hit, a failed
                    // acceleration or a non-finite increment).  That step stays
                    // uncommitted and is finished below.  Every active ray of a pass
                    // has taken the same number of steps, so the end of the ray is
                    // the end of the march for all of them.
                    const int k0 = pass * A.S + it;
                    const int n = min(wend - it, min(A.S - it, A.n_end - k0));
                    const bool objs = (sm[0] | sm[1] | sm[2] | sm[3] | omask) != 0;
                    int j = 0;
                    bool event = false, fail = false;
                    float hit_s = 2.f;
                    int hit_id = -1;
                    if (act) {
                        int ck = 0, ck_j = 0;  // TAPE: the next checkpoint and the step before which it is due
                        if constexpr (TAPE) {
                            ck = (k0 + A.ckpt_every - 1) / A.ckpt_every;
                            ck_j = ck * A.ckpt_every - k0;
                        }
                        auto checkpoint = [&]() {
                            if constexpr (TAPE) {
                                if (j == ck_j) {
                                    write_ckpt(A, id, ck, xh, xl, y);
                                    ck++;
                                    ck_j += A.ckpt_every;
                                }
                            }
                        };
                        V3<float> dx, dv;
                        auto march = [&](const auto &accel) {
                            auto step = [&](V3<float> p, V3<float> &dx, V3<float> &dv) {
                                const bool ok = fixed_step<STEP>(accel, p, y, A.h, dx, dv);
                                return ok && finite6(dx, dv);
                            };
                            // most windows list no object: a lean loop of their own
                            if (!objs) {
#pragma unroll 1
                                for (; j < n; ++j) {
                                    checkpoint();
                                    V3<float> dx, dv;
                                    if (ballot(!step(xh + xl, dx, dv))) break;
                                    two_sum_add(xh.x, xl.x, dx.x);
                                    two_sum_add(xh.y, xl.y, dx.y);
                                    two_sum_add(xh.z, xl.z, dx.z);
                                    y = y + dv;
                                }
                            }
#pragma unroll 1
                            for (; j < n; ++j) {
                                checkpoint();
                                const V3<float> p = xh + xl;
                                if (FLAT && KIND != KIND_EUCLID && bmask == 0) {
                                    // objects but no bump in the window
                                    dx = free_step<STEP>(y, A.h);
                                    dv = mk(0.f, 0.f, 0.f);
                                    fail = !finite6(dx, dv);
                                } else {
                                    fail = !step(p, dx, dv);
                                }
                                if (!fail) chord_scan(sm, omask, ns, np, SPH, PLN, TOR, xh, xl, p, dx, hit_s, hit_id);
                                event = ballot(fail || hit_id >= 0) != 0;
                                if (event) break;
                                two_sum_add(xh.x, xl.x, dx.x);
                                two_sum_add(xh.y, xl.y, dx.y);
                                two_sum_add(xh.z, xl.z, dx.z);
                                y = y + dv;
                            }
                        };
                        if constexpr (LIST) {
                            constexpr bool AN = KIND == KIND_GANISO;
                            const int nb = __popcll(bmask);
                            if (nb == 1) march(HeldAcc<AN, 1>(Bs, bmask));
                            else if (nb == 2) march(HeldAcc<AN, 2>(Bs, bmask));
                            else march(ListAcc<AN>{list, groups});
                        } else if (KIND == KIND_GRAPH && !(DENSE && __popcll(bmask) > DENSE_WALK)) {
                            march(GraphWalk{Bs, bmask, cutm});
                        } else if (KIND != KIND_GRAPH || DENSE) {
                            march(Acc32<KIND, false, true>{Bs, bmask, A.twist_amp, A.twist_theta0, nullptr, nullptr});
                        }
                        steps += j;
                        acc_pass += j;
                        if (event) {
                            if (fail) {
                                write_out(A, qbase + pix, xh + xl, (float)steps * A.h, y, -2, steps);
                                if (TAPE) A.tape_hit[(int64_t)(qbase + pix) * rti::TAPE_REC + 11] = __int_as_float(-1);
                                alive = false;
                            } else {
                                acc_pass++;  // a hit step was integrated: count it
                                if (hit_id >= 0) {
                                    alive = false;
                                } else {
                                    two_sum_add(xh.x, xl.x, dx.x);
                                    two_sum_add(xh.y, xl.y, dx.y);
                                    two_sum_add(xh.z, xl.z, dx.z);
                                    y = y + dv;
                                    steps++;
                                }
                            }
                        }
                        if (alive && steps >= A.n_end) {
                            write_out(A, qbase + pix, xh + xl, (float)steps * A.h, y, -1, steps);
                            if (TAPE) A.tape_hit[(int64_t)(qbase + pix) * rti::TAPE_REC + 11] = __int_as_float(-1);
                            alive = false;
                        }
                    }
                    // (the same for every active lane)
                    it += __builtin_amdgcn_readlane(j + (event ? 1 : 0), __builtin_ctzll(am));
                    push_hits(act && hit_id >= 0, hit_s, hit_id, A.h);
                    continue;
                }
                // wave statistics (work counting only; the lane count is also DP5's attempt count)
                if (COUNT || STEP == STEP_RK45) st_lane += __popcll(am);
                if (COUNT) {
                    st_wave++;
                    st_bl += __popcll(bmask);
                    st_ol += __popcll(sm[0]) + __popcll(sm[1]) + __popcll(sm[2]) + __popcll(sm[3]) + __popcll(omask);
                }

                if (TAPE && act && steps % A.ckpt_every == 0) write_ckpt(A, id, steps / A.ckpt_every, xh, xl, y);
                Acc32<KIND, COUNT, true> acc{Bs, bmask, A.twist_amp, A.twist_theta0, &c_eval, &c_bump};
                // The step is computed, its chord tested against the scene on
                // the state before the step, and only then committed: a hit
                // records that pre-step state without keeping copies of it.
                bool hit = false;
                int hit_id = -1;
                int park_b = -1;  // SURR: sphere the lane parked on in this step
                float hit_s = 2.f, hstep = A.h;
                if (act) {
                    V3<float> p = xh + xl;
                    V3<float> dx, dv;
                    bool ok, accepted = true;
                    if constexpr (STEP == STEP_RK45) {
                        bool ok0 = true;
                        if (need_a0) {
                            ok0 = acc(p, y, A0);
                            need_a0 = false;
                        }
                        hstep = fminf(hc, A.t_max - (th + tl));
                        V3<float> Anew = A0, ex, ev;
                        ok = step_dp5<float>(acc, p, y, hstep, Anew, dx, dv, ex, ev) && ok0;
                        att++;
                        V3<float> pn = p + dx, yn = y + dv;
                        auto sc = [&](float a, float b) { return A.atol + A.rtol * fmaxf(fabsf(a), fabsf(b)); };
                        float e2 = 0.f, r;
                        r = ex.x / sc(p.x, pn.x); e2 = fmaf(r, r, e2);
                        r = ex.y / sc(p.y, pn.y); e2 = fmaf(r, r, e2);
                        r = ex.z / sc(p.z, pn.z); e2 = fmaf(r, r, e2);
                        r = ev.x / sc(y.x, yn.x); e2 = fmaf(r, r, e2);
                        r = ev.y / sc(y.y, yn.y); e2 = fmaf(r, r, e2);
                        r = ev.z / sc(y.z, yn.z); e2 = fmaf(r, r, e2);
                        float en = sqrtf(e2 * (1.0f / 6.0f));
                        float fac = en > 0.f ? 0.9f * exp2f(-0.2f * __log2f(en)) : 5.0f;
                        fac = fminf(fmaxf(fac, 0.2f), 5.0f);
                        if (en <= 1.0f) {
                            hc = fminf(hstep * fac, A.h_max);
                            A0 = Anew;
                        } else {
                            accepted = false;
                            hc = hstep * fminf(fac, 1.0f);
                            if (hc < A.h_min || att > 8 * A.max_steps) ok = false;
                        }
                    } else if constexpr (STEP == STEP_RK4) {
                        if constexpr (SURR) {
                            // jumps and partial entry steps shift the step grid: the
                            // last step is clipped to land on min(t_max, max_steps h)
                            const float t_lim = fminf(A.t_max, (float)A.max_steps * A.h);
                            // (a remainder within rounding of h is a full step, so a ray
                            // that never parked takes exactly the plain trace's steps)
                            const float rem = t_lim - ((float)steps * A.h + (th + tl));
                            hstep = rem < A.h * (1.0f - 1e-5f) ? fmaxf(rem, 0.f) : A.h;
                        }
                        ok = step_rk4<float>(acc, p, y, hstep, dx, dv);
                    } else {
                        ok = step_euler<float>(acc, p, y, A.h, dx, dv);
                    }
                    bool done_fail = !ok || !finite6(dx, dv);
                    bool done_miss = false;
                    if (!done_fail && accepted) {
                        if (COUNT) c_obj += lane_objs;
                        // ---- segment versus scene, chord [x, x + dx] (a scalar branch:
                        // most wave iterations list no object)
                        if ((!BATCH || replay) && (sm[0] | sm[1] | sm[2] | sm[3] | omask) != 0) {
                            chord_scan(sm, omask, ns, np, SPH, PLN, TOR, xh, xl, p, dx, hit_s, hit_id);
                        }
                        // ---- chord entering an eligible support sphere (SURR)
                        float ent_s = 2.f;
                        int ent_b = -1;
                        if constexpr (SURR) {
                            uint64_t em = emask;
                            while (em) {
                                const int b = __builtin_ctzll(em);
                                em &= em - 1;
                                const float4 c0 = A.surr_sb[2 * b];
                                V3<float> o = mk((xh.x - c0.x) + xl.x, (xh.y - c0.y) + xl.y, (xh.z - c0.z) + xl.z);
                                const float o2 = dot(o, o);
                                const V3<float> on = o + dx;
                                if (b != skip && o2 >= c0.w && dot(on, on) < c0.w) {
                                    // smaller root of |o + s dx|^2 = R^2
                                    const float B = dot(o, dx), C = o2 - c0.w, DD = dot(dx, dx);
                                    const float disc = fmaxf(B * B - DD * C, 0.f);
                                    const float sr = fminf(fmaxf((-B - sqrtf(disc)) / DD, 0.f), 1.f);
                                    if (sr < ent_s) {
                                        ent_s = sr;
                                        ent_b = b;
                                    }
                                }
                            }
                            // park only while enough passes remain to finish the ray afterwards
                            if (ent_b >= 0 && (A.n_passes - 1 - pass) * A.S < A.max_steps - steps) ent_b = -1;
                        }
                        if (SURR && ent_b >= 0 && !(hit_id >= 0 && hit_s < ent_s)) {
                            two_sum_add(xh.x, xl.x, ent_s * dx.x);
                            two_sum_add(xh.y, xl.y, ent_s * dx.y);
                            two_sum_add(xh.z, xl.z, ent_s * dx.z);
                            y = y + ent_s * dv;
                            two_sum_add(th, tl, ent_s * hstep);
                            parked = true;
                            park_b = ent_b;
                            hit_id = -1;
                        } else if (hit_id >= 0) {
                            hit = true;
                            acc_pass++;  // the hit step was integrated: count it
                        } else {
                            // commit the step
                            two_sum_add(xh.x, xl.x, dx.x);
                            two_sum_add(xh.y, xl.y, dx.y);
                            two_sum_add(xh.z, xl.z, dx.z);
                            y = y + dv;
                            acc_pass++;
                            bool clipped = false;
                            if (STEP == STEP_RK45) {
                                two_sum_add(th, tl, hstep);
                                steps++;
                            } else if (SURR && hstep < A.h) {
                                // clipped last step: its length goes to t, not to the step count
                                two_sum_add(th, tl, hstep);
                                clipped = true;
                            } else {
                                steps++;
                            }
                            // RK45 lands on t_max up to float rounding of the clipped last step
                            float t = (STEP == STEP_RK45) ? th + tl : (float)steps * A.h + (SURR ? th + tl : 0.f);
                            float t_end = (STEP == STEP_RK45) ? A.t_max * (1.0f - 1e-6f) : A.t_max;
                            if constexpr (CARRY_T) done_miss = steps >= A.max_steps || t >= t_end || clipped;
                            else done_miss = steps >= A.n_end;
                            if constexpr (BATCH) {
                                if (!replay) {
                                    const V3<float> q = xh + xl;
                                    bmin = mk(fminf(bmin.x, q.x), fminf(bmin.y, q.y), fminf(bmin.z, q.z));
                                    bmax = mk(fmaxf(bmax.x, q.x), fmaxf(bmax.y, q.y), fmaxf(bmax.z, q.z));
                                }
                            }
                        }
                    }
                    if (BATCH && !replay && (done_fail || done_miss)) {
                        // the output waits until the window's box test clears this lane
                        fin = done_fail ? 2 : 1;
                    } else if (done_fail || done_miss) {
                        write_out(A, qbase + pix, xh + xl,
                                  STEP == STEP_RK45 ? th + tl : (float)steps * A.h + (SURR ? th + tl : 0.f), y,
                                  done_fail ? -2 : -1, steps);
                        if (TAPE) A.tape_hit[(int64_t)(qbase + pix) * rti::TAPE_REC + 11] = __int_as_float(-1);
                    }
                    if (done_fail || done_miss || hit) alive = false;
                }
                push_hits(hit, hit_s, hit_id, hstep);
                if constexpr (SURR) {
                    // ---- queue the rays that parked on a support sphere in this step
                    const bool now = park_b >= 0;
                    const uint64_t pm = ballot(now);
                    if (pm) {
                        int base = 0;
                        if (lane == 0) base = atomicAdd(pass_ctr + rti::CTR_XQ, __popcll(pm));
                        base = uniform_i(__shfl(base, 0));
                        if (now) {
                            const int net = __float_as_int(A.surr_sb[2 * park_b + 1].y);
                            const int rank = atomicAdd(A.xctl + net, 1);
                            A.xq[base + mbcnt64(pm)] = make_int4(id, park_b, rank, 0);
                        }
                    }
                }
                if constexpr (BATCH) {
                    wi++;
                    if (!replay) it_m++;
                    if (replay) {
                        if (wi >= wlen) {
                            replay = false;
                            hold = false;
                            wi = 0;
                        }
                    } else if (wi == A.K || ballot(alive && it_m < A.S) == 0) {
                        // ---- end of the march: the lanes' polygon boxes against
                        // the window's objects
                        bool cand = false;
                        if (inb) {
                            // margin: FP32 rounding of the positions and of the
                            // chord tests, far below it
                            const float eps = 1e-3f + 1e-5f * fmaxf(fmaxf(fabsf(bmin.x), fabsf(bmax.x)),
                                                                   fmaxf(fmaxf(fabsf(bmin.y), fabsf(bmax.y)),
                                                                         fmaxf(fabsf(bmin.z), fabsf(bmax.z))));
                            const float lo[3] = {bmin.x - eps, bmin.y - eps, bmin.z - eps};
                            const float hi[3] = {bmax.x + eps, bmax.y + eps, bmax.z + eps};
#pragma unroll
                            for (int w = 0; w < 4; ++w) {
                                uint64_t m = sm[w];
                                while (m) {
                                    const int b = __builtin_ctzll(m);
                                    m &= m - 1;
                                    const float4 sp = SPH[64 * w + b];
                                    cand |= box_dist2(sp.x, sp.y, sp.z, lo, hi) <= sp.w * sp.w;
                                }
                            }
                            uint64_t m = omask;
                            while (m) {
                                const int b = __builtin_ctzll(m);
                                m &= m - 1;
                                if (b < 8) {
                                    const float4 pl = PLN[b];
                                    const float cx = 0.5f * (lo[0] + hi[0]), cy = 0.5f * (lo[1] + hi[1]),
                                                cz = 0.5f * (lo[2] + hi[2]);
                                    const float ex = 0.5f * (hi[0] - lo[0]), ey = 0.5f * (hi[1] - lo[1]),
                                                ez = 0.5f * (hi[2] - lo[2]);
                                    const float c = pl.x * cx + pl.y * cy + pl.z * cz - pl.w;
                                    cand |= fabsf(c) <= fabsf(pl.x) * ex + fabsf(pl.y) * ey + fabsf(pl.z) * ez;
                                } else {
                                    const float *tp = TOR + 8 * (b - 8);
                                    const float rr = tp[6] + tp[7];
                                    cand |= box_dist2(tp[0], tp[1], tp[2], lo, hi) <= rr * rr;
                                }
                            }
                        }
                        if (fin && !cand) {
                            write_out(A, qbase + pix, xh + xl, (float)steps * A.h, y, fin == 2 ? -2 : -1, steps);
                            fin = 0;
                        }
                        if (ballot(cand)) {
                            if (cand) {
                                const float4 *sv = batch_save();
                                const float4 a = sv[threadIdx.x], b = sv[256 + threadIdx.x], c = sv[512 + threadIdx.x];
                                xh = mk(a.x, a.y, a.z);
                                xl = mk(a.w, b.x, b.y);
                                y = mk(b.z, b.w, c.x);
                                steps = __float_as_int(c.y);
                                acc_pass = __float_as_int(c.z);
                                alive = true;
                                fin = 0;
                            }
                            hold = !cand;
                            replay = true;
                            wlen = wi;
                            st_br++;
                        }
                        wi = 0;
                        inb = false;
                    }
                }
                it++;
            }

            // ---- survivors keep their state in place; the chunk's alive mask
            // and the per-set counts feed the ordered compaction after the pass
            uint64_t sv = ballot(alive);
            if (lane == 0) A.cmask[chunk] = sv;
            if (sv) {
                if (lane == 0) atomicAdd(pass_ctr + rti::CTR_SURV + set, __popcll(sv));
                if (alive) {
                    float *__restrict__ dst = st + ((int64_t)(id >> 6) * rti::Q_NFIELDS * 64 + (id & 63));
                    auto P = [&](int f, float v) { dst[f * 64] = v; };
                    P(rti::Q_XH, xh.x);
                    P(rti::Q_XH + 1, xh.y);
                    P(rti::Q_XH + 2, xh.z);
                    P(rti::Q_XL, xl.x);
                    P(rti::Q_XL + 1, xl.y);
                    P(rti::Q_XL + 2, xl.z);
                    P(rti::Q_Y, y.x);
                    P(rti::Q_Y + 1, y.y);
                    P(rti::Q_Y + 2, y.z);
                    if constexpr (CARRY_T) {
                        P(rti::Q_TH, th);
                        P(rti::Q_TL, tl);
                        P(rti::Q_H, hc);
                        P(rti::Q_ATT, __int_as_float(att));
                    }
                    P(rti::Q_STEPS, __int_as_float(steps));
                    if constexpr (SURR) P(rti::Q_SKIP, __int_as_float(skip));
                }
            }
            // accepted steps of this chunk
            int acc_l = acc_pass;
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) acc_l += __shfl_xor(acc_l, o);
            st_steps += (unsigned)uniform_i(acc_l);
            if (COUNT) {
                unsigned v[3] = {c_eval, c_bump, c_obj};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    unsigned x = v[q];
#pragma unroll
                    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
                    v[q] = (unsigned)uniform_i((int)x);
                }
                st_ev += v[0];
                st_be += v[1];
                st_ot += v[2];
            }
        }
    }
    if (lane == 0) {
        if (BATCH) {
            atomicAdd(A.stats + rti::ST_BATCH_WIN, st_bw);
            atomicAdd(A.stats + rti::ST_BATCH_REPLAY, st_br);
        }
        if (st_rays) atomicAdd(A.stats + rti::ST_RAYS, st_rays);
        atomicAdd(A.stats + rti::ST_STEPS, st_steps);
        atomicAdd(A.stats + rti::ST_ATTEMPTS, STEP == STEP_RK45 ? st_lane : st_steps);
        if (COUNT) {
            atomicAdd(A.stats + rti::ST_WAVE_ITERS, st_wave);
            atomicAdd(A.stats + rti::ST_LANE_ITERS, st_lane);
            atomicAdd(A.stats + rti::ST_BUMP_LIST, st_bl);
            atomicAdd(A.stats + rti::ST_OBJ_LIST, st_ol);
            atomicAdd(A.stats + rti::ST_ACC_EVALS, st_ev);
            atomicAdd(A.stats + rti::ST_BUMP_EVALS, st_be);
            atomicAdd(A.stats + rti::ST_OBJ_TESTS, st_ot);
        }
    }
}

// =============================================================== refinement
__device__ __forceinline__ double obj_F64(int id, V3<double> x, int ns, int np, const double *__restrict__ SPD,
                                          const double *__restrict__ PLD, const double *__restrict__ TOD) {
    if (id < ns) {
        const double *s = SPD + 4 * id;
        V3<double> d = mk(x.x - s[0], x.y - s[1], x.z - s[2]);
        return dot(d, d) - s[3] * s[3];
    }
    id -= ns;
    if (id < np) {
        const double *p = PLD + 4 * id;
        return p[0] * x.x + p[1] * x.y + p[2] * x.z - p[3];
    }
    return torus_sdf<double>(TOD + 8 * (id - np), x);
}

// COUNT: also counts the acceleration evaluations, the bumps inside their
// cut at them (graph metric) and the integrator steps (work statistics).
// Occupancy: the graph-metric RK4 refine is compiled for 4 waves per SIMD
// (128 VGPRs, 36 B of spills; 3.5% faster than 3 waves at 156 VGPRs); the
// other kinds need 144-204 VGPRs, and 3 or 4 waves measured no faster.
template <int KIND, int STEP, bool COUNT = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KIND == KIND_GRAPH && STEP == STEP_RK4 ? 4 : 1, 8))) void k_refine(TraceArgs A, const double *__restrict__ BD,
                                                const double *__restrict__ SPD, const double *__restrict__ PLD,
                                                const double *__restrict__ TOD) {
    const int n = A.ctr[rti::CTR_REFINE];
    const int HW = A.width * A.height;
    unsigned c_eval = 0, c_bump = 0, c_step = 0;  // COUNT only
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += gridDim.x * blockDim.x) {
        float4 r0, r1, r2, r3, r4;
        double tk_hi, tk_lo, h, sc;
        int obj, oi, k;
        uint64_t mask;
        if (!A.surr && compact_record(STEP, false)) {
            const float4 *rec = A.rec + 4 * (int64_t)r;
            r0 = rec[0], r1 = rec[1], r2 = rec[2], r3 = rec[3];
            tk_hi = tk_lo = 0.0;
            h = A.h;
            sc = r2.y;
            obj = __float_as_int(r2.z), oi = __float_as_int(r2.w), k = __float_as_int(r3.x);
            mask = (uint64_t)(uint32_t)__float_as_int(r3.y) | ((uint64_t)(uint32_t)__float_as_int(r3.z) << 32);
        } else {
            const float4 *rec = A.rec + rti::REC_F4 * (int64_t)r;
            r0 = rec[0], r1 = rec[1], r2 = rec[2], r3 = rec[3], r4 = rec[4];
            tk_hi = r2.y, h = r2.z;
            sc = r2.w;
            obj = __float_as_int(r3.x), oi = __float_as_int(r3.y), k = __float_as_int(r3.z);
            tk_lo = r3.w;
            mask = (uint64_t)(uint32_t)__float_as_int(r4.x) | ((uint64_t)(uint32_t)__float_as_int(r4.y) << 32);
        }
        V3<double> x = mk((double)r0.x + (double)r0.w, (double)r0.y + (double)r1.x, (double)r0.z + (double)r1.y);
        V3<double> y = mk((double)r1.z, (double)r1.w, (double)r2.x);
        int set = oi / HW;
        const double *Bs = BD + (int64_t)set * A.n_bumps * (is_deform(KIND) ? DEFORM_D : 8);
        double amp = A.twist_amp, th0 = A.twist_theta0;
        auto acc = [&](V3<double> p, V3<double> v, V3<double> &a) -> bool {
            if constexpr (COUNT) c_eval++;
            if constexpr (KIND == KIND_GRAPH) {
                a = graph_accel_f64(Bs, mask, p, v, COUNT ? &c_bump : nullptr);
                return true;
            } else if constexpr (KIND == KIND_TWIST) {
                return twist_accel<double>(amp, th0, p, v, a);
            } else if constexpr (KIND == KIND_ZTWIST) {
                a = ztwist_accel<double>(p, v);
                return true;
            } else if constexpr (is_deform(KIND)) {
                return deform_accel<double, false, KIND == KIND_DEFORM_ROT>(Bs, mask, p, v, a);
            } else if constexpr (KIND == KIND_GANISO) {
                a = graph_aniso_accel<double>(Bs, mask, p, v);
                return true;
            } else if constexpr (KIND == KIND_GQUAD) {
                a = graph_quad_accel<double>(mk(Bs[0], Bs[1], Bs[2]), p, v);
                return true;
            } else {
                a = mk(0.0, 0.0, 0.0);
                return true;
            }
        };
        // every probe of the bisection restarts from the same state, so the
        // first stage a(x_k, y_k) is evaluated once
        V3<double> a0;
        acc(x, y, a0);
        auto step = [&](double hs, V3<double> &xo, V3<double> &yo) {
            if constexpr (COUNT) c_step++;
            V3<double> dx, dv;
            if constexpr (STEP == STEP_RK45) {
                V3<double> A1 = a0, ex, ev;
                step_dp5<double>(acc, x, y, hs, A1, dx, dv, ex, ev);
            } else if constexpr (STEP == STEP_RK4) {
                step_rk4<double>(acc, x, y, hs, dx, dv, &a0);
            } else {
                step_euler<double>(acc, x, y, hs, dx, dv, &a0);
            }
            xo = x + dx;
            yo = y + dv;
        };
        double F0 = obj_F64(obj, x, A.n_spheres, A.n_planes, SPD, PLD, TOD);
        V3<double> x1, y1;
        step(h, x1, y1);
        double F1 = obj_F64(obj, x1, A.n_spheres, A.n_planes, SPD, PLD, TOD);
        double s = sc;
        if ((F0 > 0.0) != (F1 > 0.0)) {
            // The bracket [lo, hi] of the sign change is narrowed to a width
            // of 2^-bisect_iters, as bisection would, but by regula falsi with
            // the Illinois modification (the value at an end kept twice in a
            // row is halved), the first probe at the segment's FP32 root: a
            // handful of probes instead of one per halving, since the implicit
            // function is nearly linear across one step.  When two probes
            // have not halved the bracket the next one is a plain halving, so
            // the bracket halves at least every third probe.
            const bool pos0 = F0 > 0.0;
            const double tol = ldexp(1.0, -A.bisect_iters);
            double lo = 0.0, hi = 1.0, flo = F0, fhi = F1;
            double w_ref = 1.0;
            int kept = 0, since = 0;  // end kept by the last probe (-1 lo, +1 hi); probes since the last check
            bool halve = false;
            for (int i = 0; i < 3 * A.bisect_iters + 2 && hi - lo > tol; ++i) {
                double m = i == 0 ? sc : (halve ? 0.5 * (lo + hi) : lo + (hi - lo) * (flo / (flo - fhi)));
                if (!(m > lo && m < hi)) m = 0.5 * (lo + hi);
                V3<double> xm, ym;
                step(m * h, xm, ym);
                const double fm = obj_F64(obj, xm, A.n_spheres, A.n_planes, SPD, PLD, TOD);
                if (fm == 0.0) {
                    lo = hi = m;
                    break;
                }
                if ((fm > 0.0) == pos0) {
                    lo = m;
                    flo = fm;
                    if (kept == 1) fhi *= 0.5;
                    kept = 1;
                } else {
                    hi = m;
                    fhi = fm;
                    if (kept == -1) flo *= 0.5;
                    kept = -1;
                }
                halve = false;
                if (++since == 2) {
                    halve = hi - lo > 0.5 * w_ref;
                    w_ref = hi - lo;
                    since = 0;
                }
            }
            s = 0.5 * (lo + hi);
        }
        V3<double> xs, ys;
        step(s * h, xs, ys);
        // RK4 and Euler: k steps of h, plus (surrogate) jumps and partial steps
        double tk = STEP == STEP_RK45 ? tk_hi + tk_lo : (double)k * (double)A.h + (tk_hi + tk_lo);
        A.out_hit[3 * (int64_t)oi + 0] = (float)xs.x;
        A.out_hit[3 * (int64_t)oi + 1] = (float)xs.y;
        A.out_hit[3 * (int64_t)oi + 2] = (float)xs.z;
        A.out_t[oi] = (float)(tk + s * h);
        A.out_id[oi] = obj;
        double nrm = 1.0 / sqrt(dot(ys, ys));
        A.out_dir[3 * (int64_t)oi + 0] = (float)(ys.x * nrm);
        A.out_dir[3 * (int64_t)oi + 1] = (float)(ys.y * nrm);
        A.out_dir[3 * (int64_t)oi + 2] = (float)(ys.z * nrm);
        if (A.out_steps) A.out_steps[oi] = k + 1;
        if (A.tape_hit) {
            float *tr = A.tape_hit + (int64_t)oi * rti::TAPE_REC;
            tr[0] = r0.x;
            tr[1] = r0.y;
            tr[2] = r0.z;
            tr[3] = r0.w;
            tr[4] = r1.x;
            tr[5] = r1.y;
            tr[6] = r1.z;
            tr[7] = r1.w;
            tr[8] = r2.x;
            tr[9] = (float)s;
            tr[10] = __int_as_float(k);
            tr[11] = __int_as_float(obj);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(A.stats + rti::ST_REFINED, (unsigned long long)n);
    if constexpr (COUNT) {
        unsigned v[3] = {c_eval, c_bump, c_step};
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) v[q] += __shfl_xor(v[q], o);
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(A.stats + rti::ST_REF_EVALS, (unsigned long long)v[0]);
            atomicAdd(A.stats + rti::ST_REF_BUMPS, (unsigned long long)v[1]);
            atomicAdd(A.stats + rti::ST_REF_STEPS, (unsigned long long)v[2]);
        }
    }
}

// ====================================================== ordered compaction
// After pass p: survivors of chunk c (alive mask cmask[c]) move to the
// sorted list of pass p+1 at
//   pad_base[set] + (survivors in chunks < c) + (rank in chunk) - (survivors in sets < set)
// where pad_base[set] rounds every earlier set up to whole chunks.  Sorted
// ids keep 64 consecutive survivors spatially close (same or adjacent
// tiles), which keeps the per-wave culling windows tight.
__global__ __launch_bounds__(1024) void k_chunk_scan(TraceArgs A, int pass) {
    __shared__ int sh[1024];
    const int nch = A.ctr[rti::CTR_PASS0 + pass * rti::CTR_PASS_WORDS + rti::CTR_NCH];
    const int nblk = (nch + rti::SCAN_BLOCK - 1) / rti::SCAN_BLOCK;
    for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
        int c = b * rti::SCAN_BLOCK + threadIdx.x;
        int v = c < nch ? __popcll(A.cmask[c]) : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            int u = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
            __syncthreads();
            sh[threadIdx.x] += u;
            __syncthreads();
        }
        if (c < nch) A.cscan[c] = sh[threadIdx.x] - v;
        if (threadIdx.x == 1023) A.bscan[b] = sh[1023];
        __syncthreads();
    }
}

__global__ __launch_bounds__(1024) void k_block_scan(TraceArgs A, int pass) {
    __shared__ int sh[1024];
    __shared__ int carry;
    const int nch = A.ctr[rti::CTR_PASS0 + pass * rti::CTR_PASS_WORDS + rti::CTR_NCH];
    const int nblk = (nch + rti::SCAN_BLOCK - 1) / rti::SCAN_BLOCK;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nblk; base += 1024) {
        int i = base + threadIdx.x;
        int v = i < nblk ? A.bscan[i] : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            int u = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
            __syncthreads();
            sh[threadIdx.x] += u;
            __syncthreads();
        }
        if (i < nblk) A.bscan[i] = carry + sh[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == 1023) carry += sh[1023];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_scatter(TraceArgs A, int pass) {
    const int lane = lane_id();
    const int *pc = A.ctr + rti::CTR_PASS0 + pass * rti::CTR_PASS_WORDS;
    const int nch = pc[rti::CTR_NCH];
    // per-set survivor counts of this pass: unpadded and chunk-padded prefixes
    int cnt = lane < A.n_sets ? pc[rti::CTR_SURV + lane] : 0;
    int excl = wave_incl_scan(cnt) - cnt;
    int pad = (cnt + 63) & ~63;
    int pexcl = wave_incl_scan(pad) - pad;
    const int *__restrict__ ids_in = A.ids[pass & 1];
    int *__restrict__ ids_out = A.ids[(pass + 1) & 1];
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int nwaves = (gridDim.x * blockDim.x) >> 6;
    for (int c = wave; c < nch; c += nwaves) {
        uint64_t m = A.cmask[c];
        if (!m) continue;
        bool alive = (m >> lane) & 1ull;
        int id = alive ? (pass == 0 ? c * 64 + lane : ids_in[c * 64 + lane]) : 0;
        int s = id / A.T;
        int rank = A.bscan[c / rti::SCAN_BLOCK] + A.cscan[c] + mbcnt64(m);
        int pos = __shfl(pexcl, s) + rank - __shfl(excl, s);
        if (alive) ids_out[pos] = id;
    }
}

__global__ void k_reset(int *ctr, int n_words, unsigned long long *stats) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += gridDim.x * blockDim.x) ctr[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x < rti::ST_N) stats[threadIdx.x] = 0;
}

template <int KIND, int STEP, bool SURR, bool TAPE = false>
hipError_t launch_pass(const TraceArgs &a, const rti::DeviceData &d, int p, int grid, hipStream_t s) {
    if constexpr (STEP != STEP_RK45 && !SURR && !TAPE) {
        if (a.batch) {
            hipLaunchKernelGGL((k_trace_pass<KIND, STEP, false, false, false, true>), dim3(grid), dim3(256), 0, s, a,
                               p, d.bump_f, d.sph_f, d.pln_f, d.tor_f);
            return hipGetLastError();
        }
    }
    if constexpr (has_small_variant(KIND, STEP) && !SURR) {
        // the small-launch variant: the first pass by its known chunk count, a
        // later pass by the survivors (each variant reads the count and only
        // one proceeds; frames that are small to begin with need one launch)
        const int chunks = a.n_sets * a.tiles_x * a.tiles_y;
        if (!a.count && a.lat_chunks > 0 && (p > 0 || chunks <= a.lat_chunks))
            hipLaunchKernelGGL((k_trace_pass<KIND, STEP, false, false, TAPE, false, true>),
                               dim3(std::min(grid, (a.lat_chunks + 3) / 4)), dim3(256), 0, s, a, p, d.bump_f, d.sph_f,
                               d.pln_f, d.tor_f);
        if (!a.count && a.lat_chunks > 0 && chunks <= a.lat_chunks) return hipGetLastError();
    }
    if constexpr (few_fly(KIND, STEP) && !SURR && !TAPE) {
        if (!a.count && a.n_bumps > FLY_DEFORMS) {
            hipLaunchKernelGGL((k_trace_pass<KIND, STEP, false, false, false, false, false, false>), dim3(grid), dim3(256),
                               0, s, a, p, d.bump_f, d.sph_f, d.pln_f, d.tor_f);
            return hipGetLastError();
        }
    }
    if constexpr (has_dense(KIND, STEP) && !SURR && !TAPE) {
        if (!a.count && a.n_bumps > SPARSE_BUMPS) {
            hipLaunchKernelGGL((k_trace_pass<KIND, STEP, false, false, false, false, false, true, true>), dim3(grid),
                               dim3(256), 0, s, a, p, d.bump_f, d.sph_f, d.pln_f, d.tor_f);
            return hipGetLastError();
        }
    }
    if (a.count)
        hipLaunchKernelGGL((k_trace_pass<KIND, STEP, true, SURR, TAPE>), dim3(grid), dim3(256), 0, s, a, p,
                           d.bump_f, d.sph_f, d.pln_f, d.tor_f);
    else
        hipLaunchKernelGGL((k_trace_pass<KIND, STEP, false, SURR, TAPE>), dim3(grid), dim3(256), 0, s, a, p,
                           d.bump_f, d.sph_f, d.pln_f, d.tor_f);
    return hipGetLastError();
}

template <int KIND, int STEP>
hipError_t launch_kind_step(const TraceArgs &a, const rti::DeviceData &d, int n_passes, int grid, int rgrid,
                            hipStream_t s, hipEvent_t *ev, const rti::SurrArgs *S, int mlp_blocks) {
    const int scan_blocks = std::min((a.max_chunks + rti::SCAN_BLOCK - 1) / rti::SCAN_BLOCK, 1024);
    const int scatter_blocks = std::max(1, std::min((a.max_chunks + 3) / 4, 4096));
    for (int p = 0; p < n_passes; ++p) {
        if (p > 0) {
            // ordered compaction of the survivors of pass p-1 (not timed as a pass)
            hipLaunchKernelGGL(k_chunk_scan, dim3(scan_blocks), dim3(1024), 0, s, a, p - 1);
            hipLaunchKernelGGL(k_block_scan, dim3(1), dim3(1024), 0, s, a, p - 1);
            hipLaunchKernelGGL(k_scatter, dim3(scatter_blocks), dim3(256), 0, s, a, p - 1);
            if (ev) (void)hipEventRecord(ev[2 * n_passes + 2 + p], s);
        }
        hipError_t e;
        if constexpr (KIND == KIND_GRAPH && STEP == STEP_RK4) {
            if (a.tape_ck) {
                e = launch_pass<KIND, STEP, false, true>(a, d, p, grid, s);
                if (e != hipSuccess) return e;
                if (ev) (void)hipEventRecord(ev[2 + p], s);
                continue;
            }
            if (a.surr) {
                e = launch_pass<KIND, STEP, true>(a, d, p, grid, s);
                if (e != hipSuccess) return e;
                if (ev) (void)hipEventRecord(ev[2 + p], s);
                // crossings parked in pass p (not timed as a pass)
                e = rti::launch_surr_stage(a, *S, d.bump_f, p, mlp_blocks, s);
                if (e != hipSuccess) return e;
                if (ev) (void)hipEventRecord(ev[3 * n_passes + 3 + p], s);
                continue;
            }
        }
        e = launch_pass<KIND, STEP, false>(a, d, p, grid, s);
        if (e != hipSuccess) return e;
        if (ev) (void)hipEventRecord(ev[2 + p], s);
    }
    if (a.count)
        hipLaunchKernelGGL((k_refine<KIND, STEP, true>), dim3(rgrid), dim3(256), 0, s, a, d.bump_d, d.sph_d, d.pln_d,
                           d.tor_d);
    else
        hipLaunchKernelGGL((k_refine<KIND, STEP>), dim3(rgrid), dim3(256), 0, s, a, d.bump_d, d.sph_d, d.pln_d,
                           d.tor_d);
    hipError_t e = hipGetLastError();
    if (ev) (void)hipEventRecord(ev[2 + n_passes], s);
    return e;
}

template <int KIND, int STEP> int occ() {
    int n = 0;
    // (of the flying and the other variant, the one that more blocks fit)
    constexpr bool fly = !few_fly(KIND, STEP);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, k_trace_pass<KIND, STEP, false, false, false, false, false, fly>, 256, 0) != hipSuccess)
        return 1;
    return n > 0 ? n : 1;
}

}  // namespace

namespace rti {

bool has_small_variant(int kind, int step) { return ::has_small_variant(kind, step); }

bool supported(int kind, int step) {
    return kind >= 0 && kind <= 7 && step >= 0 && step <= 2;
}

#define RT_DISPATCH(KIND, FN, ...)                                                 \
    switch (step) {                                                                \
    case STEP_RK4: return FN<KIND, STEP_RK4>(__VA_ARGS__);                         \
    case STEP_RK45: return FN<KIND, STEP_RK45>(__VA_ARGS__);                       \
    default: return FN<KIND, STEP_EULER>(__VA_ARGS__);                             \
    }

int trace_blocks_per_cu(int kind, int step) {
    switch (kind) {
    case KIND_EUCLID: RT_DISPATCH(KIND_EUCLID, occ)
    case KIND_GRAPH: RT_DISPATCH(KIND_GRAPH, occ)
    case KIND_TWIST: RT_DISPATCH(KIND_TWIST, occ)
    case KIND_ZTWIST: RT_DISPATCH(KIND_ZTWIST, occ)
    case KIND_DEFORM: RT_DISPATCH(KIND_DEFORM, occ)
    case KIND_DEFORM_ROT: RT_DISPATCH(KIND_DEFORM_ROT, occ)
    case KIND_GANISO: RT_DISPATCH(KIND_GANISO, occ)
    default: RT_DISPATCH(KIND_GQUAD, occ)
    }
}

// Workspace of the allocation-free trace: one array per GPU, held by the
// code object until the process ends.  Host code never passes `scratch`
// itself to a kernel (on the host it names a stand-in, not device memory):
// it uses the address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[RT_NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(int device, void **ptr) {
    constexpr int MAX_DEV = 64;
    static std::mutex mu;
    static void *addr[MAX_DEV] = {};
    if (!ptr || device < 0 || device >= MAX_DEV) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int prev = -1;
        hipError_t e = hipGetDevice(&prev);
        if (e != hipSuccess) return e;
        if (prev != device && (e = hipSetDevice(device)) != hipSuccess) return e;
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (prev != device) (void)hipSetDevice(prev);  // restore the caller's device, best effort
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

hipError_t launch_trace(const TraceArgs &a, const DeviceData &d, int n_passes, int grid, int rgrid, hipStream_t s,
                        hipEvent_t *ev, const SurrArgs *S, int mlp_blocks) {
    int words = CTR_PASS0 + n_passes * CTR_PASS_WORDS + CTR_SURR_WORDS;
    if (ev) (void)hipEventRecord(ev[0], s);
    hipLaunchKernelGGL(k_reset, dim3(64), dim3(256), 0, s, a.ctr, words, a.stats);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (ev) (void)hipEventRecord(ev[1], s);
    const int step = a.step_kind;
    // checkpoint tapes and learned crossings exist for the graph metric with RK4 only
    if ((a.tape_ck || a.surr) && !(a.kind == KIND_GRAPH && step == STEP_RK4)) return hipErrorInvalidValue;
    switch (a.kind) {
    case KIND_EUCLID: RT_DISPATCH(KIND_EUCLID, launch_kind_step, a, d, n_passes, grid, rgrid, s, ev, S, mlp_blocks)
    case KIND_GRAPH: RT_DISPATCH(KIND_GRAPH, launch_kind_step, a, d, n_passes, grid, rgrid, s, ev, S, mlp_blocks)
    case KIND_TWIST: RT_DISPATCH(KIND_TWIST, launch_kind_step, a, d, n_passes, grid, rgrid, s, ev, S, mlp_blocks)
    case KIND_ZTWIST: RT_DISPATCH(KIND_ZTWIST, launch_kind_step, a, d, n_passes, grid, rgrid, s, ev, S, mlp_blocks)
    case KIND_DEFORM: RT_DISPATCH(KIND_DEFORM, launch_kind_step, a, d, n_passes, grid, rgrid, s, ev, S, mlp_blocks)
    case KIND_DEFORM_ROT: RT_DISPATCH(KIND_DEFORM_ROT, launch_kind_step, a, d, n_passes, grid, rgrid, s, ev, S, mlp_blocks)
    case KIND_GANISO: RT_DISPATCH(KIND_GANISO, launch_kind_step, a, d, n_passes, grid, rgrid, s, ev, S, mlp_blocks)
    default: RT_DISPATCH(KIND_GQUAD, launch_kind_step, a, d, n_passes, grid, rgrid, s, ev, S, mlp_blocks)
    }
}

}  // namespace rti
