// Kernels of the surrogate MLP (6 -> 256 -> 256 -> 256 -> 6, SiLU): the
// first layer (K = 6) and the output layer (N = 6) in FP32 on the vector
// units (1% of the FLOPs), the two 256x256 products on the BF16 matrix
// cores with FP32 accumulation, and the AdamW update.
//
// Forward products use three-term split bf16: a value v is carried as
// hi = bf16(v) and lo = bf16(v - hi), and A B is accumulated as
// Al Bh + Ah Bl + Ah Bh (the dropped Al Bl is ~2^-16 relative), which gives
// the network near-FP32 accuracy; plain bf16 forward products leave a
// relative error floor of about 1e-3 in the learned map.  The backward
// products (signals and weight gradients) stay single bf16.
//
// A training step is four launches around the update: the forward and the
// backward pass each take a 64-row tile of one network through all layers
// in one workgroup, with the tile's activations or signals in LDS, then the
// weight gradients of both 256x256 layers, then the sums of the FP32
// layers' and biases' row partials.  What crosses memory between them is what
// the weight gradients and the backward pass need: z2, z3 (FP32) and, as
// tiles with the row running fastest, h1, h2, dz2, dz3 (bf16), which is
// the order in which a lane of the weight-gradient product takes them.
// 64 networks x 1024 rows, per training step without the data generator:
// 680 us with one launch per layer and reduction, 375 us with these.
// The arithmetic is that of the single launches, operation by operation: the
// correctly rounded quotients of the SiLUs, the order of every sum.
//
// Lane l of a 16x16x32 MFMA supplies A[l%16][8(l/16) .. 8(l/16)+7] and
// B[8(l/16) .. +7][l%16] and receives D[4(l/16) + j][l%16], j = 0..3.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "rt_internal.hpp"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// The networks are MLP_P values apart, an even but not a multiple of four:
// 16-byte accesses at the alignment of the element.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x8u __attribute__((ext_vector_type(8), aligned(2)));

constexpr int TM = 64;         // rows of a tile
constexpr int H = rti::MLP_H;  // 256
constexpr int AROW = 264;      // bf16 row of an activation tile in LDS (528 bytes: fragment reads spread over the banks)
constexpr int NT = 512;        // threads of a tile's workgroup: eight waves of 32 output columns each
constexpr int FROW = 260;      // FP32 row of a tile in LDS
// Rows per partial sum of the FP32 layers' weight gradients.
constexpr int GRAD_ROWS = 32;

// XCD-aware tile order.  Workgroups go to the 8 XCDs round-robin by their
// linear id, and each XCD has its own L2.  Tiles are numbered with x
// fastest, then y, then z, and XCD k takes the k-th contiguous eighth of that
// order, so that one network's weights and operands are read by one XCD.
// The grid is 1-D, 8 * ceil(tiles / 8) workgroups; returns false for the
// padding.
__device__ __forceinline__ bool xcd_tile(int nx, int ny, int nz, int &x, int &y, int &z) {
    const int T = nx * ny * nz;
    const int per = (T + 7) / 8;
    const int b = blockIdx.x;
    const int t = (b & 7) * per + (b >> 3);
    if ((b >> 3) >= per || t >= T) return false;
    x = t % nx;
    y = (t / nx) % ny;
    z = t / (nx * ny);
    return true;
}
inline unsigned xcd_grid(int nx, int ny, int nz) { return 8u * (unsigned)(((int64_t)nx * ny * nz + 7) / 8); }

// SiLU of N pre-activations and its parts, the quotients correctly rounded.
// The tiles are bound by vector issue, so while every |z| of the wave is at
// most ACT_FAST, where neither a quotient nor a residual can leave the normal
// range, n / d takes the hardware reciprocal of d (shared by z / d and 1 / d),
// one Newton step and two residual corrections: the sequence that a division
// compiles to, without its scaling and fix-up.  Beyond, the division itself.
// (Rounding to last place matters here: a changed bit of an activation can
// move its bf16 part by 2^-9, and a training run carries that on.)
constexpr float ACT_FAST = 80.0f;
__device__ __forceinline__ float quotient(float n, float d, float r) {
    float q = n * r;
    q = fmaf(fmaf(-d, q, n), r, q);
    return fmaf(fmaf(-d, q, n), r, q);
}
struct Act {
    float d, r;  // 1 + exp(-z); its reciprocal to about a bit of the last place
    bool fast;
    __device__ __forceinline__ Act(float z, bool f) : d(1.0f + __expf(-z)), r(0.f), fast(f) {
        if (!fast) return;
        r = __builtin_amdgcn_rcpf(d);
        r = fmaf(fmaf(-d, r, 1.0f), r, r);
    }
    __device__ __forceinline__ float over(float n) const { return fast ? quotient(n, d, r) : n / d; }
};
__device__ __forceinline__ float dsilu(float z, float s) { return s * (1.0f + z * (1.0f - s)); }
// f(fast) with fast known at compile time: whether all |z[0..N)| of the wave are
// at most ACT_FAST (a NaN passes through either way).
template <int N, class Z, class F> __device__ __forceinline__ void act_range(const Z &z, F f) {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) m = fmaxf(m, fabsf(z[i]));
    if (__ballot(m > ACT_FAST) == 0) f(std::true_type{});
    else f(std::false_type{});
}
template <int N, class Z> __device__ __forceinline__ void silu(const Z &z, float (&h)[N]) {
    act_range<N>(z, [&](auto fast) {
#pragma unroll
        for (int i = 0; i < N; ++i) h[i] = Act(z[i], fast).over(z[i]);
    });
}
// a[i] *= silu'(z[i])
template <int N, class Z> __device__ __forceinline__ void times_dsilu(const Z &z, float (&a)[N]) {
    act_range<N>(z, [&](auto fast) {
#pragma unroll
        for (int i = 0; i < N; ++i) a[i] = a[i] * dsilu(z[i], Act(z[i], fast).over(1.0f));
    });
}

// W2 and W3 of the FP32 master as the two bf16 parts, in the order a wave reads
// them as the B operand of h W^T (B(k, n) = W[n][k]): [layer][part] then
// fragment (n/16, k/32), lane, 8 consecutive k.  A thread splits 8 k.  Split
// once per call instead of by every tile, and a fragment is one contiguous
// kilobyte; rows of the master are a kilobyte apart, which spreads a load of
// sixteen of them over four of L2's sixteen channels.
__device__ __forceinline__ void split8(f32x4 u0, f32x4 u1, bf16x8 &hi, bf16x8 &lo) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v = e < 4 ? u0[e & 3] : u1[e & 3];
        hi[e] = (__bf16)v;
        lo[e] = (__bf16)(v - (float)hi[e]);
    }
}
constexpr int WSPLIT = rti::MLP_WSPLIT;
__global__ __launch_bounds__(256) void k_mlp_wsplit(const float *__restrict__ params, int64_t stride,
                                                    __bf16 *__restrict__ ws) {
    const int g = blockIdx.y, t = blockIdx.x * 256 + threadIdx.x;  // 2 layers x 16 x 8 x 64
    const int l = t >> 13, f = t & 8191, lane = f & 63;
    const int n = (f >> 9) * 16 + (lane & 15), k = ((f >> 6) & 7) * 32 + (lane >> 4) * 8;
    const float *src = params + (int64_t)g * stride + (l == 0 ? rti::OFF_W2 : rti::OFF_W3) + n * H + k;
    bf16x8 hi, lo;
    split8(*(const f32x4u *)src, *(const f32x4u *)(src + 4), hi, lo);
    __bf16 *dst = ws + (int64_t)g * WSPLIT + (int64_t)l * 2 * H * H + f * 8;
    *(bf16x8 *)dst = hi;
    *(bf16x8 *)(dst + H * H) = lo;
}

// Sum over the wave by the butterfly l ^ 32, 16, 8, 4, 2, 1, without LDS: half
// and row swaps, then rotations within rows of 16 (after the l ^ 8 step the
// rotation by 4 meets the same values as l ^ 4).
template <int CTRL> __device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float wave_sum(float v) {
    const unsigned u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const unsigned w = __float_as_uint(v);
    const auto b = __builtin_amdgcn_permlane16_swap(w, w, false, false);
    v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    v = dpp_add<0x128>(v);  // row rotation by 8
    v = dpp_add<0x124>(v);  // row rotation by 4
    v = dpp_add<0x4E>(v);   // quad permutation l ^ 2
    return dpp_add<0xB1>(v);  // l ^ 1
}

// ================================================================= forward
// Where a tile's results go for a backward pass.
struct KeepTile {
    float *x;          // [64][6] inputs
    float *z2;         // pre-activations of layer 2 in accumulator order: [wave][i][j][lane][4]
    float *z3;         // [64][256]
    __bf16 *h1t, *h2t; // [256][64]
};

// One 64-row tile (M valid rows, the rest zero inputs) of the network at Pg.
// Eight waves, wave w owning output columns [32 w, 32 w + 32) of the two
// products; the tile's activations sit in LDS as the two bf16 parts, the
// weights' two parts (Wg) stream through L2 as whole fragments, the next slice
// of 32 k on its way while the current one is multiplied.  Bound by the matrix
// cores' 3 x 16.8 MFLOP per tile next to the vector work of the SiLUs; 68 KB
// of LDS and at most 128 registers keep two workgroups, four waves per SIMD, on
// a CU, so one's vector work runs under the other's products (64 networks x
// 1024 rows: 110 us; with four waves of 64 columns, two per SIMD, 125 against
// 112 with these before the weights were split once and the quotients exact).
// DIRECT: the weights are read from the FP32 master and split by the tile, for
// networks of a single tile, whose split would be written and read back once.
template <bool KEEP, bool DIRECT = false>
__device__ __forceinline__ void forward_tile(char *smem, float (*Xs)[6], const float *__restrict__ Pg,
                                             const __bf16 *__restrict__ Wg, const float *__restrict__ X, float *__restrict__ Y, int M,
                                             const KeepTile &K) {
    __bf16(*Ah)[AROW] = reinterpret_cast<__bf16(*)[AROW]>(smem);
    __bf16(*Al)[AROW] = Ah + TM;
    float(*Hf)[FROW] = reinterpret_cast<float(*)[FROW]>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4, kq = grp * 8;
    for (int e = tid; e < TM * 6; e += NT) {
        const float v = e < 6 * M ? X[e] : 0.f;
        Xs[e / 6][e % 6] = v;
        if constexpr (KEEP) K.x[e] = v;
    }
    __syncthreads();
    {   // layer 1, FP32: thread = unit and half of the rows
        const int o = tid & (H - 1);
        const float *W = Pg + rti::OFF_W1 + o * 6;
        const float w0 = W[0], w1 = W[1], w2 = W[2], w3 = W[3], w4 = W[4], w5 = W[5];
        const float b = Pg[rti::OFF_B1 + o];
        const int rh = (tid >> 8) * (TM / 2);
#pragma unroll 1
        for (int r0 = rh; r0 < rh + TM / 2; r0 += 8) {
            float z[8], h[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int r = r0 + u;
                z[u] = b;
                z[u] = fmaf(w0, Xs[r][0], z[u]);
                z[u] = fmaf(w1, Xs[r][1], z[u]);
                z[u] = fmaf(w2, Xs[r][2], z[u]);
                z[u] = fmaf(w3, Xs[r][3], z[u]);
                z[u] = fmaf(w4, Xs[r][4], z[u]);
                z[u] = fmaf(w5, Xs[r][5], z[u]);
            }
            silu(z, h);
            bf16x8 hi;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                hi[u] = (__bf16)h[u];
                Ah[r0 + u][o] = hi[u];
                Al[r0 + u][o] = (__bf16)(h[u] - (float)hi[u]);
            }
            if constexpr (KEEP) *(bf16x8 *)(K.h1t + o * TM + r0) = hi;
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int l = 0; l < 2; ++l) {
        const __bf16 *__restrict__ W = Wg + l * 2 * H * H + (wave * 2 * 8 * 64 + lane) * 8;
        const float *__restrict__ Wf = Pg + (l == 0 ? rti::OFF_W2 : rti::OFF_W3) + (wave * 32 + col) * H + kq;
        const float *__restrict__ bias = Pg + (l == 0 ? rti::OFF_B2 : rti::OFF_B3) + wave * 32 + col;
        f32x4 acc[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        bf16x8 nh[2], nl[2];
        f32x4 nf[2][2];
        auto load = [&](int k) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if constexpr (DIRECT) {
                    const float *src = Wf + 16 * j * H + 32 * k;
                    nf[j][0] = *(const f32x4u *)src;
                    nf[j][1] = *(const f32x4u *)(src + 4);
                } else {
                    nh[j] = *(const bf16x8 *)(W + (j * 8 + k) * 64 * 8);
                    nl[j] = *(const bf16x8 *)(W + (j * 8 + k) * 64 * 8 + H * H);
                }
            }
        };
        load(0);
#pragma unroll 2
        for (int k0 = 0; k0 < H; k0 += 32) {
            bf16x8 bh[2], bl[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if constexpr (DIRECT) {
                    split8(nf[j][0], nf[j][1], bh[j], bl[j]);
                } else {
                    bh[j] = nh[j];
                    bl[j] = nl[j];
                }
            }
            load(min(k0 / 32 + 1, 7));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bf16x8 ah = *(const bf16x8 *)&Ah[16 * i + col][k0 + kq];
                const bf16x8 al = *(const bf16x8 *)&Al[16 * i + col][k0 + kq];
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[j], acc[i][j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[j], acc[i][j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[j], acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = wave * 32 + 16 * j + col;
            const float bn = bias[16 * j];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * i + 4 * grp;
                f32x4 z;
#pragma unroll
                for (int e = 0; e < 4; ++e) z[e] = acc[i][j][e] + bn;
                float h[4];
                silu(z, h);
                if (l == 0) {
                    if constexpr (KEEP) *(f32x4 *)(K.z2 + (((wave * 4 + i) * 2 + j) * 64 + lane) * 4) = z;
                    bf16x4 hi;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        hi[e] = (__bf16)h[e];
                        Ah[r + e][n] = hi[e];
                        Al[r + e][n] = (__bf16)(h[e] - (float)hi[e]);
                    }
                    if constexpr (KEEP) *(bf16x4 *)(K.h2t + n * TM + r) = hi;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (KEEP) K.z3[(r + e) * H + n] = z[e];
                        Hf[r + e][n] = h[e];
                    }
                }
            }
        }
        __syncthreads();
    }
    // output layer, FP32: one wave per row, lane l taking k = l + 64 q in order
    // of q, then the butterfly sum over the lanes, then the bias
    {
        float w4[6][4];
#pragma unroll
        for (int o = 0; o < 6; ++o)
#pragma unroll
            for (int q = 0; q < 4; ++q) w4[o][q] = Pg[rti::OFF_W4 + o * H + lane + 64 * q];
        const float b4 = lane < 6 ? Pg[rti::OFF_B4 + lane] : 0.f;
        for (int m = wave; m < M; m += NT / 64) {
            float h[4], a[6];
#pragma unroll
            for (int q = 0; q < 4; ++q) h[q] = Hf[m][lane + 64 * q];
#pragma unroll
            for (int o = 0; o < 6; ++o) {
                float t = w4[o][0] * h[0];
#pragma unroll
                for (int q = 1; q < 4; ++q) t = fmaf(w4[o][q], h[q], t);
                a[o] = wave_sum(t);
            }
            if (lane < 6) {
                float v = a[0];
#pragma unroll
                for (int o = 1; o < 6; ++o) v = lane == o ? a[o] : v;
                Y[6 * m + lane] = b4 + v;
            }
        }
    }
    __syncthreads();
}

constexpr int TILE_LDS = 2 * TM * AROW * 2;  // both bf16 parts, or one FP32 tile
static_assert(TILE_LDS >= TM * FROW * 4, "FP32 tile exceeds the LDS block");

// y = MLP(x) for n networks of B rows each, keeping what the backward needs.
template <bool DIRECT>
__global__ __launch_bounds__(NT, 4) void k_mlp_fwd(const float *__restrict__ params, const float *__restrict__ X,
                                                    float *__restrict__ Y, int n, int B, rti::MlpWork w) {
    __shared__ __attribute__((aligned(16))) char smem[TILE_LDS];
    __shared__ float Xs[TM][6];
    const int tiles = (B + TM - 1) / TM;
    int t, one, g;
    if (!xcd_tile(tiles, 1, n, t, one, g)) return;
    const int m0 = t * TM;
    const int64_t T = (int64_t)g * tiles + t;
    const KeepTile K{w.xf + T * TM * 6, w.z2 + T * TM * H, w.z3 + T * TM * H, w.h1t + T * TM * H, w.h2t + T * TM * H};
    forward_tile<true, DIRECT>(smem, Xs, params + g * rti::MLP_P, w.ws + (int64_t)g * WSPLIT, X + ((int64_t)g * B + m0) * 6, Y + ((int64_t)g * B + m0) * 6,
                       min(TM, B - m0), K);
}

// Rows grouped by network (ctl: row and tile offsets): persistent workgroups
// over the tile list.
__device__ __forceinline__ void infer_tiles(const int *__restrict__ ctl, const rti::SurrArgs &S) {
    __shared__ __attribute__((aligned(16))) char smem[TILE_LDS];
    __shared__ float Xs[TM][6];
    const int total_tiles = ctl[rti::XC_TILE + 64];
    const int lane = threadIdx.x & 63;
    for (int t = blockIdx.x; t < total_tiles; t += gridDim.x) {
        // network of tile t: the last one whose first tile is <= t
        const int toff = lane < S.n_nets ? ctl[rti::XC_TILE + lane] : 0x7fffffff;
        const int g = __builtin_amdgcn_readfirstlane(__popcll(__ballot(toff <= t)) - 1);
        const int off = ctl[rti::XC_ROW + g], cnt = ctl[rti::XC_ROW + g + 1] - off;
        const int m0 = (t - ctl[rti::XC_TILE + g]) * TM;
        forward_tile<false>(smem, Xs, S.params + (int64_t)g * S.stride, S.wsplit + (int64_t)g * WSPLIT, S.xin + 6 * (int64_t)(off + m0),
                            S.xout + 6 * (int64_t)(off + m0), min(TM, cnt - m0), KeepTile{});
    }
}

// The tracer's crossings (offsets made on the device) and a caller's rows
// (offsets by value: nothing to upload or wait for).
__global__ __launch_bounds__(NT, 4) void k_mlp_infer(const int *__restrict__ ctl, const rti::SurrArgs S) {
    infer_tiles(ctl, S);
}
__global__ __launch_bounds__(NT, 4) void k_mlp_infer_rows(const rti::GroupCtl C, const rti::SurrArgs S) {
    infer_tiles(C.w, S);
}

// ================================================================ backward
// W2 and W3 of the bf16 copy in the order a wave reads them as the B operand
// of dz W (B(k, n) = W[k][n]): fragment (n/16, k/32), lane, 8 consecutive k.
// A thread takes 8 k x 8 n.
__global__ __launch_bounds__(256) void k_mlp_wfrag(const __bf16 *__restrict__ wb, __bf16 *__restrict__ wt) {
    const int g = blockIdx.y, t = blockIdx.x * 256 + threadIdx.x;  // 2 layers x 32 x 32
    const int l = t >> 10, k8 = (t >> 5) & 31, n8 = t & 31;
    const __bf16 *src = wb + (int64_t)g * rti::MLP_P + (l == 0 ? rti::OFF_W2 : rti::OFF_W3) + k8 * 8 * H + n8 * 8;
    bf16x8 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = *(const bf16x8u *)(src + k * H);
    __bf16 *dst = wt + ((int64_t)g * 2 + l) * H * H;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        bf16x8 o;
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = v[k][n];
        const int nn = n8 * 8 + n, lane = (k8 & 3) * 16 + (nn & 15);
        *(bf16x8 *)(dst + (((nn >> 4) * 8 + (k8 >> 2)) * 64 + lane) * 8) = o;
    }
}

// acc = A W for the 64 rows of A in LDS and this wave's 32 columns; W as
// fragments, or (DIRECT, for networks of a single tile) row by row as it is.
template <bool DIRECT>
__device__ __forceinline__ void signal_product(const __bf16 (*A)[AROW], const __bf16 *__restrict__ w, int wave,
                                               int lane, f32x4 acc[4][2]) {
    const int col = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const __bf16 *__restrict__ W = DIRECT ? w + kq * H + wave * 32 + col : w + ((wave * 2) * 8 * 64 + lane) * 8;
#pragma unroll 2
    for (int k = 0; k < 8; ++k) {
        bf16x8 b[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if constexpr (DIRECT) {
#pragma unroll
                for (int e = 0; e < 8; ++e) b[j][e] = W[(32 * k + e) * H + 16 * j];
            } else {
                b[j] = *(const bf16x8 *)(W + (j * 8 + k) * 64 * 8);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bf16x8 a = *(const bf16x8 *)&A[16 * i + col][32 * k + kq];
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[j], acc[i][j], 0, 0, 0);
        }
    }
}

// A 64-row tile of one network from dy back to the first layer's gradient:
//   dz3 = (dy W4) silu'(z3), dz2 = (dz3 W3) silu'(z2), dz1 = (dz2 W2) silu'(z1),
// the signals rounded to bf16 for the products and the weight gradients,
// z1 formed again from the inputs.  Between the products the tile goes
// through LDS in FP32, and a thread walks down its column: the bias sums and
// the FP32 layers' weight-gradient partials in row order, and the column's
// bf16 values, which are contiguous in the transposed signal matrices.
// Bound by the 0.3 MB that a tile reads and writes and by the column walks.
template <bool DIRECT>
__global__ __launch_bounds__(NT, 4) void k_mlp_bwd(const float *__restrict__ params, const __bf16 *__restrict__ wb,
                                                   const float *__restrict__ DY, int n, int B, rti::MlpWork w) {
    __shared__ __attribute__((aligned(16))) char smem[TILE_LDS];
    __shared__ float Xs[TM][6], Ds[TM][6], S0[H];
    __bf16(*A)[AROW] = reinterpret_cast<__bf16(*)[AROW]>(smem);
    float(*F)[FROW] = reinterpret_cast<float(*)[FROW]>(smem);
    const int tiles = (B + TM - 1) / TM, nch = (B + GRAD_ROWS - 1) / GRAD_ROWS;
    int t, one, g;
    if (!xcd_tile(tiles, 1, n, t, one, g)) return;
    const int m0 = t * TM, M = min(TM, B - m0);
    const int64_t T = (int64_t)g * tiles + t;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    // the column walks: column c, rows [32 half, 32 half + 32)
    const int c = tid & (H - 1), half = tid >> 8, rh = half * GRAD_ROWS;
    const float *__restrict__ Pg = params + g * rti::MLP_P;
    const float *__restrict__ dy = DY + ((int64_t)g * B + m0) * 6;
    for (int e = tid; e < TM * 6; e += NT) {
        Xs[e / 6][e % 6] = w.xf[T * TM * 6 + e];
        Ds[e / 6][e % 6] = e < 6 * M ? dy[e] : 0.f;
    }
    __syncthreads();
    auto write_part = [&](float *part, const float a[7]) {
        const int ch = 2 * t + half;
        if (ch < nch) {
            float *dst = part + ((int64_t)g * nch + ch) * 7 * H + c;
#pragma unroll
            for (int i = 0; i < 7; ++i) dst[i * H] = a[i];
        }
    };
    // a column's sum over the tile's rows in order (called by all threads)
    auto column_sum = [&](const float (&v)[GRAD_ROWS], float *out) {
        float s = 0.f;
        if (half == 0) {
#pragma unroll
            for (int u = 0; u < GRAD_ROWS; ++u) s += v[u];
            S0[c] = s;
        }
        __syncthreads();
        if (half == 1) {
            s = S0[c];
#pragma unroll
            for (int u = 0; u < GRAD_ROWS; ++u) s += v[u];
            out[T * H + c] = s;
        }
    };
    {   // output layer
        float w4[6], a[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, dz[GRAD_ROWS];
#pragma unroll
        for (int o = 0; o < 6; ++o) w4[o] = Pg[rti::OFF_W4 + o * H + c];
        const float *__restrict__ z3 = w.z3 + (T * TM + rh) * H + c;
        __bf16 *__restrict__ dzt = w.dz3t + (T * H + c) * TM + rh;
        // (dz: first the column of z3, then, row by row, its signal)
#pragma unroll
        for (int u = 0; u < GRAD_ROWS; ++u) dz[u] = z3[u * H];
        act_range<GRAD_ROWS>(dz, [&](auto fast) {
#pragma unroll
            for (int r0 = 0; r0 < GRAD_ROWS; r0 += 8) {
                bf16x8 pk;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int m = rh + r0 + u;
                    const float z = dz[r0 + u];
                    const Act t(z, fast);
                    const float h = t.over(z);
                    float dh = 0.f;
#pragma unroll
                    for (int o = 0; o < 6; ++o) {
                        const float d = Ds[m][o];
                        dh = fmaf(d, w4[o], dh);
                        a[o] = fmaf(d, h, a[o]);
                    }
                    dz[r0 + u] = dh * dsilu(z, t.over(1.0f));
                    pk[u] = (__bf16)dz[r0 + u];
                    A[m][c] = pk[u];
                    if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (four rows in registers at a time)
                }
                *(bf16x8 *)(dzt + r0) = pk;
            }
        });
        if (c < 6)
            for (int u = 0; u < GRAD_ROWS; ++u) a[6] += Ds[rh + u][c];
        write_part(w.part4, a);
        column_sum(dz, w.cs3);
    }
    // (column_sum's barrier: the tile of signals is complete)
    f32x4 acc[4][2];
    const __bf16 *__restrict__ wg = wb + g * rti::MLP_P;
    signal_product<DIRECT>(A, DIRECT ? wg + rti::OFF_W3 : w.wt + ((int64_t)g * 2 + 1) * H * H, wave, lane, acc);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const f32x4 z = *(const f32x4 *)(w.z2 + T * TM * H + (((wave * 4 + i) * 2 + j) * 64 + lane) * 4);
            float d[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            times_dsilu(z, d);
#pragma unroll
            for (int e = 0; e < 4; ++e) F[16 * i + 4 * grp + e][wave * 32 + 16 * j + col] = d[e];
            __builtin_amdgcn_sched_barrier(0);  // (keeps the unrolled tiles from holding all of z at once)
        }
    __syncthreads();
    {
        float dz[GRAD_ROWS];
        bf16x8 pk[GRAD_ROWS / 8];
        __bf16 *__restrict__ dzt = w.dz2t + (T * H + c) * TM + rh;
#pragma unroll
        for (int q = 0; q < GRAD_ROWS / 8; ++q) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                dz[8 * q + u] = F[rh + 8 * q + u][c];
                pk[q][u] = (__bf16)dz[8 * q + u];
            }
            *(bf16x8 *)(dzt + 8 * q) = pk[q];
            __builtin_amdgcn_sched_barrier(0);
        }
        column_sum(dz, w.cs2);  // its barrier: the FP32 tile has been read
#pragma unroll
        for (int q = 0; q < GRAD_ROWS / 8; ++q)
#pragma unroll
            for (int u = 0; u < 8; ++u) A[rh + 8 * q + u][c] = pk[q][u];
    }
    __syncthreads();
    signal_product<DIRECT>(A, DIRECT ? wg + rti::OFF_W2 : w.wt + ((int64_t)g * 2) * H * H, wave, lane, acc);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int n1 = wave * 32 + 16 * j + col;
        float w1[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) w1[q] = Pg[rti::OFF_W1 + n1 * 6 + q];
        const float b1 = Pg[rti::OFF_B1 + n1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * i + 4 * grp;
            float z[4], d[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                z[e] = b1;
#pragma unroll
                for (int q = 0; q < 6; ++q) z[e] = fmaf(w1[q], Xs[r + e][q], z[e]);
                d[e] = acc[i][j][e];
            }
            times_dsilu(z, d);
#pragma unroll
            for (int e = 0; e < 4; ++e) F[r + e][n1] = d[e];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();
    {   // first layer
        float a[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int u = 0; u < GRAD_ROWS; ++u) {
            const float d = F[rh + u][c];
#pragma unroll
            for (int q = 0; q < 6; ++q) a[q] = fmaf(d, Xs[rh + u][q], a[q]);
            a[6] += d;
        }
        write_part(w.part1, a);
    }
}

// Weight gradients of both 256x256 layers: dW[o][i] = sum_b dz[b][o] h[b][i],
// with dz and h as [256][64] tiles, so that a lane's eight consecutive b of
// an operand are one 16-byte load and nothing is transposed here.  A 64x64
// tile of one layer of one network per block; bound by the 256 KB that the tile
// of a batch of 1024 reads through L2.
struct WgradTile {
    const __bf16 *A, *B;  // this lane's first element of the tile's dz and h columns
    float *C;
};
__device__ __forceinline__ bool wgrad_tile(int n, int tiles, const rti::MlpWork &w, float *grad, WgradTile &t) {
    int tx, ty, gl;
    if (!xcd_tile(4, 4, 2 * n, tx, ty, gl)) return false;
    const int g = gl >> 1, l = gl & 1, m0 = ty * 64, n0 = tx * 64, lane = threadIdx.x & 63;
    const int64_t base = ((int64_t)g * tiles * H + (lane & 15)) * TM + (lane >> 4) * 8;
    t.A = (l ? w.dz3t : w.dz2t) + base + m0 * TM;
    t.B = (l ? w.h2t : w.h1t) + base + n0 * TM;
    t.C = grad + g * rti::MLP_P + (l ? rti::OFF_W3 : rti::OFF_W2) + (int64_t)m0 * H + n0;
    return true;
}

// Batches of whole 128 rows: the four waves split the batch in contiguous
// quarters, each accumulating the whole tile (4x4 16x16x32 MFMA tiles) straight
// from L2, and the partial tiles are added in a fixed order,
// (w0 + w2) + (w1 + w3).
__global__ __launch_bounds__(256, 4) void k_mlp_wgrad(int n, int tiles, rti::MlpWork w, float *__restrict__ grad) {
    __shared__ __attribute__((aligned(16))) float R[2][64][64];
    WgradTile t;
    if (!wgrad_tile(n, tiles, w, grad, t)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int ns = 2 * tiles, s0 = ns * wave / 4, s1 = ns * (wave + 1) / 4;
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 a[4], b[4];
    auto load = [&](int s) {
        const int64_t o = (int64_t)(s >> 1) * TM * H + (s & 1) * 32;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = *(const bf16x8 *)(t.A + o + 16 * i * TM);
            b[i] = *(const bf16x8 *)(t.B + o + 16 * i * TM);
        }
    };
    load(s0);
#pragma unroll 2
    for (int s = s0; s < s1; ++s) {
        bf16x8 ca[4], cb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ca[i] = a[i];
            cb[i] = b[i];
        }
        load(s + 1 < s1 ? s + 1 : s);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ca[i], cb[j], acc[i][j], 0, 0, 0);
    }
    // (32 KB of LDS: four workgroups on a CU)
    auto each = [&](auto f) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) f(R[wave & 1][16 * i + 4 * grp + e][16 * j + col], acc[i][j][e]);
    };
    if (wave >= 2) each([](float &r, float v) { r = v; });
    __syncthreads();
    if (wave < 2) each([](float &r, float v) { r = v + r; });
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = q * 16 + (tid >> 4), c = (tid & 15) * 4;
        const f32x4 v0 = *(const f32x4 *)&R[0][r][c], v1 = *(const f32x4 *)&R[1][r][c];
        *(f32x4u *)(t.C + (int64_t)r * H + c) = v0 + v1;
    }
}

// Other batches: one chain of sums through the whole batch in order, each wave a
// 32x32 corner of the tile.  The waves share the operands through LDS, whole
// fragments as the lanes loaded them, the next 64 rows on their way while the
// current ones are multiplied (37 networks x 1329 rows: 109 us with every wave
// loading its own operands, 74 with these; the four quarters, which would
// round differently, 68).
__global__ __launch_bounds__(256, 4) void k_mlp_wgrad_rows(int n, int tiles, int slices, rti::MlpWork w, float *__restrict__ grad) {
    __shared__ bf16x8 S[2][2][2][4][64];  // [buffer][slice of 32 rows][A or B][16 columns][lane]
    WgradTile t;
    if (!wgrad_tile(n, tiles, w, grad, t)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave >> 1) * 2, wn = (wave & 1) * 2;  // in tiles of 16
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // wave: slice wave >> 1 of operand wave & 1
    const __bf16 *__restrict__ src = (wave & 1 ? t.B : t.A) + (wave >> 1) * 32;
    bf16x8 v[4] = {};
    auto load = [&](int q) {
        if (2 * q + (wave >> 1) >= slices) return;  // (padding rows alone: not multiplied)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *(const bf16x8 *)(src + (int64_t)q * TM * H + 16 * i * TM);
    };
    auto store = [&](int q) {
#pragma unroll
        for (int i = 0; i < 4; ++i) S[q & 1][wave >> 1][wave & 1][i][lane] = v[i];
    };
    load(0);
    store(0);
    load(min(1, tiles - 1));
    __syncthreads();
    for (int q = 0; q < tiles; ++q) {
        bf16x8 a[2][2], b[2][2];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[s][i] = S[q & 1][s][0][wm + i][lane];
                b[s][i] = S[q & 1][s][1][wn + i][lane];
            }
        // the other buffer was read before the last barrier
        store(q + 1);
        load(min(q + 2, tiles - 1));
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (2 * q + s >= slices) break;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s][i], b[s][j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }
    // the tile through LDS (free after the last barrier) to whole rows
    float(*R)[68] = reinterpret_cast<float(*)[68]>(&S[0][0][0][0][0]);
    static_assert(sizeof(S) >= 64 * 68 * sizeof(float), "output tile exceeds the staging block");
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) R[(wm + i) * 16 + 4 * (lane >> 4) + e][(wn + j) * 16 + (lane & 15)] = acc[i][j][e];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = q * 16 + (threadIdx.x >> 4), c = (threadIdx.x & 15) * 4;
        *(f32x4u *)(t.C + (int64_t)r * H + c) = *(const f32x4 *)&R[r][c];
    }
}

// Sums of the row partials in order: block (q, g) takes one of the 16 sums of
// network g, thread = unit.
__global__ __launch_bounds__(256) void k_mlp_sums(int B, rti::MlpWork w, float *__restrict__ grad) {
    const int q = blockIdx.x, g = blockIdx.y, o = threadIdx.x;
    const int tiles = (B + TM - 1) / TM, nch = (B + GRAD_ROWS - 1) / GRAD_ROWS;
    const float *__restrict__ src;
    int cnt, stride;
    if (q < 14) {
        src = (q < 7 ? w.part1 : w.part4) + ((int64_t)g * nch * 7 + (q < 7 ? q : q - 7)) * H + o;
        cnt = nch;
        stride = 7 * H;
    } else {
        src = (q == 14 ? w.cs2 : w.cs3) + (int64_t)g * tiles * H + o;
        cnt = tiles;
        stride = H;
    }
    float s = 0.f;
#pragma unroll 8
    for (int c = 0; c < cnt; ++c) s += src[(int64_t)c * stride];
    float *__restrict__ G = grad + (int64_t)g * rti::MLP_P;
    if (q < 6) G[rti::OFF_W1 + o * 6 + q] = s;
    else if (q == 6) G[rti::OFF_B1 + o] = s;
    else if (q < 13) G[rti::OFF_W4 + (q - 7) * H + o] = s;
    else if (q == 13) {
        if (o < 6) G[rti::OFF_B4 + o] = s;
    } else G[(q == 14 ? rti::OFF_B2 : rti::OFF_B3) + o] = s;
}

// AdamW with bias correction; refreshes the bf16 copy of the parameters.
__global__ void k_adamw(float *__restrict__ p, __bf16 *__restrict__ pb, float *__restrict__ m, float *__restrict__ v,
                        const float *__restrict__ gr, int64_t n, float lr, float b1, float b2, float eps, float wd,
                        float c1, float c2) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        float g = gr[i];
        float mi = b1 * m[i] + (1.f - b1) * g;
        float vi = b2 * v[i] + (1.f - b2) * g * g;
        m[i] = mi;
        v[i] = vi;
        float pi = p[i] - lr * ((mi * c1) / (sqrtf(vi * c2) + eps) + wd * p[i]);
        p[i] = pi;
        pb[i] = (__bf16)pi;
    }
}

// dy = 2 (y - t) / batch and per-block squared-error sums in a fixed order: 256
// chains, each adding its elements in order, then a tree.  A chain's elements
// are loaded by four threads, MSE_LOADS each at once, and pass through LDS (64
// networks x 1024 rows: 13.6 us with the chain's thread loading them, 6.2
// with these).
constexpr int MSE_LOADS = 6;
__global__ __launch_bounds__(1024) void k_mse_grad(const float *__restrict__ y, const float *__restrict__ t,
                                                  float *__restrict__ dy, int64_t n, float inv_batch,
                                                  float *__restrict__ part) {
    __shared__ float D[4 * MSE_LOADS][256], sh[256];
    const int lane = threadIdx.x & 255, q = threadIdx.x >> 8;
    const int64_t stride = (int64_t)gridDim.x * 256;
    float acc = 0.f;
    for (int64_t i0 = blockIdx.x * 256; i0 < n; i0 += 4 * MSE_LOADS * stride) {
        const int64_t i = i0 + lane + q * stride;
        float a[MSE_LOADS], b[MSE_LOADS];
#pragma unroll
        for (int u = 0; u < MSE_LOADS; ++u) {
            const int64_t k = min(i + 4 * u * stride, n - 1);
            a[u] = y[k];
            b[u] = t[k];
        }
#pragma unroll
        for (int u = 0; u < MSE_LOADS; ++u) {
            const float d = a[u] - b[u];
            D[4 * u + q][lane] = d;
            if (i + 4 * u * stride < n) dy[i + 4 * u * stride] = 2.f * d * inv_batch;
        }
        __syncthreads();
        if (q == 0) {
#pragma unroll
            for (int u = 0; u < 4 * MSE_LOADS; ++u) {
                const float d = D[u][lane];
                if (i + u * stride < n) acc += d * d;
            }
        }
        __syncthreads();
    }
    if (q == 0) sh[lane] = acc;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

}  // namespace

namespace rti {

hipError_t launch_adamw(float *p, __bf16 *pb, float *m, float *v, const float *g, int64_t n, float lr, float b1,
                        float b2, float eps, float wd, int step, hipStream_t s) {
    float c1 = 1.0f / (1.0f - powf(b1, (float)step)), c2 = 1.0f / (1.0f - powf(b2, (float)step));
    int blocks = (int)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_adamw, dim3(blocks), dim3(256), 0, s, p, pb, m, v, g, n, lr, b1, b2, eps, wd, c1, c2);
    return hipGetLastError();
}

hipError_t launch_mse_grad(const float *y, const float *t, float *dy, int64_t n, int batch, float *part, int nblk,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_mse_grad, dim3(nblk), dim3(1024), 0, s, y, t, dy, n, 1.0f / (float)batch, part);
    return hipGetLastError();
}

// Networks whose re-laid weights the workspace holds at once (0.5 MB each; larger
// calls take their networks in turns of this many).  Networks of a single tile
// need none, and go in one turn: their tiles read the weights as they are (forward
// and backward of 2048 networks of 4 rows 0.75 + 1.19 ms with re-laid weights,
// 0.41 + 0.67 as they are; 64 of 16 rows 0.054 + 0.070, and 0.047 + 0.059).
constexpr int MLP_TURN = 256;
static int networks_a_turn(int n, int batch) { return batch <= TM ? n : std::min(n, MLP_TURN); }

// Workspace of n networks of batch rows: the tiles are whole, their rows past
// the batch hold the forward of zero inputs and zero signals.  The forward's and
// the backward's weights share their room: each pass lays them out first.
template <class F> static void mlp_layout(int n, int batch, MlpWork &w, F take) {
    const size_t tiles = ((size_t)batch + TM - 1) / TM, nch = ((size_t)batch + GRAD_ROWS - 1) / GRAD_ROWS;
    const size_t rows = (size_t)n * tiles * TM;
    w.xf = (float *)take(rows * MLP_IN * 4);
    w.z2 = (float *)take(rows * MLP_H * 4);
    w.z3 = (float *)take(rows * MLP_H * 4);
    w.h1t = (__bf16 *)take(rows * MLP_H * 2);
    w.h2t = (__bf16 *)take(rows * MLP_H * 2);
    w.dz2t = (__bf16 *)take(rows * MLP_H * 2);
    w.dz3t = (__bf16 *)take(rows * MLP_H * 2);
    w.ws = w.wt = (__bf16 *)take(batch <= TM ? 0 : (size_t)networks_a_turn(n, batch) * MLP_WSPLIT * 2);
    w.part1 = (float *)take(n * nch * 7 * MLP_H * 4);
    w.part4 = (float *)take(n * nch * 7 * MLP_H * 4);
    w.cs2 = (float *)take(n * tiles * MLP_H * 4);
    w.cs3 = (float *)take(n * tiles * MLP_H * 4);
}

size_t mlp_work_bytes(int n_nets, int batch) {
    size_t total = 0;
    MlpWork w;
    mlp_layout(n_nets, batch, w, [&](size_t bytes) {
        total += (bytes + 255) & ~(size_t)255;
        return (void *)nullptr;
    });
    return total;
}

void mlp_work_carve(void *base, int n_nets, int batch, MlpWork &w) {
    char *p = (char *)base;
    mlp_layout(n_nets, batch, w, [&](size_t bytes) {
        char *r = p;
        p += (bytes + 255) & ~(size_t)255;
        return (void *)r;
    });
}

// The workspace from network g on.
static MlpWork from_net(MlpWork w, int64_t g, int B) {
    const int64_t tiles = (B + TM - 1) / TM, nch = (B + GRAD_ROWS - 1) / GRAD_ROWS, e = g * tiles * TM * MLP_H;
    w.xf += g * tiles * TM * MLP_IN;
    w.z2 += e;
    w.z3 += e;
    w.h1t += e;
    w.h2t += e;
    w.dz2t += e;
    w.dz3t += e;
    w.part1 += g * nch * 7 * MLP_H;
    w.part4 += g * nch * 7 * MLP_H;
    w.cs2 += g * tiles * MLP_H;
    w.cs3 += g * tiles * MLP_H;
    return w;
}

void launch_wsplit(const float *params, int64_t stride, int n, __bf16 *ws, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_wsplit, dim3(64, n), dim3(256), 0, s, params, stride, ws);
}

// y = MLP(x) for n_nets networks of batch rows each, keeping what a backward
// pass needs in the workspace.
hipError_t mlp_forward(int n, int B, const float *params, const float *x, float *y, const MlpWork &work, hipStream_t s) {
    const int turn = networks_a_turn(n, B);
    for (int64_t g = 0; g < n; g += turn) {
        const int m = (int)std::min<int64_t>(turn, n - g);
        const MlpWork w = from_net(work, g, B);
        const float *p = params + g * MLP_P;
        const float *xg = x + g * B * MLP_IN;
        float *yg = y + g * B * MLP_OUT;
        const dim3 grid(xcd_grid((B + TM - 1) / TM, 1, m));
        if (B <= TM) {
            hipLaunchKernelGGL(k_mlp_fwd<true>, grid, dim3(NT), 0, s, p, xg, yg, m, B, w);
        } else {
            launch_wsplit(p, MLP_P, m, w.ws, s);
            hipLaunchKernelGGL(k_mlp_fwd<false>, grid, dim3(NT), 0, s, p, xg, yg, m, B, w);
        }
    }
    return hipGetLastError();
}

// grad = dL/dparams given dy = dL/dy, using the workspace of the last forward.
hipError_t mlp_backward(int n, int B, const __bf16 *wb, const float *params, const float *dy, float *grad,
                        const MlpWork &work, hipStream_t s) {
    const int tiles = (B + TM - 1) / TM;
    const int turn = networks_a_turn(n, B);
    for (int64_t g = 0; g < n; g += turn) {
        const int m = (int)std::min<int64_t>(turn, n - g);
        const MlpWork w = from_net(work, g, B);
        float *G = grad + g * MLP_P;
        const float *p = params + g * MLP_P, *d = dy + g * B * MLP_OUT;
        const __bf16 *b = wb + g * MLP_P;
        const dim3 grid(xcd_grid(tiles, 1, m));
        if (tiles == 1) {
            hipLaunchKernelGGL(k_mlp_bwd<true>, grid, dim3(NT), 0, s, p, b, d, m, B, w);
        } else {
            hipLaunchKernelGGL(k_mlp_wfrag, dim3(8, m), dim3(256), 0, s, b, w.wt);
            hipLaunchKernelGGL(k_mlp_bwd<false>, grid, dim3(NT), 0, s, p, b, d, m, B, w);
        }
        if (B % 128 == 0)
            hipLaunchKernelGGL(k_mlp_wgrad, dim3(xcd_grid(4, 4, 2 * m)), dim3(256), 0, s, m, tiles, w, G);
        else
            hipLaunchKernelGGL(k_mlp_wgrad_rows, dim3(xcd_grid(4, 4, 2 * m)), dim3(256), 0, s, m, tiles, (B + 31) / 32, w, G);
        hipLaunchKernelGGL(k_mlp_sums, dim3(16, m), dim3(256), 0, s, B, w, G);
    }
    return hipGetLastError();
}

hipError_t launch_mlp_rows(const GroupCtl &C, const SurrArgs &S, int blocks, hipStream_t s) {
    launch_wsplit(S.params, S.stride, S.n_nets, const_cast<__bf16 *>(S.wsplit), s);
    hipLaunchKernelGGL(k_mlp_infer_rows, dim3(blocks), dim3(NT), 0, s, C, S);
    return hipGetLastError();
}

hipError_t launch_mlp_grouped(const int *ctl, const SurrArgs &S, int blocks, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_infer, dim3(blocks), dim3(NT), 0, s, ctl, S);
    return hipGetLastError();
}

}  // namespace rti
