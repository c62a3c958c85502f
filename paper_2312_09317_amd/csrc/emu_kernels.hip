// Kernels of the summary-statistics emulator: a 6 -> 256 -> 256 -> 256 -> 8
// MLP with the exact (erf) GELU after each hidden layer, bf16 operands on the
// gfx950 matrix cores with fp32 accumulation, fp32 master weights and Adam.
//
// Every product uses v_mfma_f32_16x16x32_bf16, its k-steps in increasing
// order.  For that instruction lane l supplies row l % 16 of the A tile and
// column l % 16 of the B tile, eight consecutive k each (k block l / 16, the
// same for A and B, so the pairing of k between the two operands is fixed
// whatever order the unit adds them in), and receives rows 4 (l / 16) ..
// 4 (l / 16) + 3 of column l % 16 of the 16 x 16 result.
//
// A forward pass is one launch, a training step two (three past 1,024 rows):
// rows_kernel takes a few batch rows through every layer, forward and back,
// the activations in LDS; grads_kernel reduces over the batch and applies
// Adam.
#include <type_traits>

#include "emu_internal.hpp"

namespace cpm {
namespace emu {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// fp32 -> bf16, round to nearest even (the hardware conversion).
__device__ __forceinline__ uint16_t to_bf16(float f)
{
    const __bf16 h = (__bf16)f;
    uint16_t u;
    __builtin_memcpy(&u, &h, 2);
    return u;
}

// 1 + erf(z / sqrt 2), twice the standard normal distribution function of z.
__device__ __forceinline__ float twice_phi(float z) { return 1.0f + erff(z * 0.70710678118654752f); }

// GELU(z) = z Phi(z), with tp = twice_phi(z).
__device__ __forceinline__ float gelu(float z, float tp) { return 0.5f * z * tp; }

// d/dz z Phi(z) = Phi(z) + z phi(z).
__device__ __forceinline__ float gelu_grad(float z, float tp)
{
    return 0.5f * tp + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

__device__ __forceinline__ bf16x8 load8(const uint16_t *p)
{
    const uint4 v = *reinterpret_cast<const uint4 *>(p);
    bf16x8 r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Workgroup barrier over LDS only: weights on their way from memory, and
// stores on their way to it, stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Target transform of output c: log(t + off) when its offset is positive.
__device__ __forceinline__ float to_target_space(float t, float off) { return off > 0.f ? logf(t + off) : t; }
__device__ __forceinline__ float from_target_space(float u, float off) { return off > 0.f ? expf(u) - off : u; }

// All layers of a few batch rows, MT tiles of RV rows, on one workgroup of
// WAVES waves, each holding 16 / WAVES of a layer's 16-column tiles.
//
// The launches of one product each that this replaces (4 forward, 25 a
// training step) waited on each other and passed activations, their
// transposes and pre-activations through memory: 137 us a training step of
// 256 rows, 200 us a forward pass of 65,536 (now 21 and 77).  Here the
// activations stay in LDS, pre-activations in registers, and the next layer's weights load while
// a layer is worked on (MT = 1).  What is left: at 65,536 rows the issue of
// the GELUs (about 45 instructions per hidden unit and row); at a few hundred rows
// the weights' way into each CU (0.6 MB forward and back) and the chain of
// layers.
//
// RV = 4 spreads a small batch over four times the workgroups: the A tile
// repeats its four rows, so every lane group of the result holds all four and
// group g keeps row g, one element per lane instead of four on a quarter of
// the CUs.
template <int RV, int MT, int WAVES, bool TRAIN>
__global__ void __launch_bounds__(64 * WAVES) rows_kernel(RowArgs a)
{
    static_assert(RV == 4 || RV == kTile, "rows per tile: all, or one per lane group");
    static_assert(WAVES >= MT, "the last layer takes a wave per tile of rows");
    constexpr int R = RV * MT, NT = kHidden / kTile / WAVES, KS = kHidden / kStep;
    constexpr int E = RV == kTile ? 4 : 1;  // rows of a result tile per lane
    constexpr int kPitch = kHidden + 8;     // row stride 4 banks past a multiple of all: conflict-free 16-byte reads
    constexpr bool kPrefetch = MT == 1;
    __shared__ __align__(16) uint16_t act[R * kPitch];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, col = lane & 15, grp = lane >> 4;
    const int row0 = blockIdx.x * R;
    const int steps = a.n_pad / kStep;  // k-steps of the transposed operands

    // fragments of layer operand w for this wave's column tiles
    auto load_w = [&](const uint16_t *w, auto &f) {
        constexpr int K = sizeof(f[0]) / sizeof(f[0][0]);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int k = 0; k < K; ++k) f[t][k] = load8(w + ((size_t)(wave * NT + t) * K + k) * (kTile * kStep) + lane * 8);
    };
    bf16x8 f1[NT][1], fa[NT][KS], fb[NT][KS], f4[KS];
    float bias[3][NT];
    load_w(a.c.w[0], f1);
    if (kPrefetch) load_w(a.c.w[1], fa);
    const int64_t b_at[4] = {kB1, kB2, kB3, kB4};
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int t = 0; t < NT; ++t) bias[l][t] = a.params[b_at[l] + (wave * NT + t) * kTile + col];

    // z-scored inputs, zero beyond column 6 and row n
    for (int i = tid; i < R * kInPad; i += 64 * WAVES) {
        const int r = i / kInPad, c = i % kInPad, m = row0 + r;
        float v = 0.f;
        if (m < a.n && c < kIn) v = (a.x[(size_t)m * kIn + c] - a.norm[c]) / a.norm[kIn + c];
        const uint16_t b = to_bf16(v);
        act[r * kPitch + c] = b;
        if (TRAIN && c < kTile) a.in_t[0][frag_at(c, m, steps)] = b;
    }
    lds_barrier();

    f32x4 acc[MT][NT];
    // acc = rows in LDS . operand, K k-steps
    auto a_frag = [&](int mt, int k) { return load8(act + (mt * RV + col % RV) * kPitch + k * kStep + grp * 8); };
    auto product = [&](auto &f) {
        constexpr int K = sizeof(f[0]) / sizeof(f[0][0]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const bf16x8 x = a_frag(mt, k);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[mt][t] = mfma(x, f[t][k], acc[mt][t]);
            }
    };
    // element e of this lane in a result tile, and its row
    auto element = [&](const f32x4 &v, int e) {
        if (E == 4) return v[e];
        const float lo = grp & 1 ? v[1] : v[0], hi = grp & 1 ? v[3] : v[2];
        return grp & 2 ? hi : lo;
    };
    auto row_of = [&](int mt, int e) { return mt * RV + (E == 4 ? 4 * grp + e : grp); };
    // this lane's values of one column to LDS (row-major) and, in training,
    // to the transposed operand
    auto put = [&](int mt, int n, const uint16_t (&h)[E], uint16_t *t_out) {
#pragma unroll
        for (int e = 0; e < E; ++e) act[row_of(mt, e) * kPitch + n] = h[e];
        if (TRAIN) {
            uint16_t *o = t_out + frag_at(n, row0 + row_of(mt, 0), steps);
            if constexpr (E == 4) {
                ushort4 v;
                v.x = h[0], v.y = h[1], v.z = h[2], v.w = h[3];
                *reinterpret_cast<ushort4 *>(o) = v;
            } else {
                *o = h[0];
            }
        }
    };
    float z[3][TRAIN ? MT : 1][TRAIN ? NT : 1][E], tp[3][TRAIN ? MT : 1][TRAIN ? NT : 1][E];
    auto hidden = [&](int l) {
        lds_barrier();  // every wave has read the layer's input
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                uint16_t h[E];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const float v = element(acc[mt][t], e) + bias[l][t];
                    const float p = twice_phi(v);
                    h[e] = to_bf16(gelu(v, p));
                    if (TRAIN) z[l][mt][t][e] = v, tp[l][mt][t][e] = p;
                }
                put(mt, (wave * NT + t) * kTile + col, h, TRAIN ? a.in_t[l + 1] : nullptr);
            }
        lds_barrier();
    };
    product(f1);
    hidden(0);
    if (kPrefetch) load_w(a.c.w[2], fb);
    else load_w(a.c.w[1], fa);
    product(fa);
    hidden(1);
    if (!kPrefetch) load_w(a.c.w[2], fb);
    if (TRAIN) load_w(a.c.wt[3], f1), load_w(a.c.wt[2], fa);
    if (wave < MT) {
#pragma unroll
        for (int k = 0; k < KS; ++k) f4[k] = load8(a.c.w[3] + (size_t)k * (kTile * kStep) + lane * 8);
    }
    product(fb);
    hidden(2);
    if (TRAIN) load_w(a.c.wt[1], fb);

    // last layer: one column tile, a wave per tile of rows
    if (wave < MT) {
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k) o = mfma(a_frag(wave, k), f4[k], o);
        const bool real = col < kOut;
        const float b4 = real ? a.params[kB4 + col] : 0.f;
        const float *mean = a.norm + 2 * kIn, *sd = mean + kOut, *off = sd + kOut;
        const float mean_c = real ? mean[col] : 0.f, sd_c = real ? sd[col] : 1.f, off_c = real ? off[col] : 0.f;
        const float scale = 2.0f / (float)((int64_t)a.n * kOut);
        float loss = 0.f;
        uint16_t h[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int m = row0 + row_of(wave, e);
            const float y = element(o, e) + b4;
            float d = 0.f;
            if (real && m < a.n) {
                if (TRAIN) {
                    const float t = (to_target_space(a.targets[(size_t)m * kOut + col], off_c) - mean_c) / sd_c;
                    const float err = y - t;
                    loss += err * err;
                    d = scale * err;
                } else {
                    a.y[(size_t)m * kOut + col] = from_target_space(y * sd_c + mean_c, off_c);
                }
            }
            h[e] = to_bf16(d);
        }
        if (TRAIN) {
            // dL/dz of the last layer: columns 8..31 zero; only this wave
            // reads or writes these rows since the last barrier
            put(wave, col, h, a.dz_t[3]);
#pragma unroll
            for (int e = 0; e < E; ++e) act[row_of(wave, e) * kPitch + kTile + col] = 0;
#pragma unroll
            for (int k = 32; k > 0; k >>= 1) loss += __shfl_xor(loss, k, 64);
            if (lane == 0) a.loss_part[blockIdx.x * MT + wave] = loss;
        }
    }
    if constexpr (TRAIN) {
        // dL/dz of a hidden layer: (dL/dz of the next . its weights) GELU'(z)
        auto back = [&](int l) {
            lds_barrier();
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    uint16_t h[E];
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        h[e] = to_bf16(element(acc[mt][t], e) * gelu_grad(z[l][mt][t][e], tp[l][mt][t][e]));
                    put(mt, (wave * NT + t) * kTile + col, h, a.dz_t[l]);
                }
            lds_barrier();
        };
        lds_barrier();
        product(f1);
        back(2);
        product(fa);
        back(1);
        product(fb);
        back(0);
    }
}

__device__ __forceinline__ void put_copies(const Copies &c, int64_t i, float p)
{
    int l, o, k;
    if (i < kB1) l = 0, o = (int)i / kIn, k = (int)i - o * kIn;
    else if (i >= kW2 && i < kB2) l = 1, o = (int)(i - kW2) / kHidden, k = (int)(i - kW2) % kHidden;
    else if (i >= kW3 && i < kB3) l = 2, o = (int)(i - kW3) / kHidden, k = (int)(i - kW3) % kHidden;
    else if (i >= kW4 && i < kB4) l = 3, o = (int)(i - kW4) / kHidden, k = (int)(i - kW4) % kHidden;
    else return;  // biases have no copies
    const uint16_t b = to_bf16(p);
    c.w[l][frag_at(o, k, l == 0 ? kInPad / kStep : kHidden / kStep)] = b;
    if (l > 0) c.wt[l][frag_at(k, o, l == 3 ? kOutPad / kStep : kHidden / kStep)] = b;
}

// Parameter i and its Adam moments.
struct Moments {
    float p, m, v;
};
__device__ __forceinline__ Moments moments_of(const AdamArgs &a, int64_t i) { return {a.param[i], a.m[i], a.v[i]}; }

// Adam with bias correction on fp32 master parameter i, then its bf16 copies.
__device__ __forceinline__ void adam_step(const AdamArgs &a, int64_t i, Moments s, float g)
{
    const float m = a.beta1 * s.m + a.one_minus_beta1 * g;
    const float v = a.beta2 * s.v + a.one_minus_beta2 * g * g;
    a.m[i] = m;
    a.v[i] = v;
    const float p = s.p - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
    a.param[i] = p;
    put_copies(a.c, i, p);
}

__device__ __forceinline__ void put_grad(const GradArgs &g, int64_t i, float v)
{
    g.grad[i] = v;
    if (g.grad_out) g.grad_out[i] = v;
}

// Weight gradients dW = dZ^T . A_prev and bias gradients (the same product
// with a column of ones) over batch rows [z kSplitK, (z + 1) kSplitK) of
// workgroup z; T x T tiles per wave.  One workgroup per 32 T x 32 T block of
// W3 and W2, per 64 columns of W4 and per 64 rows of W1, and one for the
// loss.  With one split the gradient is final and Adam runs here, in the same
// launch; the weights it rewrites are read by the next step's launch only.
template <int T>
__global__ void __launch_bounds__(256) grads_kernel(GradArgs g)
{
    constexpr int kSide = kHidden / (32 * T), kBlocks = kSide * kSide;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
    int b = blockIdx.x;
    if (b == 2 * kBlocks + 8) {
        // mean squared error over the n x 8 outputs, partials in a fixed order
        if (blockIdx.y) return;
        __shared__ float red[256];
        float s = 0.f;
        for (int i = threadIdx.x; i < g.loss_parts; i += 256) s += g.loss_part[i];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const float v = red[0] / (float)((int64_t)g.n * kOut);
            g.loss[0] = v;
            if (g.loss_out) g.loss_out[0] = v;
        }
        return;
    }
    const int steps = g.n_pad / kStep;
    const int s0 = blockIdx.y * (kSplitK / kStep), s1 = min(steps, s0 + kSplitK / kStep);
    auto run = [&](auto mt_, auto nt_, int l, int m_tile, int n_tile, int64_t w_at, int64_t b_at, int rows, int cols) {
        constexpr int MT = decltype(mt_)::value, NT = decltype(nt_)::value;
        const uint16_t *A = g.dz_t[l] + (size_t)m_tile * steps * (kTile * kStep) + lane * 8;
        const uint16_t *B = g.in_t[l] + (size_t)n_tile * steps * (kTile * kStep) + lane * 8;
        // with one split, the parameters this lane will update, read while
        // the products run
        const bool update = g.update && g.splits == 1;
        auto row_at = [&](int i, int e) { return (m_tile + i) * kTile + 4 * grp + e; };
        Moments state[MT][NT][4], b_state[MT][4];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = row_at(i, e);
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int k = (n_tile + j) * kTile + col;
                    if (update && o < rows && k < cols) state[i][j][e] = moments_of(g.adam, w_at + (int64_t)o * cols + k);
                }
                if (update && o < rows && n_tile == 0 && col == 0) b_state[i][e] = moments_of(g.adam, b_at + o);
            }
        f32x4 acc[MT][NT], sum[MT];
        bf16x8 one;
#pragma unroll
        for (int i = 0; i < 8; ++i) one[i] = (__bf16)1.0f;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = sum[i];
        }
        // kAhead k-steps' fragments loaded before the first product; past the
        // end zeros, which add nothing
        constexpr int kAhead = 4;
        for (int s = s0; s < s1; s += kAhead) {
            bf16x8 x[kAhead][MT], y[kAhead][NT];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const bool in = s + u < s1;
#pragma unroll
                for (int i = 0; i < MT; ++i) x[u][i] = in ? load8(A + ((size_t)i * steps + s + u) * (kTile * kStep)) : bf16x8{};
#pragma unroll
                for (int j = 0; j < NT; ++j) y[u][j] = in ? load8(B + ((size_t)j * steps + s + u) * (kTile * kStep)) : bf16x8{};
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int i = 0; i < MT; ++i) {
#pragma unroll
                    for (int j = 0; j < NT; ++j) acc[i][j] = mfma(x[u][i], y[u][j], acc[i][j]);
                    if (n_tile == 0) sum[i] = mfma(x[u][i], one, sum[i]);
                }
        }
        auto out = [&](int64_t i, const Moments &before, float v) {
            if (g.splits > 1) {
                g.part[(int64_t)blockIdx.y * kParams + i] = v;
                return;
            }
            put_grad(g, i, v);
            if (update) adam_step(g.adam, i, before, v);
        };
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = row_at(i, e);
                if (o >= rows) continue;
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int k = (n_tile + j) * kTile + col;
                    if (k < cols) out(w_at + (int64_t)o * cols + k, state[i][j][e], acc[i][j][e]);
                }
                if (n_tile == 0 && col == 0) out(b_at + o, b_state[i][e], sum[i][e]);
            }
    };
    using I1 = std::integral_constant<int, 1>;
    using IT = std::integral_constant<int, T>;
    if (b < 2 * kBlocks) {
        const int l = b < kBlocks ? 2 : 1;
        b -= l == 2 ? 0 : kBlocks;
        const int m = (b / kSide * 2 + (wave & 1)) * T, n = (b % kSide * 2 + (wave >> 1)) * T;
        run(IT{}, IT{}, l, m, n, l == 2 ? kW3 : kW2, l == 2 ? kB3 : kB2, kHidden, kHidden);
    } else if (b < 2 * kBlocks + 4) {
        run(I1{}, I1{}, 3, 0, (b - 2 * kBlocks) * 4 + wave, kW4, kB4, kOut, kHidden);
    } else {
        run(I1{}, I1{}, 0, (b - 2 * kBlocks - 4) * 4 + wave, 0, kW1, kB1, kHidden, kIn);
    }
}

// The splits' partial gradients added in order, then the Adam step.
__global__ void __launch_bounds__(256) finish_grads_kernel(GradArgs g)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= kParams) return;
    float s = 0.f;
    for (int z = 0; z < g.splits; ++z) s += g.part[(int64_t)z * kParams + i];
    put_grad(g, i, s);
    if (g.update) adam_step(g.adam, i, moments_of(g.adam, i), s);
}

__global__ void __launch_bounds__(256) adam_kernel(AdamArgs a, const float *grad)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < kParams) adam_step(a, i, moments_of(a, i), grad[i]);
}

__global__ void __launch_bounds__(256) copies_kernel(Copies c, const float *params)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < kParams) put_copies(c, i, params[i]);
}

__device__ void block_sums(double &s1, double &s2, double *r1, double *r2)
{
    r1[threadIdx.x] = s1;
    r2[threadIdx.x] = s2;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) {
            r1[threadIdx.x] += r1[threadIdx.x + k];
            r2[threadIdx.x] += r2[threadIdx.x + k];
        }
        __syncthreads();
    }
    s1 = r1[0];
    s2 = r2[0];
    __syncthreads();
}

// Column means and population standard deviations (FP64 sums) of the inputs
// (6 columns) and the targets (8 columns), the targets of the columns set in
// log_mask first mapped to log(t + off) with off = G / 100, G the geometric
// mean of the column's positive values (off = 1 if it has none):
// norm = [mean_x, sd_x, mean_t, sd_t, off_t].  The offset follows the bulk
// of a column that spans decades, where its arithmetic mean follows the
// largest values.
// A column with zero spread gets sd = 1.
__global__ void __launch_bounds__(256) fit_norm_kernel(const float *x, const float *t, int n, int log_mask,
                                                       float *norm)
{
    __shared__ double r1[256], r2[256];
    const int col = blockIdx.x;  // 0..13
    const bool is_x = col < kIn;
    const float *src = is_x ? x : t;
    const int c = is_x ? col : col - kIn;
    const int w = is_x ? kIn : kOut;
    const bool logt = !is_x && ((log_mask >> c) & 1);
    float off = 0.f;
    if (logt) {
        double s1 = 0.0, s2 = 0.0;  // sum of log t and count over t > 0
        for (int i = threadIdx.x; i < n; i += 256) {
            const float v = src[(size_t)i * w + c];
            if (v > 0.f) {
                s1 += log((double)v);
                s2 += 1.0;
            }
        }
        block_sums(s1, s2, r1, r2);
        off = s2 > 0.0 ? (float)(exp(s1 / s2) / 100.0) : 1.f;
    }
    double s1 = 0.0, s2 = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) {
        const float raw = src[(size_t)i * w + c];
        const double v = (double)(logt ? to_target_space(raw, off) : raw);
        s1 += v;
        s2 += v * v;
    }
    block_sums(s1, s2, r1, r2);
    if (threadIdx.x == 0) {
        const double mean = s1 / n;
        const double var = fmax(s2 / n - mean * mean, 0.0);
        const double sd = var > 0.0 ? sqrt(var) : 1.0;
        const int base = is_x ? 0 : 2 * kIn;
        norm[base + c] = (float)mean;
        norm[base + w + c] = (float)sd;
        if (!is_x) norm[2 * kIn + 2 * kOut + c] = off;
    }
}

__global__ void fill_f32_kernel(float *p, float v, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

unsigned blocks(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

template <int RV, int MT, int WAVES, bool TRAIN>
hipError_t rows(const RowArgs &a, int *loss_parts, hipStream_t st)
{
    // whole padded rows in training (they enter the weight gradients as
    // zeros), the real ones in a forward pass
    const unsigned grid = blocks(TRAIN ? a.n_pad : a.n, RV * MT);
    rows_kernel<RV, MT, WAVES, TRAIN><<<grid, 64 * WAVES, 0, st>>>(a);
    if (loss_parts) *loss_parts = (int)grid * MT;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_rows(const RowArgs &a, bool train, int *loss_parts, hipStream_t st)
{
    // training: four rows per workgroup while that leaves at most one per CU
    // (21.4 against 28.5 us a step of 256 rows, 26.7 against 32.8 at 1,000, but
    // 42 against 39 at 2,048), else sixteen.  Forward: sixteen rows up to two
    // workgroups per CU, then 64, whose weights serve more rows (13.4 against
    // 20.7 us at 8,192, 25.1 against 20.8 at 16,384); below 4,096 rows the
    // host's side of the call (10.4 us) hides the difference.
    if (train) return a.n <= 4 * 256 ? rows<4, 1, 16, true>(a, loss_parts, st) : rows<16, 1, 16, true>(a, loss_parts, st);
    return a.n <= 16 * 512 ? rows<16, 1, 16, false>(a, nullptr, st) : rows<16, 4, 8, false>(a, nullptr, st);
}

hipError_t launch_grads(const GradArgs &a, hipStream_t st)
{
    // one split (up to 1,024 rows): 137 workgroups of 32 x 32 blocks; several
    // splits fill the chip with 64 x 64 ones, which read each operand half as often
    if (a.splits == 1) grads_kernel<1><<<2 * 64 + 9, 256, 0, st>>>(a);
    else grads_kernel<2><<<dim3(2 * 16 + 9, (unsigned)a.splits), 256, 0, st>>>(a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.splits == 1) return e;
    finish_grads_kernel<<<blocks(kParams, 256), 256, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_adam(const AdamArgs &a, const float *grad, hipStream_t st)
{
    adam_kernel<<<blocks(kParams, 256), 256, 0, st>>>(a, grad);
    return hipGetLastError();
}

hipError_t launch_copies(const Copies &c, const float *params, hipStream_t st)
{
    copies_kernel<<<blocks(kParams, 256), 256, 0, st>>>(c, params);
    return hipGetLastError();
}

hipError_t launch_fit_norm(const float *x, const float *t, int n, int log_mask, float *norm, hipStream_t st)
{
    fit_norm_kernel<<<kIn + kOut, 256, 0, st>>>(x, t, n, log_mask, norm);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, float v, int64_t n, hipStream_t st)
{
    if (n > 0) fill_f32_kernel<<<blocks(n, 256), 256, 0, st>>>(p, v, n);
    return hipGetLastError();
}

}  // namespace emu
}  // namespace cpm
