// Learned spectral preconditioner: recording, inference table and training.
//
// The fixed Fourier-acceleration multiplier m0(p) = (alpha/2) p2max / p^2(p)
// (divided by V for the unnormalised transforms) is replaced by
//     m(p) = m0(p) * exp(o_s(p) + o_a(0)),
// where (o_s, o_a) are the outputs of a 6 -> 64 -> 64 -> 2 tanh network on the
// features of each distinct momentum tuple n_mu in [0, N_mu/2] (p^2 is even
// in every n_mu): x = (p^2_mu/4 - 1/2 for mu = 0..3, log10(theta_k)/8 + 1,
// k/64). o_a at the zero tuple sets a global step; all-zero outputs give the
// fixed multiplier exactly. Parameters (float): W1 (64x6), b1, W2 (64x64), b2,
// W3 (2x64), b3.
//
// Training signal, recorded on plain-FA trajectories: per tuple,
// P_k = sum over the +-n reflections and the four packed fields of |Z(p)|^2
// after the forward FFT, C_k = the same sum of Re[Z_{k+1}(p) conj(Z_k(p))], and
// E_k = the energy after a probe update with every multiplier scaled by sigma.
// A sample pairs iterations k and k + 1: through P_k, E_k and P_{k+1} each mode
// has a quadratic a - 2 s b + s^2 c of the factor s on its multiplier, and the
// loss is ln(sum_p (a - 2 s b + s^2 c) / sum_p a) with s = exp(o_s(p) + o_a(0)).
#pragma once

#include "gf_device.hpp"

namespace gf {

constexpr int kMlpIn = 6, kMlpH = 64, kMlpOut = 2;
constexpr int kMlpParams = kMlpH * kMlpIn + kMlpH + kMlpH * kMlpH + kMlpH + kMlpOut * kMlpH + kMlpOut;
constexpr double kRatioFloor = 1e-12;  // the training loss is ln(max(predicted residual ratio, this))
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kMlpH * kMlpIn, kOffW2 = kOffB1 + kMlpH, kOffB2 = kOffW2 + kMlpH * kMlpH,
              kOffW3 = kOffB2 + kMlpH, kOffB3 = kOffW3 + kMlpOut * kMlpH;

// Folded tuple index (first axis fastest) of the mode n of a lattice.
__device__ __forceinline__ int fold1(int n, int N) { return n <= N / 2 ? n : N - n; }

struct TupleGeom {
    int n[4];   // lattice extents
    int h[4];   // N_mu/2 + 1
    int count;  // number of tuples
};

__device__ __forceinline__ int tuple_index(const TupleGeom& tg, int nx, int ny, int nz, int nt) {
    return fold1(nx, tg.n[0]) + tg.h[0] * (fold1(ny, tg.n[1]) + tg.h[1] * (fold1(nz, tg.n[2]) + tg.h[2] * fold1(nt, tg.n[3])));
}

// -------------------------------------------------------------- recording
// Per tuple, summed over the tuple's +-n reflections and the four packed
// fields (full 4D spectra, planes ps apart): out[3i] = P = |Sk|^2,
// out[3i+1] = C = Re Sk1 conj(Sk) (Sk1: after the plain step),
// out[3i+2] = E = |Sp|^2 (Sp: after the probe step). Double.
// Thread (a, i) of a block takes reflection a of 16 of the block's tuple i of 16 and sums the four fields;
// the 16 partial sums of a tuple are added in order. (One thread per tuple left 26 blocks of dependent
// loads at 16^4: 23.8 us a launch against 5.)
constexpr int kRecordTuples = 16;
template <typename T>
__global__ void __launch_bounds__(256) k_record_tuples(const cx<T>* __restrict__ Sk, const cx<T>* __restrict__ Sk1,
                                                       const cx<T>* __restrict__ Sp, size_t ps, TupleGeom tg,
                                                       double* __restrict__ out) {
    __shared__ double red[3][16][kRecordTuples];
    const int j = threadIdx.x % kRecordTuples, a = threadIdx.x / kRecordTuples;
    const int i = blockIdx.x * kRecordTuples + j;
    double P = 0.0, C = 0.0, E = 0.0;
    if (i < tg.count) {
        int r = i, st = 1, s = 0;
        bool dup = false;  // a flipped axis whose reflection is the mode itself: another a has it
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int t = r % tg.h[m];
            r /= tg.h[m];
            const bool flip = (a >> m) & 1;
            dup |= flip && (t == 0 || 2 * t == tg.n[m]);
            s += st * (flip && t > 0 ? tg.n[m] - t : t);
            st *= tg.n[m];
        }
        if (!dup) {
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                const size_t q = (size_t)f * ps + s;
                const cx<T> z0 = Sk[q], z1 = Sk1[q], zp = Sp[q];
                P += (double)z0.re * z0.re + (double)z0.im * z0.im;
                C += (double)z1.re * z0.re + (double)z1.im * z0.im;
                E += (double)zp.re * zp.re + (double)zp.im * zp.im;
            }
        }
    }
    red[0][a][j] = P;
    red[1][a][j] = C;
    red[2][a][j] = E;
    __syncthreads();
    if (threadIdx.x < 3 * kRecordTuples) {
        const int q = threadIdx.x / kRecordTuples, ii = blockIdx.x * kRecordTuples + threadIdx.x % kRecordTuples;
        if (ii < tg.count) {
            double v = 0.0;
#pragma unroll
            for (int k = 0; k < 16; ++k) v += red[q][k][threadIdx.x % kRecordTuples];
            out[3 * ii + q] = v;
        }
    }
}

// ------------------------------------------------------------ inference
__device__ __forceinline__ void mlp_features(const float* sin2_4, float log10_theta, float k, float x[kMlpIn]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) x[m] = sin2_4[m] * 0.25f - 0.5f;
    x[4] = log10_theta * 0.125f + 1.0f;
    x[5] = k * (1.0f / 64.0f);
}

// Multiplier table for the current iteration: mtab[i] = coef / p^2 *
// exp(o_s(i) + o_a(0)) (coef = (alpha/2) p2max / V), 0 at the zero tuple;
// theta and the iteration count come from the control block. The hidden
// layer 64 x 64 is a dense contraction over the tuples and runs on the matrix
// cores: a wave takes kTableGroups groups of 16 tuples; for each, every lane
// evaluates layer 1 for the 16 hidden units k = l/16 + 4m of tuple l%16 (its
// A operand), v_mfma_f32_16x16x4f32 forms the 16 x 64 pre-activations of
// layer 2 in four 16 x 16 tiles over K = 64 (16 steps, B operands read from
// the padded W2 in LDS), and layer 3 is a sum across the 16 lanes that hold
// one tuple's hidden units. o_a is evaluated once per block at the zero
// tuple, one hidden unit per lane of wave 0. (Keeping the B operands in
// registers for several groups measured slower: 256 VGPRs, one wave per SIMD.)
typedef float f32x4 __attribute__((ext_vector_type(4)));

// tanh(x) = 1 - 2 / (exp(2x) + 1) with the hardware exponential and
// reciprocal: absolute error about 1e-7, saturating correctly at both ends
// (inference only; the training kernels use tanhf).
__device__ __forceinline__ float tanh_fast(float x) {
    return 1.0f - 2.0f * __frcp_rn(__expf(2.0f * x) + 1.0f);
}
constexpr int kTableGroups = 1;
constexpr int kTableTuplesPerBlock = 4 * 16 * kTableGroups;

template <typename T>
__global__ void __launch_bounds__(256) k_mlp_table(const float* __restrict__ params, const T* __restrict__ sin2,
                                                   TupleGeom tg, double coef, const Ctl* __restrict__ ctl,
                                                   int force, T* __restrict__ mtab) {
    if (!force && ctl->done) return;
    constexpr int W2S = kMlpH + 1;  // padded row stride of W2 in LDS
    __shared__ float w1[kMlpH * kMlpIn], b1[kMlpH], w2[kMlpH * W2S], b2[kMlpH], w3[2 * kMlpH], h1z[kMlpH];
    __shared__ float c1[kMlpH];  // b1 + the theta and k terms of layer 1, shared by every tuple
    __shared__ float oa_s;
    {
        // every load first, then the LDS stores: one memory round trip for the whole network
        constexpr int N2 = kMlpH * kMlpH / 256, N1 = (kMlpH * kMlpIn + 255) / 256;
        float r2[N2], r1[N1], rb1 = 0.f, rb2 = 0.f, rw30 = 0.f, rw31 = 0.f;
#pragma unroll
        for (int q = 0; q < N2; ++q) r2[q] = params[kOffW2 + q * 256 + threadIdx.x];
#pragma unroll
        for (int q = 0; q < N1; ++q) {
            const int i = q * 256 + threadIdx.x;
            r1[q] = i < kMlpH * kMlpIn ? params[kOffW1 + i] : 0.f;
        }
        if (threadIdx.x < kMlpH) {
            rb1 = params[kOffB1 + threadIdx.x];
            rb2 = params[kOffB2 + threadIdx.x];
            rw30 = params[kOffW3 + threadIdx.x];
            rw31 = params[kOffW3 + kMlpH + threadIdx.x];
        }
#pragma unroll
        for (int q = 0; q < N2; ++q) {
            const int i = q * 256 + threadIdx.x;
            w2[(i / kMlpH) * W2S + i % kMlpH] = r2[q];
        }
#pragma unroll
        for (int q = 0; q < N1; ++q) {
            const int i = q * 256 + threadIdx.x;
            if (i < kMlpH * kMlpIn) w1[i] = r1[q];
        }
        if (threadIdx.x < kMlpH) {
            b1[threadIdx.x] = rb1;
            b2[threadIdx.x] = rb2;
            w3[threadIdx.x] = rw30;
            w3[kMlpH + threadIdx.x] = rw31;
        }
    }
    __syncthreads();
    const float lt = (float)log10(fmax(ctl->theta, 1e-300));
    const float kk = (float)ctl->iters;
    const float b30 = params[kOffB3], b31 = params[kOffB3 + 1];
    if (threadIdx.x < kMlpH) {  // o_a: layer 1 of the zero tuple
        const int j = threadIdx.x;
        float zx[kMlpIn];
        const float zs[4] = {0.f, 0.f, 0.f, 0.f};
        mlp_features(zs, lt, kk, zx);
        const float cj = fmaf(w1[j * kMlpIn + 5], zx[5], fmaf(w1[j * kMlpIn + 4], zx[4], b1[j]));
        c1[j] = cj;
        float a = cj;
#pragma unroll
        for (int i = 0; i < 4; ++i) a = fmaf(w1[j * kMlpIn + i], zx[i], a);
        h1z[j] = tanh_fast(a);
    }
    __syncthreads();
    if (threadIdx.x < kMlpH) {  // layers 2 and 3 of the zero tuple, second output
        const int j = threadIdx.x;
        float a0 = b2[j], a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll
        for (int i = 0; i < kMlpH; i += 4) {
            a0 = fmaf(w2[j * W2S + i], h1z[i], a0);
            a1 = fmaf(w2[j * W2S + i + 1], h1z[i + 1], a1);
            a2 = fmaf(w2[j * W2S + i + 2], h1z[i + 2], a2);
            a3 = fmaf(w2[j * W2S + i + 3], h1z[i + 3], a3);
        }
        float p = w3[kMlpH + j] * tanh_fast((a0 + a1) + (a2 + a3));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) p += __shfl_xor(p, o, 64);
        if (j == 0) oa_s = p + b31;
    }
    __syncthreads();
    const double oa = (double)oa_s;
    const int l = threadIdx.x & 63, kq = l >> 4, lc = l & 15;
    // B operands: W2[unit n*16 + lc][input 4m + kq]
    const T* sx = sin2;
    const T* sy = sx + tg.n[0];
    const T* sz = sy + tg.n[1];
    const T* st = sz + tg.n[2];
    for (int grp = 0; grp < kTableGroups; ++grp) {
        const int t0 = blockIdx.x * kTableTuplesPerBlock + ((threadIdx.x >> 6) * kTableGroups + grp) * 16;
        // layer 1 for tuple t0 + lc, hidden units kq + 4m
        int ti = t0 + lc;
        if (ti >= tg.count) ti = 0;
        int c4[4], r = ti;
        for (int m = 0; m < 4; ++m) {
            c4[m] = r % tg.h[m];
            r /= tg.h[m];
        }
        const float s4[4] = {(float)sx[c4[0]], (float)sy[c4[1]], (float)sz[c4[2]], (float)st[c4[3]]};
        float x[kMlpIn];
        mlp_features(s4, lt, kk, x);
        float h1[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int j = kq + 4 * m;
            float a = c1[j];
#pragma unroll
            for (int i = 0; i < 4; ++i) a = fmaf(w1[j * kMlpIn + i], x[i], a);
            h1[m] = tanh_fast(a);
        }
        // layer 2: acc[n] holds rows 4*kq + q (tuples t0 + 4*kq + q), unit n*16 + lc
        f32x4 acc[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int m = 0; m < 16; ++m) acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(h1[m], w2[(n * 16 + lc) * W2S + 4 * m + kq], acc[n], 0, 0, 0);
        }
        // layer 3, first output: partial sums over this lane's units, then over the 16 lanes of the group
        float o0[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int j = n * 16 + lc;
#pragma unroll
            for (int q = 0; q < 4; ++q) o0[q] = fmaf(w3[j], tanh_fast(acc[n][q] + b2[j]), o0[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) o0[q] += __shfl_xor(o0[q], o, 64);
        if (lc < 4) {
            const int t = t0 + 4 * kq + lc;
            const float os = lc == 0 ? o0[0] : lc == 1 ? o0[1] : lc == 2 ? o0[2] : o0[3];
            if (t < tg.count) {
                int r2 = t, d4[4];
                for (int m = 0; m < 4; ++m) {
                    d4[m] = r2 % tg.h[m];
                    r2 /= tg.h[m];
                }
                const double p2 = (double)sx[d4[0]] + (double)sy[d4[1]] + (double)sz[d4[2]] + (double)st[d4[3]];
                mtab[t] = p2 > 0.0 ? (T)(coef / p2 * exp((double)(os + b30) + oa)) : T(0);
            }
        }
    }
}

// --------------------------------------------------------------- training
// Samples from records: record r holds (P_r, C_r, E_r) per tuple, E_r the
// energy after the probe step (every multiplier times sigma). Sample s uses
// record r = first + s*every and the next one: row s*T + i gets the features
// of tuple i at (theta[r], iteration k0 + r) and the coefficients (a, b, c)
// of the quadratic e(x) = a - 2 b x + c x^2 through the residual energies
// e(0) = P_r, e(sigma) = E_r and e(1) = P_{r+1}, with c raised to b^2/a where
// needed so that e stays >= 0; formed in double.
__global__ void __launch_bounds__(256) k_make_samples(const double* __restrict__ rec, const double* __restrict__ theta,
                                                      int first, int every, long long k0, double sigma,
                                                      int64_t nrows, TupleGeom tg, float* __restrict__ X,
                                                      float* __restrict__ tgt) {
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= nrows) return;
    const int s = (int)(row / tg.count), i = (int)(row % tg.count);
    const int64_t r = (int64_t)first + (int64_t)s * every;
    int t[4], q = i;
    for (int m = 0; m < 4; ++m) {
        t[m] = q % tg.h[m];
        q /= tg.h[m];
    }
    float s4[4];
    for (int m = 0; m < 4; ++m) {
        const double sv = sinpi((double)t[m] / (double)tg.n[m]);
        s4[m] = (float)(4.0 * sv * sv);
    }
    float x[kMlpIn];
    mlp_features(s4, (float)log10(fmax(theta[r], 1e-300)), (float)(k0 + r), x);
#pragma unroll
    for (int c = 0; c < kMlpIn; ++c) X[row * kMlpIn + c] = x[c];
    const double P = rec[(r * tg.count + i) * 3], E = rec[(r * tg.count + i) * 3 + 2];
    const double Pn = rec[((r + 1) * tg.count + i) * 3];
    const double v = (E - P - sigma * (Pn - P)) / (sigma * sigma - sigma);
    const double b = -0.5 * (Pn - P - v);
    const double c = P > 0.0 ? fmax(v, b * b / P) : v;
    tgt[row * 3] = (float)P;
    tgt[row * 3 + 1] = (float)b;
    tgt[row * 3 + 2] = (float)c;
}

// Rows are momentum tuples of samples; sample s owns rows [off[s], off[s+1]),
// its first row being the zero tuple. tgt row = (a, b, c).

// Both passes run on the matrix cores (v_mfma_f32_16x16x4f32: float products and sums), a wave taking 16 rows
// at a time, everything transposed so that no operand has to change lanes between the layers: lane l holds
// row l % 16 of the group and, of 64 hidden units, the 16 units 16 t + 4 (l / 16) + q (t, q < 4). That is
// what an instruction leaves of [units x rows] (unit tile t), and what the next one takes as its right
// operand if its K index runs over the units in the order (t, q; l / 16), which the left operand then
// follows. Layer 1 takes K = 8: the six features, 1 (times b1) and 0.
constexpr int kMlpRows = 16;            // rows of a wave's group
constexpr int kMlpStride = kMlpH + 4;   // LDS row stride: 16-byte aligned rows, consecutive rows 4 banks apart

// W2 (row j, column i), and its transpose if w2t is set, to LDS; b2 and W3 (3 x 64) to vec. Block of 256.
__device__ __forceinline__ void mlp_stage(const float* __restrict__ params, float* w2, float* w2t, float* vec) {
    constexpr int N = kMlpH * kMlpH / 256;
    float v[N], r = 0.f;  // every load before the first store: one round trip
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = params[kOffW2 + k * 256 + threadIdx.x];
    if (threadIdx.x < 3 * kMlpH)
        r = threadIdx.x < kMlpH ? params[kOffB2 + threadIdx.x] : params[kOffW3 + threadIdx.x - kMlpH];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int e = k * 256 + threadIdx.x, j = e / kMlpH, i = e % kMlpH;
        w2[j * kMlpStride + i] = v[k];
        if (w2t) w2t[i * kMlpStride + j] = v[k];
    }
    if (threadIdx.x < 3 * kMlpH) vec[threadIdx.x] = r;
}

// Left operands of layer 1, [unit 16 t + lc][K = 4 s + kq]: W1, then b1, then 0.
__device__ __forceinline__ void mlp_layer1_weights(const float* __restrict__ params, int lc, int kq, float a1[4][2]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int u = 16 * t + lc;
        a1[t][0] = params[kOffW1 + u * kMlpIn + kq];
        a1[t][1] = kq < 2 ? params[kOffW1 + u * kMlpIn + 4 + kq] : kq == 2 ? params[kOffB1 + u] : 0.f;
    }
}

// This lane's right operands of layer 1: features 4 s + kq of row `row`. Past the last row those of the last one, whose
// activations then are values of the input itself: zeros there would meet an infinite weight as NaN (with saturated
// units the gradient of the other rows is finite), and a NaN passes the zero output gradients of these lanes.
__device__ __forceinline__ void mlp_row_features(const float* __restrict__ X, int64_t row, int64_t n, int kq, float x[2]) {
    const float* r = X + (row < n ? row : n - 1) * kMlpIn;
    x[0] = r[kq];
    x[1] = kq < 2 ? r[4 + kq] : kq == 2 ? 1.f : 0.f;
}

__device__ __forceinline__ f32x4 tanh4(f32x4 z) { return f32x4{tanhf(z[0]), tanhf(z[1]), tanhf(z[2]), tanhf(z[3])}; }
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// acc[u] += sum over t, q of W[16 u + lc][16 t + 4 kq + q] v[t][q] (w at this lane's first entry): 64 matrix
// instructions. The left operands of the next t are read from LDS while those of this one are used.
__device__ __forceinline__ void mlp_contract(const float* w, const f32x4 v[4], f32x4 acc[4]) {
    f32x4 a[4], next[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = *reinterpret_cast<const f32x4*>(w + 16 * u * kMlpStride);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (t < 3) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                next[u] = *reinterpret_cast<const f32x4*>(w + 16 * u * kMlpStride + 16 * (t + 1));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] = mfma4(a[u][q], v[t][q], acc[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = next[u];
    }
}

// Hidden activations of the group's rows.
__device__ __forceinline__ void mlp_hidden(const float a1[4][2], const float x[2], const float* w2, const float* vec,
                                           int lc, int kq, f32x4 h1[4], f32x4 h2[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const f32x4 z = mfma4(a1[t][1], x[1], mfma4(a1[t][0], x[0], f32x4{0.f, 0.f, 0.f, 0.f}));
        h1[t] = tanh4(z);
    }
    f32x4 acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] = *reinterpret_cast<const f32x4*>(vec + 16 * u + 4 * kq);
    mlp_contract(w2 + lc * kMlpStride + 4 * kq, h1, acc);
#pragma unroll
    for (int u = 0; u < 4; ++u) h2[u] = tanh4(acc[u]);
}

// Forward pass: O (n x 2). The activations are not kept: the backward pass forms them again, which costs it
// less than writing and reading 512 bytes a row. 72 matrix instructions of 32 cycles per group: 12 us at 210k
// rows if the matrix cores never waited; measured 29 (60 with one row per thread and stored activations).
constexpr int kFwdMaxBlocks = 1024;  // four blocks per CU
__global__ void __launch_bounds__(256, 4) k_mlp_forward(const float* __restrict__ params, const float* __restrict__ X,
                                                     int64_t n, float* __restrict__ O) {
    __shared__ __align__(16) float w2[kMlpH * kMlpStride], vec[3 * kMlpH];
    const int l = threadIdx.x & 63, lc = l & 15, kq = l >> 4;
    mlp_stage(params, w2, nullptr, vec);
    float a1[4][2];
    mlp_layer1_weights(params, lc, kq, a1);
    const float b30 = params[kOffB3], b31 = params[kOffB3 + 1];
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * 4 * kMlpRows;
    int64_t row = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kMlpRows + lc;
    float xn[2];
    mlp_row_features(X, row, n, kq, xn);
#pragma unroll 1
    for (; row - lc < n; row += step) {
        const float x[2] = {xn[0], xn[1]};
        mlp_row_features(X, row + step, n, kq, xn);  // the next group's, on their way meanwhile
        f32x4 h1[4], h2[4];
        mlp_hidden(a1, x, w2, vec, lc, kq, h1, h2);
        float o0 = 0.f, o1 = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const f32x4 p = *reinterpret_cast<const f32x4*>(vec + kMlpH + 16 * u + 4 * kq);
            const f32x4 q = *reinterpret_cast<const f32x4*>(vec + 2 * kMlpH + 16 * u + 4 * kq);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                o0 = fmaf(p[k], h2[u][k], o0);
                o1 = fmaf(q[k], h2[u][k], o1);
            }
        }
        o0 += __shfl_xor(o0, 16, 64);
        o1 += __shfl_xor(o1, 16, 64);
        o0 += __shfl_xor(o0, 32, 64);
        o1 += __shfl_xor(o1, 32, 64);
        if (kq < 2 && row < n) O[row * 2 + kq] = kq == 0 ? o0 + b30 : o1 + b31;
    }
}

// One block per sample: loss (double) and dL/dO for the sample's rows, the
// mean over ns samples. dO is written for every row (o_a only at row 0).
constexpr int kLossThreads = 1024;  // a batch has few samples (blocks) of thousands of rows: 19 -> 11 us at 32 x 6561
__global__ void __launch_bounds__(kLossThreads) k_mlp_loss(const float* __restrict__ O, const float* __restrict__ tgt,
                                                  const int* __restrict__ off, int ns, float* __restrict__ dO,
                                                  double* __restrict__ sample_loss) {
    const int smp = blockIdx.x;
    const int r0 = off[smp], r1 = off[smp + 1];
    const double oa = O[(int64_t)r0 * 2 + 1];
    __shared__ double red[3][kLossThreads / 64];
    double asum = 0.0, lsum = 0.0;
    for (int r = r0 + threadIdx.x; r < r1; r += kLossThreads) {
        const double a = tgt[(int64_t)r * 3], b = tgt[(int64_t)r * 3 + 1], c = tgt[(int64_t)r * 3 + 2];
        const double s = exp((double)O[(int64_t)r * 2] + oa);
        asum += a;
        lsum += a - 2.0 * s * b + s * s * c;
    }
    asum = wave_sum(asum);
    lsum = wave_sum(lsum);
    const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) {
        red[0][wv] = asum;
        red[1][wv] = lsum;
    }
    __syncthreads();
    double Atot = 0.0, Ltot = 0.0;
    for (int i = 0; i < kLossThreads / 64; ++i) {
        Atot += red[0][i];
        Ltot += red[1][i];
    }
    // loss = ln(Ltot / Atot), floored at ln(kRatioFloor) with zero gradient there;
    // d loss/ds = (2 s c - 2 b) / (Ltot ns); do_s = d loss/ds * s; do_a(row 0) = sum over rows
    const bool floored = !(Ltot / Atot > kRatioFloor);
    double gsum = 0.0;
    for (int r = r0 + threadIdx.x; r < r1; r += kLossThreads) {
        const double b = tgt[(int64_t)r * 3 + 1], c = tgt[(int64_t)r * 3 + 2];
        const double s = exp((double)O[(int64_t)r * 2] + oa);
        const double g = floored ? 0.0 : (2.0 * s * c - 2.0 * b) / (Ltot * ns) * s;
        dO[(int64_t)r * 2] = (float)g;
        dO[(int64_t)r * 2 + 1] = 0.0f;
        gsum += g;
    }
    gsum = wave_sum(gsum);
    __syncthreads();
    if (l == 0) red[2][wv] = gsum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < kLossThreads / 64; ++i) t += red[2][i];
        dO[(int64_t)r0 * 2 + 1] = (float)t;
        sample_loss[smp] = log(floored ? kRatioFloor : Ltot / Atot);
    }
}

// Backward pass. A wave takes 16 rows at a time: the hidden activations again as in the
// forward pass, dz2 = (dO W3) (1 - h2^2), dz1 = (dz2 W2) (1 - h1^2) in the same lanes, and then the sums over
// rows. dW2 = sum_r dz2[r] h1[r]^T and [dW1 | db1] = sum_r dz1[r] [x[r] | 1]^T have the rows as their K index:
// the wave turns dz2, h1 and dz1 through LDS (16 x 64 each, one after another in one buffer of its own) and
// adds to accumulators in registers; db2, dW3 and db3 are added per lane. The waves' sums are added in LDS in
// wave order and the block's partial gradient (float) goes to gpart[b]; k_grad_reduce adds the partials in
// order, in double. 216 matrix instructions of 32 cycles per group: 37 us at 210k rows if the matrix
// cores never waited; measured 95 (245 with dot products on the vector units and stored activations).
//
// Two blocks per CU, the groups dealt out evenly, and one launch for every kBwdRows rows (512 additions in one
// accumulator): the rounding of the float partials stays what it is at that size, and the double sum does the rest.
// (2^24 equal rows: the gradient is off by 7.6e-6; with all rows in one launch 1.2e-4. The training step
// at 1.37M rows takes 623 us, 587 with one launch, 750 with as many blocks of 512 rows as that takes, 733 with the
// partials of one launch in a loop, which spills.)
constexpr int kBwdMaxBlocks = 512;
constexpr int64_t kBwdRows = (int64_t)kBwdMaxBlocks * 4 * 512;
__host__ __device__ constexpr int mlp_bwd_blocks(int64_t n) {
    const int64_t b = (n + 4 * kMlpRows - 1) / (4 * kMlpRows);
    return (int)(b < kBwdMaxBlocks ? b : kBwdMaxBlocks);
}
// Launches of the backward pass and rows of each (the last takes what is left).
__host__ __device__ constexpr int mlp_bwd_launches(int64_t n) { return (int)((n + kBwdRows - 1) / kBwdRows); }
__host__ __device__ constexpr int64_t mlp_bwd_rows(int64_t n) {
    const int64_t l = mlp_bwd_launches(n);
    return (n + l * kMlpRows - 1) / (l * kMlpRows) * kMlpRows;
}
__host__ __device__ constexpr int mlp_bwd_parts(int64_t n) {
    const int64_t r = mlp_bwd_rows(n), l = (n + r - 1) / r;
    return (int)(l - 1) * mlp_bwd_blocks(r) + mlp_bwd_blocks(n - (l - 1) * r);
}

__global__ void __launch_bounds__(256, 2) k_mlp_backward(const float* __restrict__ params, const float* __restrict__ X,
                                                         const float* __restrict__ dO, int64_t n,
                                                         float* __restrict__ gpart) {
    constexpr int W = kMlpH * kMlpStride;
    __shared__ __align__(16) float lds[2 * W + 3 * kMlpH + 4 * kMlpRows * kMlpStride];
    float *w2 = lds, *w2t = lds + W, *vec = lds + 2 * W;
    const int l = threadIdx.x & 63, lc = l & 15, kq = l >> 4, wv = threadIdx.x >> 6;
    float* turn = vec + 3 * kMlpH + wv * kMlpRows * kMlpStride;
    mlp_stage(params, w2, w2t, vec);
    float a1[4][2];
    mlp_layer1_weights(params, lc, kq, a1);
    __syncthreads();
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 gw2[4][4], gw1[4], gb2[4], gw30[4], gw31[4];
    float gb30 = 0.f, gb31 = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        gw1[t] = gb2[t] = gw30[t] = gw31[t] = zero;
#pragma unroll
        for (int u = 0; u < 4; ++u) gw2[t][u] = zero;
    }
    // [row lc][units 16 t + 4 kq + q] -> [row 4 s + kq][unit 16 t + lc]; the wave's LDS accesses keep their order
    auto turned = [&](const f32x4 v[4], float r[4][4]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) *reinterpret_cast<f32x4*>(turn + lc * kMlpStride + 16 * t + 4 * kq) = v[t];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int s = 0; s < 4; ++s) r[t][s] = turn[(4 * s + kq) * kMlpStride + 16 * t + lc];
        __builtin_amdgcn_wave_barrier();
    };
    struct Inputs {
        float x[2], d0, d1;
    };
    auto load = [&](int64_t row0) {
        Inputs in;
        const int64_t row = row0 + lc;
        mlp_row_features(X, row, n, kq, in.x);
        in.d0 = row < n ? dO[row * 2] : 0.f;
        in.d1 = row < n ? dO[row * 2 + 1] : 0.f;
        return in;
    };
    const int64_t step = (int64_t)gridDim.x * 4 * kMlpRows;
    int64_t row0 = ((int64_t)blockIdx.x * 4 + wv) * kMlpRows;
    Inputs next = load(row0);
#pragma unroll 1
    for (; row0 < n; row0 += step) {
        const Inputs in = next;
        next = load(row0 + step);  // the next group's, on their way meanwhile
        const float d0 = in.d0, d1 = in.d1;
        float xb[4];  // [row 4 s + kq][column lc of (x | 1 | 0)], for the end of the group
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int64_t r = row0 + 4 * s + kq;
            xb[s] = r >= n ? 0.f : lc < kMlpIn ? X[r * kMlpIn + lc] : lc == kMlpIn ? 1.f : 0.f;
        }
        f32x4 h1[4], h2[4], dz2[4], dz1[4];
        mlp_hidden(a1, in.x, w2, vec, lc, kq, h1, h2);
        gb30 += d0;
        gb31 += d1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const f32x4 p = *reinterpret_cast<const f32x4*>(vec + kMlpH + 16 * u + 4 * kq);
            const f32x4 q = *reinterpret_cast<const f32x4*>(vec + 2 * kMlpH + 16 * u + 4 * kq);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float h = h2[u][k];
                const float dz = (d0 * p[k] + d1 * q[k]) * (1.f - h * h);
                dz2[u][k] = dz;
                gb2[u][k] += dz;
                gw30[u][k] = fmaf(d0, h, gw30[u][k]);
                gw31[u][k] = fmaf(d1, h, gw31[u][k]);
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) dz1[t] = zero;
        mlp_contract(w2t + lc * kMlpStride + 4 * kq, dz2, dz1);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) dz1[t][q] *= 1.f - h1[t][q] * h1[t][q];
        float ra[4][4], rb[4][4];
        turned(dz2, ra);
        turned(h1, rb);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < 4; ++t) gw2[u][t] = mfma4(ra[u][s], rb[t][s], gw2[u][t]);
        turned(dz1, ra);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t) gw1[t] = mfma4(ra[t][s], xb[s], gw1[t]);
    }
    // sums over the 16 rows' lanes of what was added per lane
    auto rows_sum = [](float v) {
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);
        return v;
    };
    gb30 = rows_sum(gb30);
    gb31 = rows_sum(gb31);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            gb2[u][q] = rows_sum(gb2[u][q]);
            gw30[u][q] = rows_sum(gw30[u][q]);
            gw31[u][q] = rows_sum(gw31[u][q]);
        }
    __syncthreads();  // W2 is no longer needed: its place takes the block's gradient
    float* gs = lds;
    static_assert(kMlpParams <= 2 * W, "the block's gradient fits where W2 was");
    for (int w = 0; w < 4; ++w) {
        if (wv == w) {
            auto put = [&](int at, float v) { gs[at] = w == 0 ? v : gs[at] + v; };
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int j = 16 * u + 4 * kq + q;  // row of the accumulators, column lc
#pragma unroll
                    for (int t = 0; t < 4; ++t) put(kOffW2 + j * kMlpH + 16 * t + lc, gw2[u][t][q]);
                    if (lc < kMlpIn) put(kOffW1 + j * kMlpIn + lc, gw1[u][q]);
                    if (lc == kMlpIn) put(kOffB1 + j, gw1[u][q]);
                    if (lc == 0) {
                        put(kOffB2 + j, gb2[u][q]);
                        put(kOffW3 + j, gw30[u][q]);
                        put(kOffW3 + kMlpH + j, gw31[u][q]);
                    }
                }
            if (l == 0) {
                put(kOffB3, gb30);
                put(kOffB3 + 1, gb31);
            }
        }
        __syncthreads();
    }
    float* gp = gpart + (size_t)blockIdx.x * kMlpParams;
    for (int i = threadIdx.x; i < kMlpParams; i += 256) gp[i] = gs[i];
}

// Adam (Kingma and Ba 2015) of one parameter.
struct AdamStep {
    float *params, *m, *v;  // m null: no step
    float lr, b1, b2, eps, c1, c2;
    __device__ __forceinline__ void operator()(int p, float g) const {
        const float mm = b1 * m[p] + (1.f - b1) * g;
        const float vv = b2 * v[p] + (1.f - b2) * g * g;
        m[p] = mm;
        v[p] = vv;
        params[p] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    }
};

// Sum of the partial gradients in double, kGradSlices runs of consecutive partials each in order
// and then the runs in order, and the optimiser's step if one is asked for. (One thread per parameter
// waited on 410 dependent loads: 24 -> 6 us at 210k rows.)
constexpr int kGradParams = 64, kGradSlices = 16;
__global__ void __launch_bounds__(kGradParams * kGradSlices) k_grad_reduce(const float* __restrict__ gpart, int nb,
                                                                          float* __restrict__ grad, AdamStep step) {
    __shared__ double part[kGradSlices][kGradParams];
    const int c = threadIdx.x % kGradParams, sl = threadIdx.x / kGradParams, p = blockIdx.x * kGradParams + c;
    const int run = (nb + kGradSlices - 1) / kGradSlices, b1 = min(nb, (sl + 1) * run);
    double a = 0.0;
    if (p < kMlpParams) {
#pragma unroll 8
        for (int b = sl * run; b < b1; ++b) a += gpart[(size_t)b * kMlpParams + p];
    }
    part[sl][c] = a;
    __syncthreads();
    if (sl == 0 && p < kMlpParams) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kGradSlices; ++k) t += part[k][c];
        grad[p] = (float)t;
        if (step.m) step(p, (float)t);
    }
}

// The optimiser's step from a gradient, counted from 1.
__global__ void __launch_bounds__(256) k_adam(const float* __restrict__ grad, AdamStep step) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < kMlpParams) step(p, grad[p]);
}

}  // namespace gf
