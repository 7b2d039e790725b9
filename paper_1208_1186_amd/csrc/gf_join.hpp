// Measurement of the current links and forward (x, y) transform of their divergence in one kernel, for the
// plane shapes where it is the faster form (GF_JOIN_CASES): a block forms the divergence of one (z, t) plane
// in LDS, transforms it there and writes the transform. The divergence never goes to memory (128 of the 1248
// bytes per site and iteration in FP64-18) and the iteration has three launches instead of four.
//
// Two lanes per site, l and l + 32: lane half q forms U_mu(x) for mu = q (in the plane: x, y) and mu = 2 + q
// (out of it: z, t). A wave's 32 sites are whole or part x rows of up to 32 consecutive pairs p (x = p % NX,
// strip p / NX) and step through the NY / S rows of their strip, so that in the plane every link is formed
// once: the back link along y is the one of the previous row, kept in registers (the strip's first is formed
// again), the back link along x comes from the neighbouring lane, or is formed again where that lane is in
// another wave. H(x) is the y neighbour's of the previous row and the x neighbour's comes from its lane.
// Links from below in z and t are formed from memory. There is no barrier until the plane is complete.
//
// Bound in double by the L1s' misses and by the fabric's reads: a site takes 1.39 KB through the L1s against 2.0 KB
// for k_update_measure, which re-reads every back link's U0 and H, and either holds 92 to 97 lines in flight per CU
// (32^4 and 48^3 x 8, at 1.7 and 3.4 waves per SIMD; 7.7 and 10.5 TB/s). In float the vector units are nearer: 0.67 of
// the issue slots here (32^3 x 64), 0.94 there (48^3 x 8). Measured with the (x, y) pass counted
// (us): 32^4 FP64-18 184 against 192 + 27, FP64-12 148 against 178 + 27, 32^3 x 64 FP32-12 154 against
// 183 + 28, 16^4 FP64-18 14.5 against 12.5 + 4, 8^4 5.5 against 4.6 + 2.8. On 48 x 48 planes (LDS for one
// block per CU, 384 blocks at 48^3 x 8) and 24 x 24 planes it is the slower form (217 against 191, 26 against
// 24.5). The same with barriers between strips and sums in LDS: 184 and 160; with four lanes per site: 203.
#pragma once

#include "gf_fft_ct.hpp"

namespace gf {

// Value of another lane of the wave (byte address 4 * lane).
__device__ __forceinline__ float lane_get(float v, int addr) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}
__device__ __forceinline__ double lane_get(double v, int addr) {
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(addr, __double2hiint(v)),
                            __builtin_amdgcn_ds_bpermute(addr, __double2loint(v)));
}
template <typename T>
__device__ __forceinline__ cx<T> lane_get(cx<T> v, int addr) {
    return {lane_get(v.re, addr), lane_get(v.im, addr)};
}

// Sum over lanes l and l ^ 32 (both receive it).
__device__ __forceinline__ float half_sum(float v) {
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ double half_sum(double v) {
    const unsigned lo = __double2loint(v), hi = __double2hiint(v);
    auto bl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    auto bh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double(bh[0], bl[0]) + __hiloint2double(bh[1], bl[1]);
}

// Per-lane choice between two complex numbers, copied to scalars first: a choice between entries of arrays
// becomes a load at a per-lane index, which puts the arrays in scratch memory.
template <typename T>
__device__ __forceinline__ cx<T> choose(bool c, cx<T> a, cx<T> b) {
    const T ar = a.re, ai = a.im, br = b.re, bi = b.im;
    return {c ? ar : br, c ? ai : bi};
}

// Twice the anti-Hermitian part of X as nine reals: X01 - conj X10, X02 - conj X20, X12 - conj X21 and the
// imaginary parts of the diagonal. The trace leaves the sum of the links, once (taken off each link, its rounding
// raised the float descent's floor of theta by 2.5 %).
template <typename T>
struct PackedAh {
    cx<T> z[3];
    T d[3];
    __device__ __forceinline__ explicit PackedAh(const su3<T>& x) {
        z[0] = x.e[0][1] - conj(x.e[1][0]);
        z[1] = x.e[0][2] - conj(x.e[2][0]);
        z[2] = x.e[1][2] - conj(x.e[2][1]);
#pragma unroll
        for (int i = 0; i < 3; ++i) d[i] = x.e[i][i].im;
    }
    __device__ __forceinline__ void add(const PackedAh& b) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            z[i] = z[i] + b.z[i];
            d[i] += b.d[i];
        }
    }
    __device__ __forceinline__ void sub(const PackedAh& b) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            z[i] = z[i] - b.z[i];
            d[i] -= b.d[i];
        }
    }
};

// Rows 1-2 of H at site s; U0 at site s from byte offset om within the tile (direction mu). Sites below the
// bound that keeps the links' array under 4 GiB.
template <typename T>
__device__ __forceinline__ void load_rows(const cx<T>* H, uint32_t s, su3<T>& h) {
    const uint32_t o = tile_byte_offset<cx<T>>(6, s);
#pragma unroll
    for (int k = 0; k < 6; ++k) h.e[k / 3][k % 3] = ld_off(H + k * kTileSites, o);
}
template <typename T, int NE>
__device__ __forceinline__ void load_link(const Links<T, NE>& U0, uint32_t s, uint32_t om, su3<T>& u) {
    const uint32_t o = tile_byte_offset<cx<T>>(4 * NE, s) + om;
#pragma unroll
    for (int k = 0; k < NE; ++k) u.e[k / 3][k % 3] = ld_off(U0.p + k * kTileSites, o);
    if constexpr (NE == 6) third_row(u.e[0], u.e[1], u.e[2]);
}

// The plane that block b (of one XCD's consecutive run) takes. zb >= 1: z in groups of zb inside the t loop;
// 0: t fastest; -1: bricks of up to 4 z by 8 t planes, z fastest. All orders give the same bits.
__device__ __forceinline__ int plane_order(int b, int nz, int nt, int zb) {
    if (zb == 0) return b / nt + nz * (b % nt);
    if (zb > 0) return b % zb + zb * (b / (zb * nt)) + nz * ((b / zb) % nt);
    const int bz = nz % 4 == 0 ? 4 : 2, bt = nt % 8 == 0 ? 8 : nt % 4 == 0 ? 4 : 2;  // extents are even
    const int in = b % (bz * bt), brick = b / (bz * bt), nbz = nz / bz;
    return brick % nbz * bz + in % bz + nz * (brick / nbz * bt + in / bz);
}

// The last y stage of the four fields' transforms writes element e (its y) of column b % NX of field b / NX
// to memory, runs of NX consecutive sites.
template <typename T, int NX>
struct PlaneOut {
    cx<T>* q;
    size_t zps;
    static constexpr bool lds_in = false, lds_out = false;
    __device__ __forceinline__ void st(int b, int e, cx<T> v) const { q[(size_t)(b / NX) * zps + e * NX + b % NX] = v; }
};

constexpr int join_threads(int nx, int s) { return (2 * nx * s + 63) / 64 * 64; }
constexpr size_t join_lds(int nx, int ny, size_t csz) { return (size_t)(nx + ny + 4 * ny * (nx + 1)) * csz; }

// One partial (F, theta) per plane. force: measure even when the loop has stopped.
template <typename T, int NE, int NX, int NY, int S>
__global__ void __launch_bounds__(join_threads(NX, S), 2)
    k_measure_xy(Links<T, NE> U0, const cx<T>* __restrict__ H, cx<T>* __restrict__ Q, size_t zps, int nz, int nt,
                 const cx<T>* __restrict__ twgx, const cx<T>* __restrict__ twgy, double2* __restrict__ part, Ctl* ctl,
                 Batch bt, int zb, int force) {
    constexpr int RS = NX + 1, P = NX * NY, PL = NY * RS, NT = join_threads(NX, S), ROWS = NY / S;
    constexpr bool XWAVE = 32 % NX == 0;  // x neighbours are always in the half wave
    constexpr uint32_t E = sizeof(cx<T>);
    static_assert(NY % S == 0, "whole strips");
    {
        const size_t bo = boff(bt);
        U0.p = bshift(U0.p, bo);
        H = bshift(H, bo);
        Q = bshift(Q, bo);
        twgx = bshift(twgx, bo);
        twgy = bshift(twgy, bo);
        part = bshift(part, bo);
        ctl = bshift(ctl, bo);
    }
    if (!force && ctl->done) return;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double sa[NT / 64], sb[NT / 64];
    cx<T>* twx = reinterpret_cast<cx<T>*>(smem);
    cx<T>* twy = twx + NX;
    cx<T>* buf = twy + NY;
    for (int i = threadIdx.x; i < NX; i += NT) twx[i] = twgx[i];
    for (int i = threadIdx.x; i < NY; i += NT) twy[i] = twgy[i];
    const int plane = plane_order(xcd_remap(blockIdx.x, gridDim.x), nz, nt, zb);
    const int z = plane % nz, t = plane / nz;
    const int lane = threadIdx.x & 63, q = lane >> 5;
    const int p = (threadIdx.x >> 6) * 32 + (lane & 31);
    const uint32_t base = (uint32_t)plane * P;
    double fsum = 0.0, tsum = 0.0;
    if ((NX * S) % 32 == 0 || p < NX * S) {
        const int x = p % NX, y0 = p / NX * ROWS;
        // site offsets to the neighbours out of the plane
        const uint32_t pz = P, pt = (uint32_t)P * (uint32_t)nz;
        const uint32_t fz = z == nz - 1 ? 0u - (uint32_t)(nz - 1) * pz : pz;
        const uint32_t ft = t == nt - 1 ? 0u - (uint32_t)(nt - 1) * pt : pt;
        const uint32_t bz = z == 0 ? (uint32_t)(nz - 1) * pz : 0u - pz;
        const uint32_t bk = t == 0 ? (uint32_t)(nt - 1) * pt : 0u - pt;
        const uint32_t dfw = q == 0 ? fz : ft, dbk = q == 0 ? bz : bk;
        // lanes of the x neighbours, if they are in this half wave
        const int lf = x == NX - 1 ? lane - (NX - 1) : lane + 1, lb = x == 0 ? lane + NX - 1 : lane - 1;
        const bool fin = XWAVE || lf >> 5 == q, bin = XWAVE || lb >> 5 == q;
        const uint32_t om_in = (uint32_t)(q * NE * kTileSites) * E, om_out = (uint32_t)((2 + q) * NE * kTileSites) * E;
        su3<T> h0, h, hy, u;
        load_rows(H, base + (uint32_t)(y0 * NX + x), h0);
        const uint32_t sy0 = base + (uint32_t)((y0 == 0 ? NY - 1 : y0 - 1) * NX + x);
        load_rows(H, sy0, h);
        load_link(U0, sy0, (uint32_t)(NE * kTileSites) * E, u);
        third_row(h.e[0], h.e[1], h.e[2]);
        third_row(h0.e[0], h0.e[1], h0.e[2]);
        PackedAh<T> carry(updated_link(h, u, h0));  // the y link from below (the lanes of x do not use it)
#pragma unroll 1
        for (int r = 0; r < ROWS; ++r) {
            const int y = y0 + r;
            const uint32_t s = base + (uint32_t)(y * NX + x);
            load_rows(H, base + (uint32_t)((y == NY - 1 ? 0 : y + 1) * NX + x), hy);
            load_link(U0, s, om_in, u);
            third_row(h0.e[0], h0.e[1], h0.e[2]);
            // in the plane: x + 1 from its lane, y + 1 loaded
#pragma unroll
            for (int k = 0; k < 6; ++k)
                h.e[k / 3][k % 3] = choose(q == 0, lane_get(h0.e[k / 3][k % 3], 4 * lf), hy.e[k / 3][k % 3]);
            if constexpr (!XWAVE) {
                if (!fin && q == 0) load_rows(H, base + (uint32_t)(y * NX + (x == NX - 1 ? 0 : x + 1)), h);
            }
            third_row(h.e[0], h.e[1], h.e[2]);
            su3<T> un = updated_link(h0, u, h);
            double f = (double)un.e[0][0].re + (double)un.e[1][1].re + (double)un.e[2][2].re;
            const PackedAh<T> own(un);
            PackedAh<T> acc = carry;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                acc.z[i] = choose(q == 0, lane_get(own.z[i], 4 * lb), carry.z[i]);
                const T db = lane_get(own.d[i], 4 * lb), dc = carry.d[i];
                acc.d[i] = q == 0 ? db : dc;
            }
            if constexpr (!XWAVE) {
                if (!bin && q == 0) {
                    const uint32_t sx = base + (uint32_t)(y * NX + (x == 0 ? NX - 1 : x - 1));
                    su3<T> hx, ux;
                    load_rows(H, sx, hx);
                    load_link(U0, sx, 0u, ux);
                    third_row(hx.e[0], hx.e[1], hx.e[2]);
                    acc = PackedAh<T>(updated_link(hx, ux, h0));
                }
            }
            acc.sub(own);
            carry = own;
            // out of the plane: z or t
            load_rows(H, s + dfw, h);
            load_link(U0, s, om_out, u);
            third_row(h.e[0], h.e[1], h.e[2]);
            un = updated_link(h0, u, h);
            f += (double)un.e[0][0].re + (double)un.e[1][1].re + (double)un.e[2][2].re;
            acc.sub(PackedAh<T>(un));
            load_rows(H, s + dbk, h);
            load_link(U0, s + dbk, om_out, u);
            acc.add(PackedAh<T>(updated_link(h, u, h0)));
            fsum += f;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                acc.z[i] = {half_sum(acc.z[i].re), half_sum(acc.z[i].im)};
                acc.d[i] = half_sum(acc.d[i]);
            }
            const T tr = (acc.d[0] + acc.d[1] + acc.d[2]) / T(3);
            const cx<T> diag = {T(2) * (acc.d[0] - tr), T(2) * (acc.d[1] - tr)};
            // this lane's two fields: 0 and 1, or 2 and 3
            const cx<T> va = choose(q == 0, acc.z[0], acc.z[2]), vb = choose(q == 0, acc.z[1], diag);
            cx<T>* d = buf + 2 * q * PL + y * RS + x;
            d[0] = va;
            d[PL] = vb;
            const double d0 = vb.re, d1 = vb.im;
            tsum += 2.0 * (double)norm2(va) + (q == 0 ? 2.0 * (double)norm2(vb) : d0 * d0 + d1 * d1 + (d0 + d1) * (d0 + d1));
#pragma unroll
            for (int k = 0; k < 6; ++k) h0.e[k / 3][k % 3] = hy.e[k / 3][k % 3];
        }
    }
    fsum = wave_sum(fsum);
    tsum = wave_sum(tsum);
    if (lane == 0) {
        sa[threadIdx.x >> 6] = fsum;
        sb[threadIdx.x >> 6] = tsum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) {
            a += sa[i];
            b += sb[i];
        }
        part[plane] = make_double2(a, b);
        if (blockIdx.x == 0) ctl->pending = 1;
    }
    fft_rows_ct<NX, 0, 1, Rows<4 * NY, 1, 4 * NY, RS, 0>, NT, T, false>(buf, twx);
    using RY = Rows<4 * NX, RS, NX, 1, PL>;
    fft_rows_io<NY, 0, 1, RY, NT, T, false>(buf, twy, LdsIo<RY, T>{buf}, PlaneOut<T, NX>{Q + base, zps}, threadIdx.x);
}

}  // namespace gf
