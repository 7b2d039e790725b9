// Monte Carlo generator of the input ensembles: SU(3) Wilson-action heatbath
// (Cabibbo-Marinari over three SU(2) subgroups, Kennedy-Pendleton sampling),
// over-relaxation, and the multi-hit average of temporal links. The paper
// gauge-fixes thermalised configurations (Section 3) and applies multi-hit to
// the temporal links first (Section 1); it does not state the algorithms, so
// the standard ones are used:
//
//   local weight of U = U_mu(x):  exp((beta/3) Re Tr(U A)),
//   A = sum_{nu != mu} [U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag + U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)]
//
// For a row pair (i, j) of W = U A, r = (Re(w00+w11), -Im(w01+w10), -Re(w01-w10), -Im(w00-w11))/2,
// k = |r|, V = (r0 + i r.sigma)/k; heatbath s = X V with x0 ~ sqrt(1-x0^2) exp(2 beta k x0 / 3)
// (Kennedy and Pendleton 1985) and a uniform direction; over-relaxation s = V^2. U <- s U for the
// pairs (0,1), (0,2), (1,2) in turn.
//
// Random numbers: Philox4x32-10 (Salmon, Moraes, Dror and Shaw 2011), key = the 64-bit seed, counter
// (link index 4s + mu, sweep or tag, (hit << 20) | (pair << 16) | call, purpose: 0 sweep, 1 multi-hit);
// one call gives two doubles in (0, 1] of 53 bits each. Every link's numbers depend only on its
// counter, so the result does not depend on the launch shape.
//
// The sweeps run on an even/odd copy of the links in the handle's workspace: one array per parity, site s
// at index s >> 1 (x is fastest and Nx is even, so s and s ^ 1 share an index and differ in parity), kept
// in tiles of 64 indices with the 36 matrix elements of a tile one after another, 1 KB each. A wave's 64
// lanes take consecutive sites of one parity, so every load and store of a link element is one run of
// 1 KB (two at tile borders), and a tile's links lie in one 36 KB run. One thread per link; links of one
// direction and one parity share no staple, so each (mu, parity) half is one launch. The canonical links
// ([site][mu][row][col]) are packed before the first sweep of a call and unpacked after the last.
#pragma once

#include "gf_device.hpp"

namespace gf {

constexpr int kMcThreads = 128;
constexpr int kMcAttempts = 64;

struct McGeom {
    int n[4];
    int half_x;  // Nx / 2
    long long vol;
};

struct McKey {
    unsigned k0, k1;
    unsigned word1;   // sweep or tag
    unsigned purpose;
};

// Philox4x32-10 on the counter (link, key.word1, word2, key.purpose). Only the link differs between the
// lanes of a wave, so after two rounds half of the state still is the same for all of them: the products
// with the link (round 1) and with what round 1 makes of it (round 2) are the same for every call on one
// link and are formed once (McStream), and the other products of those rounds are scalar. 16 vector
// products a call are left of 20, and they are most of a call's time.
struct McStream {
    unsigned lo1, hi2, lo2;  // low word of round 1's product with the link, both of round 2's
};

__device__ __forceinline__ McStream mc_stream(const McKey& key, unsigned link) {
    const unsigned long long p = 0xD2511F53ull * (unsigned long long)link;
    const unsigned c2 = (unsigned)(p >> 32) ^ key.purpose ^ key.k1;
    const unsigned long long q = 0xCD9E8D57ull * (unsigned long long)c2;
    return {(unsigned)p, (unsigned)(q >> 32), (unsigned)q};
}

__device__ __forceinline__ void philox4x32_10(const McKey& key, const McStream& st, unsigned word2, unsigned c[4]) {
    // round 1: counter words 0, 1 become hi1 ^ word1 ^ k0 and lo1 of the product with word2
    const unsigned long long p1 = 0xCD9E8D57ull * (unsigned long long)word2;
    const unsigned a0 = (unsigned)(p1 >> 32) ^ key.word1 ^ key.k0, a1 = (unsigned)p1;
    // round 2
    unsigned k0 = key.k0 + 0x9E3779B9u, k1 = key.k1 + 0xBB67AE85u;
    const unsigned long long p0 = 0xD2511F53ull * (unsigned long long)a0;
    c[0] = st.hi2 ^ (a1 ^ k0);
    c[1] = st.lo2;
    c[2] = st.lo1 ^ ((unsigned)(p0 >> 32) ^ k1);
    c[3] = (unsigned)p0;
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        const unsigned long long q0 = 0xD2511F53ull * (unsigned long long)c[0];
        const unsigned long long q1 = 0xCD9E8D57ull * (unsigned long long)c[2];
        c[0] = (unsigned)(q1 >> 32) ^ c[1] ^ k0;
        c[1] = (unsigned)q1;
        c[2] = (unsigned)(q0 >> 32) ^ c[3] ^ k1;
        c[3] = (unsigned)q0;
    }
}

// The two uniforms of Philox call `call` for this link, pair and hit.
__device__ __forceinline__ void mc_uniforms(const McKey& key, const McStream& st, int hit, int pair, int call, double& a,
                                            double& b) {
    unsigned c[4];
    philox4x32_10(key, st, ((unsigned)hit << 20) | ((unsigned)pair << 16) | (unsigned)call, c);
    const unsigned long long ma = ((unsigned long long)c[0] << 21) | (c[1] >> 11);
    const unsigned long long mb = ((unsigned long long)c[2] << 21) | (c[3] >> 11);
    const double scale = 1.1102230246251565e-16;  // 2^-53
    a = ((double)ma + 1.0) * scale;
    b = ((double)mb + 1.0) * scale;
}

__device__ __forceinline__ su3<double> mc_load(const double2* __restrict__ links, long long s, int mu) {
    const double2* p = links + (s * 4 + mu) * 9;
    su3<double> m;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const double2 v = p[k];
        m.e[k / 3][k % 3] = {v.x, v.y};
    }
    return m;
}

// Even/odd tiles: element e of U_mu at site s, of parity par, is entry (mu*9 + e) of tile (s >> 1) / 64.
constexpr int kMcTile = 64;
constexpr int kMcEntries = 36;
struct McTiles {
    double2* p;
    size_t hp;  // elements per entry and parity (a multiple of the tile)
};

__device__ __forceinline__ int mc_parity(const int c[4]) { return (c[0] + c[1] + c[2] + c[3]) & 1; }

// The first entry of U_mu at index h of parity par; entry e is e * kMcTile further on.
__device__ __forceinline__ double2* eo_at(const McTiles& P, unsigned h, int par, int mu) {
    return P.p + (size_t)par * kMcEntries * P.hp + ((size_t)(h / kMcTile) * kMcEntries + mu * 9) * kMcTile + h % kMcTile;
}

__device__ __forceinline__ su3<double> eo_load(const McTiles& P, unsigned h, int par, int mu) {
    const double2* q = eo_at(P, h, par, mu);
    su3<double> m;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const double2 v = q[k * kMcTile];
        m.e[k / 3][k % 3] = {v.x, v.y};
    }
    return m;
}

__device__ __forceinline__ void eo_store(const McTiles& P, unsigned h, int par, int mu, const su3<double>& m) {
    double2* q = eo_at(P, h, par, mu);
#pragma unroll
    for (int k = 0; k < 9; ++k) q[k * kMcTile] = {m.e[k / 3][k % 3].re, m.e[k / 3][k % 3].im};
}

// a * b^dagger
__device__ __forceinline__ su3<double> mc_mul_adj(const su3<double>& a, const su3<double>& b) {
    su3<double> c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<double> s = cmulc(a.e[i][0], b.e[j][0]);
            s = cfmac(s, a.e[i][1], b.e[j][1]);
            s = cfmac(s, a.e[i][2], b.e[j][2]);
            c.e[i][j] = s;
        }
    return c;
}

// a^dagger * b
__device__ __forceinline__ su3<double> mc_adj_mul(const su3<double>& a, const su3<double>& b) {
    su3<double> c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<double> s = cmul(conj(a.e[0][i]), b.e[0][j]);
            s = cfma(s, conj(a.e[1][i]), b.e[1][j]);
            s = cfma(s, conj(a.e[2][i]), b.e[2][j]);
            c.e[i][j] = s;
        }
    return c;
}

__device__ __forceinline__ long long mc_site(const McGeom& g, const int c[4]) {
    return c[0] + (long long)g.n[0] * (c[1] + (long long)g.n[1] * (c[2] + (long long)g.n[2] * c[3]));
}

__device__ __forceinline__ long long mc_step(const McGeom& g, const int c[4], int mu, int d) {
    int e[4] = {c[0], c[1], c[2], c[3]};
    e[mu] += d;
    if (e[mu] < 0) e[mu] += g.n[mu];
    if (e[mu] >= g.n[mu]) e[mu] -= g.n[mu];
    return mc_site(g, e);
}

// A site and its neighbours one step up and down every axis, as site numbers (below 2^30: 2^32 links).
struct McSite {
    unsigned s, up[4], dn[4];
};

// Coordinates of site s.
__device__ __forceinline__ void mc_coords(const McGeom& g, unsigned s, int c[4]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const unsigned n = (unsigned)g.n[d], q = s / n;
        c[d] = (int)(s - q * n);
        s = q;
    }
    c[3] = (int)s;
}

// Block blk of a sweep over (x, y) planes of `plane` items, `threads` a block: the planes are visited with
// z in groups of kMcZGroup inside the t loop, so that a plane's t neighbours were read kMcZGroup planes
// earlier by the same XCD (whose blocks are consecutive, xcd_remap) and are still in its L2 (half-sweep at
// 32^4: 223 us with blocks dealt round-robin, 193 in groups of 4, 197 and 194 in groups of 2 and 8). Every
// link's update is independent of the order.
constexpr unsigned kMcZGroup = 4;
__device__ __forceinline__ unsigned mc_plane_order(const McGeom& g, unsigned blk, unsigned plane, unsigned threads) {
    const unsigned nz = (unsigned)g.n[2], nt = (unsigned)g.n[3];
    if (plane % threads != 0 || nz % kMcZGroup != 0 || nz <= kMcZGroup) return blk;
    const unsigned bpp = plane / threads, pl = blk / bpp, off = blk - pl * bpp;
    const unsigned z = pl % kMcZGroup + kMcZGroup * (pl / (kMcZGroup * nt)), t = (pl / kMcZGroup) % nt;
    return (z + nz * t) * bpp + off;
}

// The same for planes of a multiple of eight blocks, as dealt to the XCDs in turn: XCD k takes the k-th band of rows
// of every plane, so that the z and t neighbours of its sites are its own on lattices of any length (one hit, against
// consecutive planes: 32 x 64 x 8 x 8 91 -> 73 us, 32^3 x 16 288 -> 268, 32^4 548 -> 515; plain order in bands of
// blocks without the z groups: 131 at 32^2 x 16^2 as here, 549 at 32^4; all with 19 registers in scratch memory).
__device__ __forceinline__ unsigned mc_band_order(const McGeom& g, unsigned blk, unsigned plane, unsigned threads) {
    const unsigned bpp = plane / threads;
    if (plane % threads != 0 || bpp % 8 != 0)
        return mc_plane_order(g, (unsigned)xcd_remap(blk, gridDim.x), plane, threads);
    const unsigned nz = (unsigned)g.n[2], nt = (unsigned)g.n[3], bpx = bpp / 8, i = blk / 8, pl = i / bpx;
    const unsigned off = blk % 8 * bpx + i % bpx;
    if (nz % kMcZGroup != 0 || nz <= kMcZGroup) return pl * bpp + off;
    const unsigned z = pl % kMcZGroup + kMcZGroup * (pl / (kMcZGroup * nt)), t = (pl / kMcZGroup) % nt;
    return (z + nz * t) * bpp + off;
}

__device__ __forceinline__ McSite mc_neighbours(const McGeom& g, const int c[4]) {
    McSite m;
    m.s = (unsigned)mc_site(g, c);
    unsigned st = 1;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const unsigned wrap = (unsigned)(g.n[d] - 1) * st;
        m.up[d] = c[d] == g.n[d] - 1 ? m.s - wrap : m.s + st;
        m.dn[d] = c[d] == 0 ? m.s + wrap : m.s - st;
        st *= (unsigned)g.n[d];
    }
    return m;
}

__device__ __forceinline__ su3<double> mc_zero_matrix() {
    su3<double> a;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) a.e[i][j] = {0.0, 0.0};
    return a;
}

__device__ __forceinline__ void mc_add(su3<double>& a, const su3<double>& b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) a.e[i][j] = a.e[i][j] + b.e[i][j];
}

// Staple sum of U_MU at a site of parity p from the even/odd tiles: for every other axis nu the upper staple,
// then the lower. Neighbours one step away have parity 1 - p, two steps away (x + mu - nu, the two steps are
// independent) parity p. MU is a template parameter so that the three planes unroll and the loads of one run
// ahead of the products of another.
template <int MU>
__device__ __forceinline__ su3<double> eo_staples(const McTiles& P, const McSite& m, int p) {
    su3<double> a = mc_zero_matrix();
#pragma unroll
    for (int nu = 0; nu < 4; ++nu) {
        if (nu == MU) continue;
        const unsigned s_pm = m.up[MU], s_mn = m.dn[nu];
        {
            const su3<double> t = mc_mul_adj(eo_load(P, s_pm >> 1, 1 - p, nu), eo_load(P, m.up[nu] >> 1, 1 - p, MU));
            mc_add(a, mc_mul_adj(t, eo_load(P, m.s >> 1, p, nu)));
        }
        {
            const su3<double> mb =
                mul(eo_load(P, s_mn >> 1, 1 - p, MU), eo_load(P, (s_pm + (s_mn - m.s)) >> 1, p, nu));
            mc_add(a, mc_adj_mul(mb, eo_load(P, s_mn >> 1, 1 - p, nu)));
        }
    }
    return a;
}

struct Su2 {
    cx<double> m00, m01, m10, m11;
};

__device__ __forceinline__ Su2 su2_quat(double a0, double a1, double a2, double a3) {
    return {{a0, a3}, {a2, a1}, {-a2, a1}, {a0, -a3}};
}

__device__ __forceinline__ Su2 su2_mul(const Su2& a, const Su2& b) {
    return {cmul(a.m00, b.m00) + cmul(a.m01, b.m10), cmul(a.m00, b.m01) + cmul(a.m01, b.m11),
            cmul(a.m10, b.m00) + cmul(a.m11, b.m10), cmul(a.m10, b.m01) + cmul(a.m11, b.m11)};
}

__device__ __forceinline__ void su2_embed_left(const Su2& s, su3<double>& m, int i, int j) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cx<double> ri = m.e[i][c], rj = m.e[j][c];
        m.e[i][c] = cmul(s.m00, ri) + cmul(s.m01, rj);
        m.e[j][c] = cmul(s.m10, ri) + cmul(s.m11, rj);
    }
}

// One Cabibbo-Marinari update of u with staple sum a. Returns the number of pairs left unchanged
// because every Kennedy-Pendleton attempt was rejected.
template <bool OR>
__device__ __forceinline__ int mc_cm_update(su3<double>& u, const su3<double>& a, double beta, const McKey& key,
                                            const McStream& st, int hit) {
    su3<double> w = mul(u, a);
    int rejected = 0;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const int i = p == 2 ? 1 : 0, j = p == 0 ? 1 : 2;
        const cx<double> w00 = w.e[i][i], w01 = w.e[i][j], w10 = w.e[j][i], w11 = w.e[j][j];
        const double r0 = (w00.re + w11.re) / 2.0, r1 = -(w01.im + w10.im) / 2.0;
        const double r2 = -(w01.re - w10.re) / 2.0, r3 = -(w00.im - w11.im) / 2.0;
        const double k = sqrt(r0 * r0 + r1 * r1 + r2 * r2 + r3 * r3);
        if (!(k > 0.0)) continue;
        const Su2 v = su2_quat(r0 / k, r1 / k, r2 / k, r3 / k);
        Su2 s;
        if (OR) {
            s = su2_mul(v, v);
        } else {
            // the angles are 2 pi times a uniform: cospi and sincospi reduce them exactly, without the general
            // reduction of a radian argument (with the second wave per SIMD, 118 -> 90 us a hit at 32^4)
            const double alpha = 2.0 * beta * k / 3.0;
            double x0 = 1.0;
            bool ok = false;
            for (int t = 1; t <= kMcAttempts && !ok; ++t) {
                double u1, u2, u3, u4;
                mc_uniforms(key, st, hit, p, 2 * t - 1, u1, u2);
                mc_uniforms(key, st, hit, p, 2 * t, u3, u4);
                const double cs = cospi(2.0 * u2);
                const double delta = -(log(u1) + cs * cs * log(u3)) / alpha;
                if (u4 * u4 <= 1.0 - 0.5 * delta) {
                    x0 = 1.0 - delta;
                    ok = true;
                }
            }
            if (!ok) {
                ++rejected;
                continue;
            }
            double cu, pu;
            mc_uniforms(key, st, hit, p, 0, cu, pu);
            const double cos_t = 2.0 * cu - 1.0;
            const double sin_t = sqrt(fmax(0.0, 1.0 - cos_t * cos_t));
            double sin_p, cos_p;
            sincospi(2.0 * pu, &sin_p, &cos_p);
            const double rad = sqrt(fmax(0.0, 1.0 - x0 * x0));
            s = su2_mul(su2_quat(x0, rad * sin_t * cos_p, rad * sin_t * sin_p, rad * cos_t), v);
        }
        su2_embed_left(s, u, i, j);
        su2_embed_left(s, w, i, j);
    }
    return rejected;
}

// One (MU, parity) half-sweep: thread h updates the h-th link of direction MU among the sites of the
// given parity, in lexicographic order. Block b adds its count of rejected pair updates to rej[b]
// (plain stores: the launches of a sweep are ordered on one stream).
//
// Bound by memory: a lane reads 19 matrices (2.7 KB), which the L1s do not hold between lanes, so every one
// is an L2 read, and the field itself (576 B per site) comes through the L2s once if the blocks in flight
// stay close together. The launch therefore asks for LDS it does not use, which holds a CU to few blocks:
// over-relaxation two (four waves; 32^4: 193 -> 156 us a half-sweep, 158 with three KB less, 165 with one
// block), heatbath three (its arithmetic wants more waves: 183 -> 178 us, 198 with two).
constexpr size_t kMcLdsHeatbath = 50000, kMcLdsOverrelax = 64000;
template <int MU, bool OR>
__global__ void __launch_bounds__(kMcThreads) k_mc_update(McTiles P, McGeom g, int parity, double beta, McKey key,
                                                          unsigned* __restrict__ rej) {
    __shared__ unsigned red[kMcThreads];
    const unsigned h = mc_plane_order(g, (unsigned)xcd_remap(blockIdx.x, gridDim.x),
                                      (unsigned)(g.half_x * g.n[1]), kMcThreads) * kMcThreads + threadIdx.x;
    unsigned rj = 0;
    if (h < (unsigned)(g.vol / 2)) {
        int c[4];
        mc_coords(g, 2 * h, c);
        c[0] += mc_parity(c) != parity;
        const McSite m = mc_neighbours(g, c);
        const su3<double> a = eo_staples<MU>(P, m, parity);
        su3<double> u = eo_load(P, m.s >> 1, parity, MU);
        rj = (unsigned)mc_cm_update<OR>(u, a, beta, key, OR ? McStream{} : mc_stream(key, m.s * 4 + MU), 0);
        eo_store(P, m.s >> 1, parity, MU, u);
    }
    if (OR) return;
    red[threadIdx.x] = rj;
    __syncthreads();
    for (int w = kMcThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0 && red[0]) rej[blockIdx.x] += red[0];
}

// Canonical links <-> even/odd tiles. A block moves kMcIoSites consecutive sites (kMcIoSites / 2 indices of
// either parity) through LDS, so that the canonical side is one contiguous run and the tile side runs of
// kMcIoSites / 2 elements (32^4: one thread per site took 282 us in and 407 out; 200 and 240 this way, the
// last with the reunitarisation, a pass of 182 us before). A site's row in LDS is 37 elements (36 + 1).
constexpr int kMcIoSites = 64;
constexpr int kMcIoRow = kMcEntries + 1;

// Parity of site s.
__device__ __forceinline__ int mc_site_parity(const McGeom& g, unsigned s) {
    int c[4];
    mc_coords(g, s, c);
    return mc_parity(c);
}

__global__ void __launch_bounds__(256) k_mc_pack(const double2* __restrict__ links, McTiles P, McGeom g) {
    __shared__ double2 row[kMcIoSites * kMcIoRow];
    const unsigned s0 = blockIdx.x * kMcIoSites;
    const unsigned left = (unsigned)g.vol - s0, ns = left < kMcIoSites ? left : kMcIoSites;
    const double2* src = links + (size_t)s0 * kMcEntries;
    for (unsigned i = threadIdx.x; i < ns * kMcEntries; i += 256) row[(i / kMcEntries) * kMcIoRow + i % kMcEntries] = src[i];
    __syncthreads();
    // lane q of a wave: parity q / 32, index q % 32; the waves share the 36 entries
    const unsigned q = threadIdx.x & 63, w = threadIdx.x >> 6, i = q & 31;
    if (2 * i < ns) {
        const int par = (int)(q >> 5), odd = mc_site_parity(g, s0 + 2 * i) != par;  // which of the two sites has it
        double2* dst = eo_at(P, (s0 >> 1) + i, par, 0);
        for (unsigned k = w * 9; k < w * 9 + 9; ++k) dst[k * kMcTile] = row[(2 * i + odd) * kMcIoRow + k];
    }
}

// Every link is reunitarised on its way out (the end of a call's last sweep).
__global__ void __launch_bounds__(256) k_mc_unpack(McTiles P, McGeom g, double2* __restrict__ links) {
    __shared__ double2 row[kMcIoSites * kMcIoRow];
    const unsigned s0 = blockIdx.x * kMcIoSites;
    const unsigned left = (unsigned)g.vol - s0, ns = left < kMcIoSites ? left : kMcIoSites;
    const unsigned q = threadIdx.x & 63, mu = threadIdx.x >> 6, i = q & 31;
    if (2 * i < ns) {
        const int par = (int)(q >> 5), odd = mc_site_parity(g, s0 + 2 * i) != par;
        su3<double> m = eo_load(P, (s0 >> 1) + i, par, (int)mu);
        reunitarize(m);
        double2* dst = row + (2 * i + odd) * kMcIoRow + mu * 9;
#pragma unroll
        for (int k = 0; k < 9; ++k) dst[k] = {m.e[k / 3][k % 3].re, m.e[k / 3][k % 3].im};
    }
    __syncthreads();
    double2* dst = links + (size_t)s0 * kMcEntries;
    for (unsigned j = threadIdx.x; j < ns * kMcEntries; j += 256) dst[j] = row[(j / kMcEntries) * kMcIoRow + j % kMcEntries];
}

// Every link reunitarised in the tiles (between the sweeps of one call): thread per (mu, parity, index).
__global__ void __launch_bounds__(256) k_mc_reunit(McTiles P, unsigned half) {
    const unsigned h = blockIdx.x * 256 + threadIdx.x;
    if (h >= half) return;
    const int mu = (int)blockIdx.y >> 1, par = (int)blockIdx.y & 1;
    su3<double> m = eo_load(P, h, par, mu);
    reunitarize(m);
    eo_store(P, h, par, mu, m);
}

__global__ void __launch_bounds__(256) k_mc_zero(unsigned* __restrict__ p, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Sum of n counters into *out (one block, fixed order).
__global__ void __launch_bounds__(256) k_mc_count(const unsigned* __restrict__ p, int n,
                                                  unsigned long long* __restrict__ out) {
    __shared__ unsigned long long red[256];
    unsigned long long v = 0;
    for (int i = threadIdx.x; i < n; i += 256) v += p[i];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// Multi-hit average of every temporal link, out as complex double [site][row][col], straight from the
// canonical links. The staples are bound by memory (a lane's 144-byte links lie in two 128-byte lines, 5 KB
// of lines per site) and the hits by arithmetic: with two waves per SIMD one covers the other. Measured at
// 32^4 with 8 hits: 1385 us at one wave per SIMD (260 registers), 895 at two; the staple sums in a kernel
// of their own 1150, packing into the tiles first 1040. One-wave blocks: they spread evenly over the SIMDs
// of a small lattice (16^4: 125 us with two-wave blocks, 88). The plane's products in a function of their own: as the
// body of the loop they cost 19 registers in scratch memory instead of 4 (one hit: 32^4 514 -> 456 us,
// 32 x 64 x 8 x 8 73 -> 64; 8 hits 895 -> 880).
constexpr int kMhThreads = 64;
__global__ void __launch_bounds__(kMhThreads, 2) k_mc_multihit(const double2* __restrict__ links, McGeom g, double beta,
                                                               McKey key, int nhits, double2* __restrict__ out) {
    const unsigned s = mc_band_order(g, blockIdx.x, (unsigned)(g.n[0] * g.n[1]), kMhThreads) * kMhThreads + threadIdx.x;
    if (s >= (unsigned)g.vol) return;
    su3<double> a = mc_zero_matrix();
    {
        int c[4];
        mc_coords(g, s, c);
        const McSite m = mc_neighbours(g, c);
        const unsigned s_pt = m.up[3];
        auto plane = [&](int nu, unsigned s_pn, unsigned s_mn) {
            const su3<double> t = mc_mul_adj(mc_load(links, s_pt, nu), mc_load(links, s_pn, 3));
            mc_add(a, mc_mul_adj(t, mc_load(links, s, nu)));
            const su3<double> mb = mul(mc_load(links, s_mn, 3), mc_load(links, s_pt + (s_mn - s), nu));
            mc_add(a, mc_adj_mul(mb, mc_load(links, s_mn, nu)));
        };
#pragma unroll 1
        for (int nu = 0; nu < 3; ++nu)  // not unrolled: the loads of three planes in flight take the registers
            plane(nu, nu == 0 ? m.up[0] : nu == 1 ? m.up[1] : m.up[2], nu == 0 ? m.dn[0] : nu == 1 ? m.dn[1] : m.dn[2]);
    }
    su3<double> u = mc_load(links, s, 3);
    su3<double> acc = mc_zero_matrix();
    const McStream st = mc_stream(key, s * 4 + 3);
    for (int h = 0; h < nhits; ++h) {
        (void)mc_cm_update<false>(u, a, beta, key, st, h);
        mc_add(acc, u);
    }
    double2* p = out + (size_t)s * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k) p[k] = {acc.e[k / 3][k % 3].re / nhits, acc.e[k / 3][k % 3].im / nhits};
}

// Plaquette partials: block b sums Re Tr of the six plaquettes at each of its sites (fixed order).
__global__ void __launch_bounds__(256) k_mc_plaquette(const double2* __restrict__ links, McGeom g,
                                                      double* __restrict__ part) {
    __shared__ double red[256];
    const long long s = (long long)blockIdx.x * 256 + threadIdx.x;
    double v = 0.0;
    if (s < g.vol) {
        int c[4];
        long long r = s;
        for (int d = 0; d < 4; ++d) {
            c[d] = (int)(r % g.n[d]);
            r /= g.n[d];
        }
        for (int mu = 0; mu < 4; ++mu)
            for (int nu = mu + 1; nu < 4; ++nu) {
                const su3<double> t = mul(mc_load(links, s, mu), mc_load(links, mc_step(g, c, mu, 1), nu));
                const su3<double> q = mc_mul_adj(mc_mul_adj(t, mc_load(links, mc_step(g, c, nu, 1), mu)),
                                                 mc_load(links, s, nu));
                v += q.e[0][0].re + q.e[1][1].re + q.e[2][2].re;
            }
    }
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(256) k_mc_plaquette_sum(const double* __restrict__ part, int n, double scale,
                                                          double* __restrict__ out) {
    __shared__ double red[256];
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) v += part[i];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0] * scale;
}

}  // namespace gf
