// Clover term: field strength from the four plaquette leaves around each site,
// assembled into the two Hermitian 6x6 chiral blocks of
//   A = 1 - kappa c_sw sum_{mu<nu} sigma_mu,nu F_mu,nu,
// and the per-block inverse by Cholesky factorisation (FP64).
//
// In the chiral basis sigma_mu,nu = (i/2)[g_mu, g_nu] is block diagonal; with
// Pauli matrices s1, s2, s3 acting on the two spins of a block,
//   upper block (spins 0,1): s3 (F_xy - F_zt) + s2 (F_xz + F_yt) + s1 (F_yz - F_xt)
//   lower block (spins 2,3): s3 (F_xy + F_zt) + s2 (F_xz - F_yt) + s1 (F_yz + F_xt)
// so each block is [[1 - k B3, -k (B1 - i B2)], [-k (B1 + i B2), 1 + k B3]] with
// k = kappa c_sw and B1..B3 the 3x3 colour combinations above.
#include "m3.h"
#include "launch.h"

namespace cola {

namespace {

using C = cpx<double>;

constexpr int kClovSites = 64;  // sites of one block
constexpr int kClovWaves = 3;   // wavefronts of one block

// F_mu,nu(x) = traceless part of (Q - Q^H) / (8i), Q = sum of the four leaves, from the
// packed links; left in f[k][l] (LDS).  Each leaf is a product of four links built from the
// left, and starts with the link that ended the one before (13 loads instead of 16).  Q is
// summed in LDS, and the empty asm keeps the compiler from computing the sites of later
// leaves first: the registers hold the product, two links and the loads under way.
__device__ __forceinline__ void field_strength(const Geom &g, const C *U, Site s, int mu, int nu,
                                               C (*f)[kClovSites], int l) {
    const int S = g.S;
    auto add = [&](const M3 &m) {
#pragma unroll
        for (int k = 0; k < 9; ++k) f[k][l] = f[k][l] + m.a[k / 3][k % 3];
        asm volatile("" : "+v"(s.i), "+v"(s.x[0]), "+v"(s.x[1]), "+v"(s.x[2]), "+v"(s.x[3]));
    };
    M3 e;  // the link that ends one leaf and starts the next
    {      // leaf 1: U_mu(x) U_nu(x+mu) U_mu(x+nu)^H U_nu(x)^H
        M3 m = ldp(U, S, s, mu);
        mul_right(m, ldp(U, S, shifted(g, s, mu, 1), nu));
        mul_right_dag(m, ldp(U, S, shifted(g, s, nu, 1), mu));
        e = ldp(U, S, s, nu);
        mul_right_dag(m, e);
#pragma unroll
        for (int k = 0; k < 9; ++k) f[k][l] = m.a[k / 3][k % 3];
    }
    {  // leaf 2: U_nu(x) U_mu(x-mu+nu)^H U_nu(x-mu)^H U_mu(x-mu)
        const Site sm = shifted(g, s, mu, -1);
        M3 m = e;
        mul_right_dag(m, ldp(U, S, shifted(g, sm, nu, 1), mu));
        mul_right_dag(m, ldp(U, S, sm, nu));
        e = ldp(U, S, sm, mu);
        mul_right(m, e);
        add(m);
    }
    {  // leaf 3: U_mu(x-mu)^H U_nu(x-mu-nu)^H U_mu(x-mu-nu) U_nu(x-nu)
        const Site smn = shifted(g, shifted(g, s, mu, -1), nu, -1);
        M3 m = dag(e);
        mul_right_dag(m, ldp(U, S, smn, nu));
        mul_right(m, ldp(U, S, smn, mu));
        e = ldp(U, S, shifted(g, s, nu, -1), nu);
        mul_right(m, e);
        add(m);
    }
    {  // leaf 4: U_nu(x-nu)^H U_mu(x-nu) U_nu(x+mu-nu) U_mu(x)^H
        const Site sn = shifted(g, s, nu, -1);
        M3 m = dag(e);
        mul_right(m, ldp(U, S, sn, mu));
        mul_right(m, ldp(U, S, shifted(g, sn, mu, 1), nu));
        mul_right_dag(m, ldp(U, S, s, mu));
        add(m);
    }
    // (Q - Q^H) / (8i) = -(1/4) i (Q - Q^H) / 2
    M3 q;
#pragma unroll
    for (int k = 0; k < 9; ++k) q.a[k / 3][k % 3] = f[k][l];
    q = traceless_hermitian(q);
#pragma unroll
    for (int k = 0; k < 9; ++k) f[k][l] = scale(-0.25, q.a[k / 3][k % 3]);
}

// A Hermitian 6 x 6 matrix: diagonal, and the entries below it row by row.
struct H6 {
    double d[6];
    C o[15];
};
__device__ __forceinline__ constexpr int low(int r, int c) { return r * (r - 1) / 2 + c; }

// a <- a^-1 for a positive definite, through its Cholesky factor L: with M = L^-1,
// a^-1 = M^H M.  Every index is a constant after unrolling, so the factors stay in
// registers.  False if a pivot is not positive.
__device__ __forceinline__ bool hpd_inverse6(H6 &a) {
    // L in place: diagonal entries as their reciprocals
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        double d = a.d[j];
#pragma unroll
        for (int k = 0; k < j; ++k) d -= norm2(a.o[low(j, k)]);
        if (!(d > 0.0)) return false;
        const double inv = 1.0 / sqrt(d);
        a.d[j] = inv;
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            C s = a.o[low(i, j)];
#pragma unroll
            for (int k = 0; k < j; ++k) {
                const C lik = a.o[low(i, k)], ljk = a.o[low(j, k)];
                // s -= l_ik conj(l_jk)
                s = cmadd(s, C{-lik.x, -lik.y}, conj(ljk));
            }
            a.o[low(i, j)] = scale(inv, s);
        }
    }
    // M = L^-1 in place, column by column: m_ij = -(1/l_ii) sum_{k=j}^{i-1} l_ik m_kj
#pragma unroll
    for (int j = 0; j < 6; ++j)
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            C s = scale(a.d[j], a.o[low(i, j)]);
#pragma unroll
            for (int k = j + 1; k < i; ++k) s = cmadd(s, a.o[low(i, k)], a.o[low(k, j)]);
            a.o[low(i, j)] = scale(-a.d[i], s);
        }
    // a^-1 = M^H M: row r of the product needs rows >= r of M only
#pragma unroll
    for (int r = 0; r < 6; ++r) {
#pragma unroll
        for (int c = 0; c < r; ++c) {
            C s = scale(a.d[r], a.o[low(r, c)]);
#pragma unroll
            for (int k = r + 1; k < 6; ++k) s = cmadd(s, conj(a.o[low(k, r)]), a.o[low(k, c)]);
            a.o[low(r, c)] = s;  // later rows of the product use rows > r of M only
        }
        double s = a.d[r] * a.d[r];
#pragma unroll
        for (int k = r + 1; k < 6; ++k) s += norm2(a.o[low(k, r)]);
        a.d[r] = s;
    }
    return true;
}

template <typename T>
__device__ __forceinline__ void store_block(void *out, int S, int p, uint32_t i, int blk,
                                            const H6 &a) {
    struct alignas(2 * sizeof(T)) pr { T a, b; };
    const pr *q = (const pr *)out + ((size_t)(p * 36 + blk * 18)) * S;
    const uint32_t bytes = (uint32_t)S * (uint32_t)sizeof(pr), off = i * (uint32_t)sizeof(pr);
#pragma unroll
    for (int k = 0; k < 18; ++k) {
        const pr v = k < 3 ? pr{(T)a.d[2 * k], (T)a.d[2 * k + 1]}
                           : pr{(T)a.o[k - 3].x, (T)a.o[k - 3].y};
        bstore<pr>(buf_u(q + (size_t)k * S, bytes), off, v);
    }
}

// One block per 64 sites of one parity: its three wavefronts form the field strengths of two
// planes each (xy, xz, xt, yz, yt, zt) in LDS, then the first two assemble, invert and
// store one chiral block each.  Bound by the latency of the link loads (7.5 GB through the
// L2 at 24^3 x 48, 10 TB/s; the FP64 arithmetic takes 0.2 ms).  One lane per site doing
// everything, from the canonical links, held the field strengths and the 6 x 6 matrices in
// scratch memory: 1184 us at 24^3 x 48, now 724 us (six wavefronts of one plane each 766 us;
// plain instead of tile order 814 us).
__global__ void __launch_bounds__(kClovWaves * kClovSites)
    clover_build_kernel(const Geom g, const TileOrder order, const C *__restrict__ U, double kc, void *a64, void *ainv64,
                        void *a32, void *ainv32, int *bad) {
    __shared__ C F[6][9][kClovSites];
    uint32_t first, end, step;
    const uint32_t per = ((uint32_t)g.Vh + kClovSites - 1) / kClovSites;  // blocks per parity
    xcd_range(blockIdx.x, gridDim.x, 2 * per, &first, &end, &step);
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kClovSites);
    const int l = (int)threadIdx.x & (kClovSites - 1);
    // the trip count is the same for all lanes of the block (barriers inside)
    for (uint32_t b = first; b < end; b += step) {
        // both parities of a range of sites in turn: they share their links
        const uint32_t q = (b >> 1) * kClovSites + (uint32_t)l;
        const bool valid = q < (uint32_t)g.Vh;
        const Site s = tiled_site(g, order, valid ? q : 0u, (int)(b & 1u));
        if (valid) {
#pragma unroll 1
            for (int pl = w; pl < 6; pl += kClovWaves) {
                const int mu = pl < 3 ? 0 : pl < 5 ? 1 : 2;
                const int nu = pl < 3 ? pl + 1 : pl < 5 ? pl - 1 : 3;
                field_strength(g, U, s, mu, nu, F[pl], l);
            }
        }
        __syncthreads();
        if (w < 2 && valid) {
            const double sgn = w == 0 ? -1.0 : 1.0;  // upper block: F_xy - F_zt, ...
            H6 a;
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const int k = r * 3 + c;
                    // [[1 - k B3, -k (B1 - i B2)], [-k (B1 + i B2), 1 + k B3]]
                    const C b2 = F[1][k][l] + scale(-sgn, F[4][k][l]);
                    const C b1 = F[3][k][l] + scale(sgn, F[2][k][l]);
                    a.o[low(3 + r, c)] = {-kc * (b1.x - b2.y), -kc * (b1.y + b2.x)};
                    if (c > r) continue;
                    const C b3 = F[0][k][l] + scale(sgn, F[5][k][l]);
                    if (c == r) {
                        a.d[r] = 1.0 - kc * b3.x;
                        a.d[3 + r] = 1.0 + kc * b3.x;
                    } else {
                        a.o[low(r, c)] = {-kc * b3.x, -kc * b3.y};
                        a.o[low(3 + r, 3 + c)] = {kc * b3.x, kc * b3.y};
                    }
                }
            store_block<double>(a64, g.S, s.p, s.i, w, a);
            store_block<float>(a32, g.S, s.p, s.i, w, a);
            if (!hpd_inverse6(a)) {
                atomicAdd(bad, 1);
                a = H6{};
            }
            store_block<double>(ainv64, g.S, s.p, s.i, w, a);
            store_block<float>(ainv32, g.S, s.p, s.i, w, a);
        }
        __syncthreads();  // F is reused by the next pass
    }
}

}  // namespace

hipError_t launch_clover_build(const Geom &g, const void *gauge64_18, double kappa, double csw,
                               void *a64, void *ainv64, void *a32, void *ainv32, int *bad,
                               hipStream_t st) {
    const size_t per = ((size_t)g.Vh + kClovSites - 1) / kClovSites;
    size_t grid = 2 * per;
    if (grid > 65536) grid = 65536;
    hipLaunchKernelGGL(clover_build_kernel, dim3((unsigned)grid), dim3(kClovWaves * kClovSites), 0, st, g,
                       tile_order(g), (const C *)gauge64_18, kappa * csw, a64, ainv64, a32, ainv32, bad);
    return hipGetLastError();
}

}  // namespace cola
