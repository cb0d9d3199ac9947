// The molecular-dynamics step on packed fields: links U and momenta P in the packed 18-real
// layout (chunk k of the link (p, mu, i) at ((p 4 + mu) 9 + k) S + i), in which the 64 lanes
// of a wavefront, consecutive sites of one parity and one direction, access 64
// consecutive elements.
//
//   md step       P -= eps_p F_g(U), U' = exp(i eps_u P) U, sum of Re Tr (U A)
//   fermion kick  P -= eps F_f(U, X, Y)
//
// with F_g the force of the Wilson plaquette action and F_f the link-wise pseudofermion
// force (the formulas of the kernels on canonical fields).
#include "m3.h"
#include "launch.h"

namespace cola {

namespace {

using C = cpx<double>;

constexpr int kMdSites = 64;  // links of one block, all of one parity and direction
constexpr int kMdWaves = 3;   // wavefronts of one block

__device__ __forceinline__ C pick(int w, C a, C b, C c) { return w == 0 ? a : w == 1 ? b : c; }

// One block per 64 links.  Wavefront w first forms the two staples in the w-th direction
// nu != mu, then works on column w of the 3 x 3 matrices: W = U A, the force, P, the
// exponential (Taylor series by Horner on a unit vector, then squarings) and the new link.
// Matrices pass between the wavefronts through LDS.  Updating P and U in one pass reads
// the staples' links from the old field and writes another one.  Large lattices are bound
// by memory (P and U' written, P and U read: 0.58 KB per link) and the staples' loads through
// the L2 (2.7 KB per link), small ones by the chain of one block, which the split
// over columns shortens.  Separate kernels on canonical fields, one lane per link and
// three for the force, took 845 + 219 + 261 us (force, momenta, links) at 24^3 x 48 and
// 8.3 + 2.9 + 10.9 us at 8^4; this pass takes 664 and 10.0 us.
__global__ void __launch_bounds__(kMdWaves *kMdSites)
    md_step_kernel(const Geom g, const TileOrder order, const C *__restrict__ U, C *__restrict__ Un,
                   C *__restrict__ P, double beta, double eps_p, double eps_u, double *partial) {
    __shared__ C m[3][9][kMdSites];
    const uint32_t per = ((uint32_t)g.Vh + kMdSites - 1) / kMdSites;
    uint32_t first, end, step;
    xcd_range(blockIdx.x, gridDim.x, 8 * per, &first, &end, &step);
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kMdSites);
    const int l = (int)threadIdx.x & (kMdSites - 1);
    const int S = g.S;
    const uint32_t bytes = (uint32_t)S * (uint32_t)sizeof(C);
    double acc = 0.0;
    // the trip count is the same for all lanes of the block (barriers inside)
    for (uint32_t b = first; b < end; b += step) {
        // the eight (parity, direction) of a range of sites in turn: they share their links
        const int mu = (int)(b & 3u);
        const uint32_t q = (b >> 3) * kMdSites + (uint32_t)l;
        const bool valid = q < (uint32_t)g.Vh;
        const Site s = tiled_site(g, order, valid ? q : 0u, (int)((b >> 2) & 1u));
        {
            const int nu = w + (w >= mu ? 1 : 0);
            // upper: U_nu(x+mu) U_mu(x+nu)^H U_nu(x)^H
            M3 t = ldp(U, S, shifted(g, s, mu, 1), nu);
            mul_right_dag(t, ldp(U, S, shifted(g, s, nu, 1), mu));
            mul_right_dag(t, ldp(U, S, s, nu));
            // lower: U_nu(x+mu-nu)^H U_mu(x-nu)^H U_nu(x-nu)
            const Site sn = shifted(g, s, nu, -1);
            M3 v = dag(ldp(U, S, shifted(g, sn, mu, 1), nu));
            mul_right_dag(v, ldp(U, S, sn, mu));
            mul_right(v, ldp(U, S, sn, nu));
#pragma unroll
            for (int k = 0; k < 9; ++k) m[w][k][l] = t.a[k / 3][k % 3] + v.a[k / 3][k % 3];
        }
        const M3 u = ldp(U, S, s, mu);
        C *const pl = P + (size_t)((s.p * 4 + mu) * 9 + w) * S;
        const uint32_t off = s.i * (uint32_t)sizeof(C);
        C pj[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) pj[i] = bload<C>(buf_u(pl + (size_t)(3 * i) * S, bytes), off);
        __syncthreads();
        C c[3];  // column w of the matrix at hand
        {
            C a[3];
#pragma unroll
            for (int k = 0; k < 3; ++k)
                a[k] = (m[0][3 * k + w][l] + m[1][3 * k + w][l]) + m[2][3 * k + w][l];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                c[i] = cmadd(cmadd(cmul(u.a[i][0], a[0]), u.a[i][1], a[1]), u.a[i][2], a[2]);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 3; ++i) m[0][3 * i + w][l] = c[i];  // W
        __syncthreads();
        {
            // F = -(beta / 3) traceless part of i (W - W^H) / 2
            const double tr = -(m[0][0][l].y + m[0][4][l].y + m[0][8][l].y) / 3.0;
            const double f = -beta / 3.0;
            if (valid) acc += pick(w, c[0], c[1], c[2]).x;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const C wt = m[0][3 * w + i][l];
                C x = {-0.5 * (c[i].y + wt.y), 0.5 * (c[i].x - wt.x)};
                if (i == w) x = {x.x - tr, 0.0};
                pj[i] = {fma(-eps_p, f * x.x, pj[i].x), fma(-eps_p, f * x.y, pj[i].y)};
            }
        }
        if (valid) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                bstore<C>(buf_u(pl + (size_t)(3 * i) * S, bytes), off, pj[i]);
        }
        if (Un) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                m[1][3 * i + w][l] = valid ? pj[i] : C{0.0, 0.0};
            __syncthreads();
            // X = i eps_u P, halved until its Frobenius norm is at most 1/2
            M3 X;
            double nrm = 0.0;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const C v = m[1][k][l];
                X.a[k / 3][k % 3] = {-eps_u * v.y, eps_u * v.x};
                nrm += norm2(X.a[k / 3][k % 3]);
            }
            nrm = sqrt(nrm);
            int sq = 0;
            double sc = 1.0;
            while (nrm * sc > 0.5 && sq < 60) {
                sc *= 0.5;
                ++sq;
            }
            nrm *= sc;
#pragma unroll
            for (int k = 0; k < 9; ++k) X.a[k / 3][k % 3] = scale(sc, X.a[k / 3][k % 3]);
            // the order that leaves the truncation |X|^(n+1) / (n+1)! below 2.2e-20 on every lane
            const int order_n = !__any(!(nrm < 0.027))   ? 8
                                : !__any(!(nrm < 0.079)) ? 10
                                : !__any(!(nrm < 0.172)) ? 12
                                : !__any(!(nrm < 0.31))  ? 14
                                                         : 16;
            // column w of E = I + X/1 (I + X/2 (I + ...))
            C e[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) e[i] = {i == w ? 1.0 : 0.0, 0.0};
#pragma unroll
            for (int k = 16; k >= 1; --k) {
                if (k > order_n) continue;
                const double r = 1.0 / k;
                C t[3];
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    t[i] = cmadd(cmadd(cmul(X.a[i][0], e[0]), X.a[i][1], e[1]), X.a[i][2], e[2]);
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    e[i] = {fma(r, t[i].x, i == w ? 1.0 : 0.0), r * t[i].y};
            }
            auto exchange = [&] {  // m[0] = the columns of E
                __syncthreads();
#pragma unroll
                for (int i = 0; i < 3; ++i) m[0][3 * i + w][l] = e[i];
                __syncthreads();
            };
            exchange();
            // the same lane holds the same X in every wavefront: the trip count is the block's
            for (int k = 0; __any(sq > k); ++k) {
                if (sq > k) {
                    C t[3];
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        t[i] = cmadd(cmadd(cmul(m[0][3 * i][l], e[0]), m[0][3 * i + 1][l], e[1]),
                                     m[0][3 * i + 2][l], e[2]);
#pragma unroll
                    for (int i = 0; i < 3; ++i) e[i] = t[i];
                }
                exchange();
            }
            // U' = E U, then rows re-orthonormalised (row 2 = conj(row 0 x row 1))
            {
                C uj[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) uj[i] = pick(w, u.a[i][0], u.a[i][1], u.a[i][2]);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    c[i] = cmadd(cmadd(cmul(m[0][3 * i][l], uj[0]), m[0][3 * i + 1][l], uj[1]),
                                 m[0][3 * i + 2][l], uj[2]);
                    m[2][3 * i + w][l] = c[i];
                }
            }
            __syncthreads();
            C r0[3], r1[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                r0[j] = m[2][j][l];
                r1[j] = m[2][3 + j][l];
            }
            const double i0 = 1.0 / sqrt((norm2(r0[0]) + norm2(r0[1])) + norm2(r0[2]));
            C d = {0.0, 0.0};  // <row0, row1>
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                r0[j] = scale(i0, r0[j]);
                d = cmadd(d, conj(r0[j]), r1[j]);
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) r1[j] = r1[j] - cmul(d, r0[j]);
            const double i1 = 1.0 / sqrt((norm2(r1[0]) + norm2(r1[1])) + norm2(r1[2]));
#pragma unroll
            for (int j = 0; j < 3; ++j) r1[j] = scale(i1, r1[j]);
            // the cyclic successors of column w
            const C a1 = pick(w, r0[1], r0[2], r0[0]), a2 = pick(w, r0[2], r0[0], r0[1]);
            const C b1 = pick(w, r1[1], r1[2], r1[0]), b2 = pick(w, r1[2], r1[0], r1[1]);
            C *const ul = Un + (size_t)((s.p * 4 + mu) * 9 + w) * S;
            if (valid) {
                bstore<C>(buf_u(ul, bytes), off, pick(w, r0[0], r0[1], r0[2]));
                bstore<C>(buf_u(ul + (size_t)3 * S, bytes), off, pick(w, r1[0], r1[1], r1[2]));
                bstore<C>(buf_u(ul + (size_t)6 * S, bytes), off,
                          conj(cmul(a1, b2) - cmul(a2, b1)));
            }
        }
        __syncthreads();  // m is reused by the next pass
    }
    if (partial) {
        double *red = (double *)m;
        red[threadIdx.x] = acc;
        __syncthreads();
        if (threadIdx.x < kMdSites) {
            double v = (red[l] + red[kMdSites + l]) + red[2 * kMdSites + l];
#pragma unroll
            for (int o = kMdSites / 2; o > 0; o >>= 1) v += __shfl_down(v, o);
            if (l == 0) partial[blockIdx.x] = v;
        }
    }
}

// P -= eps F, F the Lie-algebra fermion force of packed X and Y: one lane per link, the
// lanes of a wavefront consecutive sites of one parity and direction, so that the
// direction's branches are scalar and every load is of consecutive elements.  Bound by
// memory (X, Y, U and P read, P written: 0.6 KB per link).  From canonical spinors into a
// force field (423 us at 24^3 x 48), and the momentum update from that (219 us); now 312 us.
__global__ void __launch_bounds__(256)
    fermion_kick_kernel(const Geom g, const TileOrder order, const C *__restrict__ U,
                        const C *__restrict__ X, const C *__restrict__ Y, C *__restrict__ P,
                        double kappa, Cplx64 ph0, Cplx64 ph1, Cplx64 ph2, Cplx64 ph3, double eps) {
    const int S = g.S;
    const uint32_t bytes = (uint32_t)S * (uint32_t)sizeof(C);
    const uint32_t per = ((uint32_t)g.Vh + 63) / 64;
    uint32_t first, end, step;
    xcd_range(blockIdx.x, gridDim.x, 2 * per, &first, &end, &step);
    const int mu = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    for (uint32_t b = first; b < end; b += step) {
        const uint32_t q = (b >> 1) * 64 + (threadIdx.x & 63u);
        if (q >= (uint32_t)g.Vh) continue;
        const Site s = tiled_site(g, order, q, (int)(b & 1u));
        const Site sf = shifted(g, s, mu, 1);
        // sum_s ((1 - g_mu) Y(x))_s X(x+mu)_s^H + X(x)_s ((1 + g_mu) Y(x+mu))_s^H over the two
        // projected components, one spinor at a time
        C G[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) G[k] = C{0.0, 0.0};
        auto half = [&](const C *v, const Site &t, double sg, C h[6]) {
            const SpinorBlock<SpinorFmt::F64> f(v + (size_t)t.p * 12 * S, S, 1);
            C sp[12];
            double unit;
            f.template load_unscaled<0>(t.i, 0, sp, &unit);
            project(mu, sg, sp, h);
        };
        C ha[6], hb[6];
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            half(pass ? X : Y, s, pass ? 1.0 : -1.0, ha);
            half(pass ? Y : X, sf, pass ? 1.0 : -1.0, hb);
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int c = 0; c < 3; ++c)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        G[a * 3 + c] = cjmadd(G[a * 3 + c], hb[k * 3 + c], ha[k * 3 + a]);
        }
        // 2 kappa conj(e+)
        const Cplx64 ph = mu == 0 ? ph0 : mu == 1 ? ph1 : mu == 2 ? ph2 : ph3;
        const bool bnd = (mu == 0   ? s.x[0]
                          : mu == 1 ? s.x[1]
                          : mu == 2 ? s.x[2]
                                    : s.x[3]) == g.L[mu] - 1;
        const C f = bnd ? C{2.0 * kappa * ph.x, -2.0 * kappa * ph.y} : C{2.0 * kappa, 0.0};
#pragma unroll
        for (int k = 0; k < 9; ++k) G[k] = cmul(f, G[k]);
        const M3 u = ldp(U, S, s, mu);
        M3 W;  // U G^H
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                C t = {0.0, 0.0};
#pragma unroll
                for (int k = 0; k < 3; ++k) t = cjmadd(t, G[c * 3 + k], u.a[a][k]);
                W.a[a][c] = t;
            }
        const M3 F = traceless_hermitian(W);
        C *const pl = P + (size_t)((s.p * 4 + mu) * 9) * S;
        const uint32_t off = s.i * (uint32_t)sizeof(C);
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const __amdgpu_buffer_rsrc_t r = buf_u(pl + (size_t)k * S, bytes);
            const C v = bload<C>(r, off), x = F.a[k / 3][k % 3];
            bstore<C>(r, off, C{fma(-eps, x.x, v.x), fma(-eps, x.y, v.y)});
        }
    }
}

// canonical [site][mu][3][3] <-> packed, 256 consecutive links of one field or two
// (blockIdx.y) per block.  The canonical side moves in contiguous runs and the links change
// layout in LDS: with one lane per link on both sides, a store touched a cache line per
// lane, and 24^3 x 48 links took 254 us (packing) and 424 us (unpacking); now 157 and 123 us.
constexpr int kLayoutLinks = 256;

template <bool PACK>
__global__ void __launch_bounds__(kLayoutLinks)
    md_layout_kernel(const Geom g, C *c0, C *c1, C *p0, C *p1) {
    __shared__ C m[kLayoutLinks * 9];
    C *const can = blockIdx.y ? c1 : c0, *const pk = blockIdx.y ? p1 : p0;
    const uint32_t n = 8u * (uint32_t)g.Vh;
    for (uint32_t base = blockIdx.x * kLayoutLinks; base < n; base += gridDim.x * kLayoutLinks) {
        const uint32_t t = base + threadIdx.x;
        const uint32_t len = 9u * (n - base < (uint32_t)kLayoutLinks ? n - base : (uint32_t)kLayoutLinks);
        C *const a = can + (size_t)base * 9;
        if constexpr (PACK) {
#pragma unroll
            for (uint32_t k = 0; k < 9; ++k) {
                const uint32_t e = k * kLayoutLinks + threadIdx.x;
                if (e < len) m[e] = a[e];
            }
            __syncthreads();
        }
        if (t < n) {
            const uint32_t s = t >> 2, row = s / (uint32_t)g.L[0];
            const uint32_t z = row / (uint32_t)g.L[1], tt = z / (uint32_t)g.L[2];
            const uint32_t p = (s - row * (uint32_t)g.L[0] + row - z * (uint32_t)g.L[1] + z -
                                tt * (uint32_t)g.L[2] + tt) & 1u;
            C *const o = pk + (size_t)((p * 4 + (t & 3u)) * 9) * g.S + (s >> 1);
            C *const q = m + threadIdx.x * 9;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                if constexpr (PACK)
                    o[(size_t)k * g.S] = q[k];
                else
                    q[k] = o[(size_t)k * g.S];
            }
        }
        if constexpr (!PACK) {
            __syncthreads();
#pragma unroll
            for (uint32_t k = 0; k < 9; ++k) {
                const uint32_t e = k * kLayoutLinks + threadIdx.x;
                if (e < len) a[e] = m[e];
            }
        }
        __syncthreads();  // m is reused by the next pass
    }
}

}  // namespace

hipError_t launch_md_pack(const Geom &g, const void *U, const void *P, void *Up, void *Pp,
                          hipStream_t st) {
    const size_t n = ((size_t)g.Vh * 8 + kLayoutLinks - 1) / kLayoutLinks;
    hipLaunchKernelGGL(md_layout_kernel<true>, dim3((unsigned)(n > 65536 ? 65536 : n), P ? 2 : 1),
                       dim3(256), 0, st, g, (C *)const_cast<void *>(U), (C *)const_cast<void *>(P),
                       (C *)Up, (C *)Pp);
    return hipGetLastError();
}

hipError_t launch_md_unpack(const Geom &g, void *U, void *P, const void *Up, const void *Pp,
                            hipStream_t st) {
    const size_t n = ((size_t)g.Vh * 8 + kLayoutLinks - 1) / kLayoutLinks;
    hipLaunchKernelGGL(md_layout_kernel<false>, dim3((unsigned)(n > 65536 ? 65536 : n), P ? 2 : 1),
                       dim3(256), 0, st, g, (C *)U, (C *)P, (C *)const_cast<void *>(Up),
                       (C *)const_cast<void *>(Pp));
    return hipGetLastError();
}

hipError_t launch_md_step(const Geom &g, const void *U, void *Unew, void *P, double beta,
                          double eps_p, double eps_u, double *partial, double *retr,
                          hipStream_t st) {
    if (U == Unew || U == P) return hipErrorInvalidValue;
    size_t grid = 8 * (((size_t)g.Vh + kMdSites - 1) / kMdSites);
    if (grid > (size_t)kRedMaxBlocks) grid = kRedMaxBlocks;
    hipLaunchKernelGGL(md_step_kernel, dim3((unsigned)grid), dim3(kMdWaves * kMdSites), 0, st, g,
                       tile_order(g), (const C *)U, (C *)Unew, (C *)P, beta, eps_p, eps_u,
                       retr ? partial : nullptr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !retr) return e;
    return launch_reduce_partials(partial, (int)grid, 1, retr, st);
}

hipError_t launch_fermion_kick(const Geom &g, const void *U, const void *X, const void *Y, void *P,
                               double kappa, const Cplx64 phase[4], double eps, hipStream_t st) {
    size_t grid = 2 * (((size_t)g.Vh + 63) / 64);
    if (grid > 65536) grid = 65536;
    hipLaunchKernelGGL(fermion_kick_kernel, dim3((unsigned)grid), dim3(256), 0, st, g,
                       tile_order(g), (const C *)U, (const C *)X, (const C *)Y, (C *)P, kappa,
                       phase[0], phase[1], phase[2], phase[3], eps);
    return hipGetLastError();
}

}  // namespace cola
