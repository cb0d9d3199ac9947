// APE smearing on packed 18-real links (the smeared links of the fat-link irrelevant clover
// operator).
#include "m3.h"
#include "launch.h"

namespace cola {

namespace {

using C = cpx<double>;

__device__ __forceinline__ C det3(const M3 &m) {
    const C c0 = cmul(m.a[1][1], m.a[2][2]) - cmul(m.a[1][2], m.a[2][1]);
    const C c1 = cmul(m.a[1][2], m.a[2][0]) - cmul(m.a[1][0], m.a[2][2]);
    const C c2 = cmul(m.a[1][0], m.a[2][1]) - cmul(m.a[1][1], m.a[2][0]);
    return cmadd(cmadd(cmul(m.a[0][0], c0), m.a[0][1], c1), m.a[0][2], c2);
}

// The SU(3) matrix nearest to V: the unitary polar factor W (V = W H, H Hermitian
// positive) by Newton's iteration X <- (g X + X^{-H} / g) / 2 with the determinant scaling
// g = |det X|^{-1/3}, X^{-H} the conjugated cofactors over conj(det X), then
// det(W)^{-1/3} with the principal cube root.  Convergence is quadratic: the error of an
// iterate is about half the square of the largest change that led to it, so the iteration
// ends with a change of at most 1e-9.
__device__ M3 project_su3(const M3 &V) {
    M3 X = V;
    for (int it = 0; it < 40; ++it) {
        const C det = det3(X);
        const double n = norm2(det), gi = cbrt(sqrt(n));  // 1 / g
        const double hg = 0.5 / gi, h = 0.5 * gi / n;
        const C hf = {h * det.x, h * det.y};  // 1 / (2 g conj(det))
        M3 Y;
        double change = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int i1 = (i + 1) % 3, i2 = (i + 2) % 3, j1 = (j + 1) % 3, j2 = (j + 2) % 3;
                const C cof = cmul(X.a[i1][j1], X.a[i2][j2]) - cmul(X.a[i1][j2], X.a[i2][j1]);
                C y = scale(hg, X.a[i][j]);
                y = cjmadd(y, cof, hf);
                change = fmax(change, fmax(fabs(y.x - X.a[i][j].x), fabs(y.y - X.a[i][j].y)));
                Y.a[i][j] = y;
            }
        X = Y;
        if (change <= 1e-9) break;
    }
    const C d = det3(X);
    const double th = atan2(d.y, d.x) / 3.0;
    const C ph = {cos(th), -sin(th)};  // det^{-1/3}
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) X.a[i][j] = cmul(X.a[i][j], ph);
    return X;
}

// One APE sweep: V_mu(x) = (1 - alpha) U_mu(x) + (alpha / 6) sum over nu != mu of the
// staples U_nu(x) U_mu(x+nu) U_nu(x+mu)^H and U_nu(x-nu)^H U_mu(x-nu) U_nu(x-nu+mu), then
// projected to SU(3).  Periodic links; reads U, writes Out (no aliasing).
//
// One lane per link; a wavefront takes 64 consecutive sites of one parity and direction, a
// block the four directions of a site range, which share their staples' links.  Bound by the
// FP64 arithmetic of the projection and the latency of the staples' loads (2.9 KB per
// link through the L2).  From canonical links, with four directions mixed in a wavefront:
// 978 us at 24^3 x 48; now 499 us (three wavefronts forming a staple direction each for
// three chunks in turn 648 us: barriers).
//
// CANON: Out is a canonical field.  The last of a call's sweeps writes that itself, the four
// directions of a site from one block into its 576 bytes: one sweep, packing included, 697 us
// at 24^3 x 48 and 19.4 us at 8^4; with a launch of its own for the layout 758 and 22.7.
template <bool CANON>
__global__ void __launch_bounds__(256)
    ape_kernel(const Geom g, const TileOrder order, const C *__restrict__ U, C *__restrict__ Out,
               double alpha) {
    const int S = g.S;
    const uint32_t bytes = (uint32_t)S * (uint32_t)sizeof(C);
    const uint32_t per = ((uint32_t)g.Vh + 63) / 64;
    uint32_t first, end, step;
    xcd_range(blockIdx.x, gridDim.x, 2 * per, &first, &end, &step);
    const int mu = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    for (uint32_t b = first; b < end; b += step) {
        const uint32_t q = (b >> 1) * 64 + (threadIdx.x & 63u);
        if (q >= (uint32_t)g.Vh) continue;
        Site s = tiled_site(g, order, q, (int)(b & 1u));
        // the empty asm keeps the compiler from loading the next staple's links before the
        // current one is summed
        auto fence = [&] {
            asm volatile("" : "+v"(s.i), "+v"(s.x[0]), "+v"(s.x[1]), "+v"(s.x[2]), "+v"(s.x[3]));
        };
        M3 A;
#pragma unroll
        for (int k = 0; k < 9; ++k) A.a[k / 3][k % 3] = C{0.0, 0.0};
#pragma unroll 1
        for (int k = 0; k < 3; ++k) {
            const int nu = k + (k >= mu ? 1 : 0);
            {
                M3 t = ldp(U, S, s, nu);
                mul_right(t, ldp(U, S, shifted(g, s, nu, 1), mu));
                mul_right_dag(t, ldp(U, S, shifted(g, s, mu, 1), nu));
                A = A + t;
            }
            fence();
            {
                const Site sm = shifted(g, s, nu, -1);
                M3 t = dag(ldp(U, S, sm, nu));
                mul_right(t, ldp(U, S, sm, mu));
                mul_right(t, ldp(U, S, shifted(g, sm, mu, 1), nu));
                A = A + t;
            }
            fence();
        }
        const M3 u = ldp(U, S, s, mu);
        const double a0 = 1.0 - alpha, a1 = alpha / 6.0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j)
                A.a[i][j] = {fma(a1, A.a[i][j].x, a0 * u.a[i][j].x),
                             fma(a1, A.a[i][j].y, a0 * u.a[i][j].y)};
        A = project_su3(A);
        if constexpr (CANON) {
            const size_t site =
                (size_t)s.x[0] +
                (size_t)g.L[0] * ((size_t)s.x[1] +
                                  (size_t)g.L[1] * ((size_t)s.x[2] + (size_t)g.L[2] * (size_t)s.x[3]));
            C *const o = Out + (site * 4 + mu) * 9;
#pragma unroll
            for (int k = 0; k < 9; ++k) o[k] = A.a[k / 3][k % 3];
            continue;
        }
        C *const o = Out + (size_t)((s.p * 4 + mu) * 9) * S;
        const uint32_t off = s.i * (uint32_t)sizeof(C);
#pragma unroll
        for (int k = 0; k < 9; ++k)
            bstore<C>(buf_u(o + (size_t)k * S, bytes), off, A.a[k / 3][k % 3]);
    }
}

}  // namespace

hipError_t launch_ape_sweep(const Geom &g, const void *U, void *Out, bool canonical, double alpha,
                            hipStream_t st) {
    if (U == Out) return hipErrorInvalidValue;
    size_t grid = 2 * (((size_t)g.Vh + 63) / 64);
    if (grid > 65536) grid = 65536;
    hipLaunchKernelGGL(canonical ? ape_kernel<true> : ape_kernel<false>, dim3((unsigned)grid),
                       dim3(256), 0, st, g, tile_order(g), (const C *)U, (C *)Out, alpha);
    return hipGetLastError();
}

}  // namespace cola
