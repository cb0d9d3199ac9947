// Hop for small launches: the eight directions of a site in eight wavefronts (FP64 and
// FP32).
//
// hop_kernel gives a (site, rhs) one lane, which takes the directions one after the other.
// A launch of few lanes then leaves most of the chip idle and waits for eight load
// latencies in a row.  Here a block owns up to 64 (site, rhs) and wavefront d computes
// direction d for all of them: its link and neighbour spinor, projection, SU(3) product,
// phase; the half spinors meet in LDS, and wavefront s < 4 adds spin s of the eight
// directions in the order of hop_kernel and applies the epilogue to its three components
// (whose own loads it issued before).  The same operations in the same order: the outputs
// agree with hop_kernel bitwise.
#pragma once

#include "hop_impl.h"

namespace cola {

// spin S of direction (MU, DIR) added into three accumulated components; w: the six half
// spinor components of the direction (boundary sign included)
template <int S, int MU, typename T>
__device__ __forceinline__ void add_spin(T sg, const cpx<T> (*w)[kDirsSites], int l,
                                         cpx<T> acc[3]) {
    // see expand_add: spin 2 and 3 receive +-(i) W0 or W1
    constexpr int half = S < 2 ? S : (MU < 2 ? 3 - S : S - 2);  // which of W0, W1
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cpx<T> v = w[3 * half + c][l];
        if constexpr (S < 2)
            acc[c] = add_s(acc[c], (T)1, v);
        else if constexpr (MU == 0)
            acc[c] = add_si(acc[c], -sg, v);
        else if constexpr (MU == 1)
            acc[c] = add_s(acc[c], S == 2 ? sg : -sg, v);
        else if constexpr (MU == 2)
            acc[c] = add_si(acc[c], S == 2 ? -sg : sg, v);
        else
            acc[c] = add_s(acc[c], sg, v);
    }
}

template <int S, typename T>
__device__ __forceinline__ void sum_spin(T sg_f, const cpx<T> (*W)[6][kDirsSites], int l,
                                         cpx<T> acc[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = {(T)0, (T)0};
    const T sg_b = -sg_f;
    add_spin<S, 3>(sg_b, W[7], l, acc);  // the order of hop_order
    add_spin<S, 0>(sg_f, W[0], l, acc);
    add_spin<S, 0>(sg_b, W[1], l, acc);
    add_spin<S, 1>(sg_f, W[2], l, acc);
    add_spin<S, 1>(sg_b, W[3], l, acc);
    add_spin<S, 2>(sg_f, W[4], l, acc);
    add_spin<S, 2>(sg_b, W[5], l, acc);
    add_spin<S, 3>(sg_f, W[6], l, acc);
}

// the half spinor of direction (MU, DIR) into w
template <int MU, int DIR, SpinorFmt SF, LinkFmt LF, bool RPH>
__device__ __forceinline__ void half_spinor(const HopArgs &a, const SpinorBlock<SF, kWalk> &in,
                                            int p, uint32_t i, const int x[4], uint32_t j,
                                            typename SpinorT<SF>::real sg_f,
                                            cpx<typename SpinorT<SF>::real> (*w)[kDirsSites],
                                            int l) {
    using T = typename SpinorT<SF>::real;
    using C = cpx<T>;
    const Geom &g = a.g;
    const T sg = DIR == 0 ? sg_f : -sg_f;
    const uint32_t n = DIR == 0 ? nb_fwd(g, i, x, MU) : nb_bwd(g, i, x, MU);
    Fetched<SF, 1> f;
    fetch_site<SF>(in, n, j, f);
    C u[3][3], h[6], r[6];
    load_link<LF, T>(a.gauge, g.S, DIR == 0 ? p : 1 - p, MU, DIR == 0 ? i : n, u);
    project(MU, sg, f.s[0], h);
    if constexpr (DIR == 0) {
        su3_mul(u, h, r);
        su3_mul(u, h + 3, r + 3);
    } else {
        su3_dag_mul(u, h, r);
        su3_dag_mul(u, h + 3, r + 3);
    }
    const bool bnd = DIR == 0 ? x[MU] == g.L[MU] - 1 : x[MU] == 0;
    if constexpr (RPH) {  // a real phase is a sign: its product is exact
        const T eta = bnd ? (T)a.phase[MU].x : (T)1;
#pragma unroll
        for (int k = 0; k < 6; ++k) w[k][l] = scale(eta, r[k]);
    } else {
        const T im = DIR == 0 ? (T)a.phase[MU].y : -(T)a.phase[MU].y;
        const C ph = bnd ? C{(T)a.phase[MU].x, im} : C{(T)1, (T)0};
#pragma unroll
        for (int k = 0; k < 6; ++k) w[k][l] = cmul(ph, r[k]);
    }
}

// Rows 3 s2 .. 3 s2 + 2 of chiral block blk of C v (s2 = 0, 1), v in LDS: the arithmetic of
// clover_apply.
template <typename CR, typename T>
__device__ __forceinline__ void clover_rows(const void *clov, int S, int p, uint32_t i, int blk,
                                            int s2, const cpx<T> (*v)[kDirsSites], int l,
                                            cpx<T> out[3]) {
    struct pair { CR a, b; };
    const pair *q = (const pair *)clov + (size_t)(p * 36 + blk * 18) * S;
    const uint32_t bytes = (uint32_t)S * (uint32_t)sizeof(pair);
    const uint32_t off = i * (uint32_t)sizeof(pair);
    auto ld = [&](int k) {
        return bload<pair, kCpolNT>(buf_u(q + (size_t)k * S, bytes), off);
    };
    cpx<T> in[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) in[c] = v[6 * blk + c][l];
    auto rows = [&](auto half) {
        constexpr int r0 = 3 * decltype(half)::value;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int r = r0 + k;
            const pair dp = ld(r / 2);
            cpx<T> s = scale(r % 2 ? (T)dp.b : (T)dp.a, in[r]);
#pragma unroll
            for (int c = 0; c < 6; ++c) {
                if (c == r) continue;
                const int hi = c < r ? r : c, lo = c < r ? c : r;
                const pair o = ld(3 + hi * (hi - 1) / 2 + lo);
                const cpx<T> e = {(T)o.a, (T)o.b};
                s = c < r ? cmadd(s, e, in[c]) : cjmadd(s, e, in[c]);
            }
            out[k] = s;
        }
    };
    if (s2 == 0)
        rows(std::integral_constant<int, 0>{});
    else
        rows(std::integral_constant<int, 1>{});
}

template <SpinorFmt SF, LinkFmt LF, typename CR, int EPI, bool RPH>
__global__ void __launch_bounds__(8 * kDirsSites) hop_dirs_kernel(const HopArgs a) {
    using T = typename SpinorT<SF>::real;
    using C = cpx<T>;
    using E = typename SpinorT<SF>::elem;
    constexpr bool CG = EPI == EPI_XPAY_CG || EPI == EPI_CLOV_XPAY_CG;
    constexpr bool CLV = EPI == EPI_CLOV || EPI == EPI_CLOV_XPAY || EPI == EPI_XPAY_CLOV ||
                         EPI == EPI_CLOV_XPAY_CG;
    constexpr bool XIN = EPI == EPI_XPAY || EPI == EPI_CLOV_XPAY || EPI == EPI_XPAY_CLOV || CG;
    __shared__ C W[8][6][kDirsSites];
    __shared__ C D[CLV ? 12 : 1][kDirsSites];  // the vector a clover block is applied to
    const Geom &g = a.g;
    // block -> chunk of sites_per_block sites (both: of each parity in turn)
    uint32_t ch, end, step;
    xcd_range(blockIdx.x, gridDim.x, gridDim.x, &ch, &end, &step);
    const int p = a.both ? (int)(ch & 1u) : a.parity;
    if (a.both) ch >>= 1;
    const size_t po = a.both ? (size_t)p * a.pstride : 0, no = a.both ? (size_t)(1 - p) * a.pstride : 0;
    const int d = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int l = (int)(threadIdx.x & 63u);
    const uint32_t R = (uint32_t)a.nrhs;
    const uint32_t sl = fdiv((uint32_t)l, a.div_groups);  // groups = nrhs
    const uint32_t j = (uint32_t)l - sl * R;
    const uint32_t i = ch * (uint32_t)a.sites_per_block + sl;
    const bool valid = sl < (uint32_t)a.sites_per_block && i < (uint32_t)g.Vh;
    const T sg_f = a.dagger ? (T)1 : (T)-1;

    // this lane's components of the epilogue's vectors (wavefronts 0-3: spin d)
    const uint32_t SR = (uint32_t)g.S * R, off = (i * R + j) * (uint32_t)sizeof(E);
    auto arrays = [&](const void *base) {
        const uint64_t stride = (uint64_t)SR * sizeof(E);
        return ArrayWalk<>((const char *)base + po + (uint64_t)(3 * d) * stride, stride,
                           SR * (uint32_t)sizeof(E));
    };
    auto own = [&](const void *base, C v[3]) {
        auto w = arrays(base);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const E e = bload<E, kCpolNT>(w.next(), off);
            v[c] = {e.x, e.y};
        }
    };
    C xv[3], cr[3];
    if (d < 4 && valid) {
        if constexpr (XIN) own(a.x, xv);
        if constexpr (CG) own(a.cg_r, cr);
    }
    // pi may be (one rhs) partial sums: loaded here, added once the neighbours are in
    __shared__ double sums[4];
    double tp[8];
    if constexpr (CG) {
        if (d < 4 && a.cg_pi_n) partial_terms(a.cg_pi, a.cg_pi_n, (int)threadIdx.x, tp);
    }
    if (valid) {
        const SpinorBlock<SF, kWalk> in((const char *)a.in + no, g.S, a.nrhs);
        int x[4];
        site_coords(g, i, p, x);
        switch (d) {
            case 0: half_spinor<0, 0, SF, LF, RPH>(a, in, p, i, x, j, sg_f, W[0], l); break;
            case 1: half_spinor<0, 1, SF, LF, RPH>(a, in, p, i, x, j, sg_f, W[1], l); break;
            case 2: half_spinor<1, 0, SF, LF, RPH>(a, in, p, i, x, j, sg_f, W[2], l); break;
            case 3: half_spinor<1, 1, SF, LF, RPH>(a, in, p, i, x, j, sg_f, W[3], l); break;
            case 4: half_spinor<2, 0, SF, LF, RPH>(a, in, p, i, x, j, sg_f, W[4], l); break;
            case 5: half_spinor<2, 1, SF, LF, RPH>(a, in, p, i, x, j, sg_f, W[5], l); break;
            case 6: half_spinor<3, 0, SF, LF, RPH>(a, in, p, i, x, j, sg_f, W[6], l); break;
            default: half_spinor<3, 1, SF, LF, RPH>(a, in, p, i, x, j, sg_f, W[7], l); break;
        }
    }
    if constexpr (CG) {
        if (d < 4 && a.cg_pi_n) {
            const double s = partial_wave(tp);
            if (l == 0) sums[d] = s;
        }
    }
    __syncthreads();
    const T ca = (T)a.a;
    C o[3];
    if (d < 4 && valid) {
        switch (d) {
            case 0: sum_spin<0, T>(sg_f, W, l, o); break;
            case 1: sum_spin<1, T>(sg_f, W, l, o); break;
            case 2: sum_spin<2, T>(sg_f, W, l, o); break;
            default: sum_spin<3, T>(sg_f, W, l, o); break;
        }
        if constexpr (EPI == EPI_XPAY || EPI == EPI_XPAY_CG || EPI == EPI_XPAY_CLOV) {
#pragma unroll
            for (int c = 0; c < 3; ++c) o[c] = add_s(xv[c], ca, o[c]);
        }
        if constexpr (CLV) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
                D[3 * d + c][l] = EPI == EPI_CLOV_XPAY || EPI == EPI_CLOV_XPAY_CG ? xv[c] : o[c];
        }
    }
    if constexpr (CLV) {
        __syncthreads();
        if (d < 4 && valid) {
            C y[3];
            clover_rows<CR, T>(a.clov, g.S, p, i, d >> 1, d & 1, D, l, y);
#pragma unroll
            for (int c = 0; c < 3; ++c)
                o[c] = EPI == EPI_CLOV_XPAY || EPI == EPI_CLOV_XPAY_CG ? add_s(y[c], ca, o[c]) : y[c];
        }
    }
    double nrm = 0.0;
    if (d < 4 && valid) {
        auto put = [&](const void *base, const C v[3]) {
            auto w = arrays(base);
#pragma unroll
            for (int c = 0; c < 3; ++c) bstore<E>(w.next(), off, E{v[c].x, v[c].y});
        };
        if constexpr (CG) {
            const double den = a.cg_pi_n ? ((sums[0] + sums[1]) + sums[2]) + sums[3] : a.cg_pi[j];
            const T al = (T)(a.cg_active[j] && den != 0.0 ? a.cg_rho[j] / den : 0.0);
#pragma unroll
            for (int c = 0; c < 3; ++c)
                o[c] = {fma(-al, o[c].x, cr[c].x), fma(-al, o[c].y, cr[c].y)};
            put(a.cg_r, o);
        } else {
            put(a.out, o);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) nrm += (double)norm2(o[c]);
    }
    if (a.want_norm) {
        // the lanes of a rhs (l, l + R, ...) in lane order, then the four spins in order
        __shared__ double red[4][kRedMaxWidth];
        const int live = a.sites_per_block * a.nrhs;
        double s = nrm;
        if (a.nrhs == 1) {
            for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m);
        } else {
            for (int m = a.nrhs; m < live; m += a.nrhs) {
                const double v = __shfl(nrm, (l + m) & 63);
                if (l + m < live) s += v;
            }
        }
        if (d < 4 && l < a.nrhs) red[d][l] = s;
        __syncthreads();
        if ((int)threadIdx.x < a.nrhs) {
            const int q = (int)threadIdx.x;
            a.partial[(size_t)q * gridDim.x + blockIdx.x] =
                ((red[0][q] + red[1][q]) + red[2][q]) + red[3][q];
        }
    }
}

template <SpinorFmt SF, LinkFmt LF, typename CR, bool RPH>
hipError_t hop_dirs_launch_epi(const HopArgs &a, int grid, hipStream_t st) {
    const dim3 gr(grid), bl(8 * kDirsSites);
    switch (a.epi) {
#define COLA_DIRS(E)                                                                       \
    case E:                                                                                \
        hipLaunchKernelGGL((hop_dirs_kernel<SF, LF, CR, E, RPH>), gr, bl, 0, st, a);       \
        return hipGetLastError();
        COLA_DIRS(EPI_NONE)
        COLA_DIRS(EPI_XPAY)
        COLA_DIRS(EPI_CLOV)
        COLA_DIRS(EPI_CLOV_XPAY)
        COLA_DIRS(EPI_XPAY_CLOV)
        COLA_DIRS(EPI_XPAY_CG)
        COLA_DIRS(EPI_CLOV_XPAY_CG)
#undef COLA_DIRS
    }
    return hipErrorInvalidValue;
}

template <SpinorFmt SF, LinkFmt LF, typename CR>
hipError_t hop_dirs_launch(const HopArgs &a, int grid, hipStream_t st) {
    // one block per sites_per_block sites (of each parity), whole sites of at most 64 lanes
    const long per = ((long)a.g.Vh + a.sites_per_block - 1) / a.sites_per_block;
    if (a.sites_per_block < 1 || a.sites_per_block * a.nrhs > kDirsSites ||
        grid != (a.both ? 2 : 1) * per)
        return hipErrorInvalidValue;
    bool real_phase = true;
    for (int mu = 0; mu < 4; ++mu) real_phase &= a.phase[mu].y == 0.0;
    if (real_phase) return hop_dirs_launch_epi<SF, LF, CR, true>(a, grid, st);
    return hop_dirs_launch_epi<SF, LF, CR, false>(a, grid, st);
}

}  // namespace cola
