// 3 x 3 complex FP64 matrices, and the links of a packed 18-real field for the kernels that
// work on links (clover blocks, smearing, the trajectory).
//
// Those read the packed field (chunk k of U_mu at (p, i) at ((p 4 + mu) 9 + k) S + i), in
// which the 64 lanes of a wavefront, consecutive checkerboard sites of one parity and one
// direction, load 64 consecutive 16-byte elements.  From the canonical field (144 bytes per
// link) the same load touches 64 cache lines, and the L1's line rate, not memory, set the
// time of these kernels.
#pragma once

#include "device.h"

namespace cola {

struct M3 {
    cpx<double> a[3][3];
};

__device__ __forceinline__ cpx<double> conj(cpx<double> a) { return {a.x, -a.y}; }

// A B, A B^H, A^H B
__device__ __forceinline__ M3 mm(const M3 &A, const M3 &B) {
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> s = cmul(A.a[i][0], B.a[0][j]);
            s = cmadd(s, A.a[i][1], B.a[1][j]);
            r.a[i][j] = cmadd(s, A.a[i][2], B.a[2][j]);
        }
    return r;
}
__device__ __forceinline__ M3 mmd(const M3 &A, const M3 &B) {
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> s = cmul(A.a[i][0], conj(B.a[j][0]));
            s = cmadd(s, A.a[i][1], conj(B.a[j][1]));
            r.a[i][j] = cmadd(s, A.a[i][2], conj(B.a[j][2]));
        }
    return r;
}
__device__ __forceinline__ M3 mdm(const M3 &A, const M3 &B) {
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> s = cmul(conj(A.a[0][i]), B.a[0][j]);
            s = cmadd(s, conj(A.a[1][i]), B.a[1][j]);
            r.a[i][j] = cmadd(s, conj(A.a[2][i]), B.a[2][j]);
        }
    return r;
}
// P <- P B, P <- P B^H, row by row (one row more than P and B in registers)
__device__ __forceinline__ void mul_right(M3 &P, const M3 &B) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        cpx<double> r[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> s = cmul(P.a[i][0], B.a[0][j]);
            s = cmadd(s, P.a[i][1], B.a[1][j]);
            r[j] = cmadd(s, P.a[i][2], B.a[2][j]);
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) P.a[i][j] = r[j];
    }
}
__device__ __forceinline__ void mul_right_dag(M3 &P, const M3 &B) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        cpx<double> r[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<double> s = cmul(P.a[i][0], conj(B.a[j][0]));
            s = cmadd(s, P.a[i][1], conj(B.a[j][1]));
            r[j] = cmadd(s, P.a[i][2], conj(B.a[j][2]));
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) P.a[i][j] = r[j];
    }
}
__device__ __forceinline__ M3 dag(const M3 &A) {
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) r.a[i][j] = conj(A.a[j][i]);
    return r;
}
__device__ __forceinline__ M3 operator+(const M3 &A, const M3 &B) {
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) r.a[i][j] = A.a[i][j] + B.a[i][j];
    return r;
}

// A site of the packed field: parity, coordinates, checkerboard index.
struct Site {
    int p;
    int x[4];
    uint32_t i;
};

__device__ __forceinline__ uint32_t cb_index(const Geom &g, const int x[4]) {
    return (uint32_t)(x[0] >> 1) +
           (uint32_t)g.Lxh * ((uint32_t)x[1] +
                              (uint32_t)g.L[1] * ((uint32_t)x[2] + (uint32_t)g.L[2] * (uint32_t)x[3]));
}

// The q-th site of parity p in tile order.
__device__ __forceinline__ Site tiled_site(const Geom &g, const TileOrder &o, uint32_t q, int p) {
    Site s;
    s.p = p;
    const uint32_t r = fdiv(q, o.cols), col = q - r * o.cols.d;
    const uint32_t tile = fdiv(r, o.lt), t = r - tile * o.lt.d;
    const uint32_t c1 = fdiv(col, o.lxh), xh = col - c1 * o.lxh.d;
    const uint32_t zl = fdiv(c1, o.dty), yl = c1 - zl * o.dty.d;
    const uint32_t tz = fdiv(tile, o.nty), ty = tile - tz * o.nty.d;
    s.x[1] = (int)(ty * o.dty.d + yl);
    s.x[2] = (int)(tz * (uint32_t)o.tz + zl);
    s.x[3] = (int)t;
    s.x[0] = 2 * (int)xh + ((s.x[1] + s.x[2] + s.x[3] + p) & 1);
    s.i = cb_index(g, s.x);
    return s;
}

// The site x + d mu (d = +-1, periodic); mu is the same for all lanes of a wavefront.
__device__ __forceinline__ Site shifted(const Geom &g, const Site &s, int mu, int d) {
    Site r;
    r.p = 1 - s.p;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int v = s.x[k] + (k == mu ? d : 0);
        v = v == g.L[k] ? 0 : v;
        r.x[k] = v < 0 ? g.L[k] - 1 : v;
    }
    r.i = cb_index(g, r.x);
    return r;
}

// U_mu at a site of the packed field; parity and direction are the same for all lanes of a
// wavefront (one buffer descriptor per chunk array, one 32-bit offset per lane)
__device__ __forceinline__ M3 ldp(const cpx<double> *U, int S, const Site &s, int mu) {
    M3 m;
    load_link<LinkFmt::F64_18, double>(U, S, s.p, mu, s.i, m.a);
    return m;
}

// Traceless part of i (W - W^H) / 2 (Hermitian, the trace and diagonal real).
__device__ __forceinline__ M3 traceless_hermitian(const M3 &W) {
    M3 X;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const cpx<double> d = {W.a[i][j].x - W.a[j][i].x, W.a[i][j].y + W.a[j][i].y};
            X.a[i][j] = {-0.5 * d.y, 0.5 * d.x};
        }
    const double tr = (X.a[0][0].x + X.a[1][1].x + X.a[2][2].x) / 3.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) X.a[i][i] = {X.a[i][i].x - tr, 0.0};
    return X;
}

}  // namespace cola
