// Canonical complex128 <-> packed per-parity structure-of-arrays conversion
// for gauge links and spinors, and the SU(3) check that guards the 12-real
// link formats.
#include "device.h"
#include "launch.h"

namespace cola {

namespace {

__device__ __forceinline__ void lex_coords(const Geom &g, uint32_t s, int x[4]) {
    x[0] = (int)(s % (uint32_t)g.L[0]);
    s /= (uint32_t)g.L[0];
    x[1] = (int)(s % (uint32_t)g.L[1]);
    s /= (uint32_t)g.L[1];
    x[2] = (int)(s % (uint32_t)g.L[2]);
    x[3] = (int)(s / (uint32_t)g.L[2]);
}

template <typename T>
__device__ __forceinline__ T to_real(double v) {
    return (T)v;
}

// PACKED: U is a packed 18-real field (consecutive lanes then take consecutive sites of one
// direction), else canonical.
template <bool PACKED>
__global__ void pack_gauge_kernel(const Geom g, const cpx<double> *__restrict__ U, void *g64_18,
                                  void *g64_12, void *g32_12, void *g16_12,
                                  unsigned long long *maxdev) {
    const uint32_t V = 2u * (uint32_t)g.Vh;
    double dev = 0.0;
    for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < V * 4u;
         t += gridDim.x * blockDim.x) {
        int mu, p;
        uint32_t i;
        cpx<double> m[9];
        if constexpr (PACKED) {
            const uint32_t a = t / (uint32_t)g.Vh;
            i = t - a * (uint32_t)g.Vh;
            p = (int)(a >> 2);
            mu = (int)(a & 3u);
            const cpx<double> *u = U + (size_t)a * 9 * (size_t)g.S + i;
#pragma unroll
            for (int k = 0; k < 9; ++k) m[k] = u[(size_t)k * (size_t)g.S];
        } else {
            const uint32_t s = t >> 2;
            mu = (int)(t & 3u);
            int x[4];
            lex_coords(g, s, x);
            p = (x[0] + x[1] + x[2] + x[3]) & 1;
            i = s >> 1;  // Lx even: checkerboard index
            const cpx<double> *u = U + (size_t)t * 9;
#pragma unroll
            for (int k = 0; k < 9; ++k) m[k] = u[k];
        }
        // SU(3) deviation: |U U^H - 1| and |det U - 1|
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                cpx<double> sacc = {0.0, 0.0};
#pragma unroll
                for (int k = 0; k < 3; ++k) sacc = cmadd(sacc, m[a * 3 + k], cpx<double>{m[b * 3 + k].x, -m[b * 3 + k].y});
                const double re = sacc.x - (a == b ? 1.0 : 0.0);
                dev = fmax(dev, fmax(fabs(re), fabs(sacc.y)));
            }
        const cpx<double> c0 = cmul(m[4], m[8]) - cmul(m[5], m[7]);
        const cpx<double> c1 = cmul(m[5], m[6]) - cmul(m[3], m[8]);
        const cpx<double> c2 = cmul(m[3], m[7]) - cmul(m[4], m[6]);
        cpx<double> det = cmul(m[0], c0);
        det = cmadd(det, m[1], c1);
        det = cmadd(det, m[2], c2);
        dev = fmax(dev, fmax(fabs(det.x - 1.0), fabs(det.y)));
        if (!(dev <= 1e300)) dev = 1e300;  // NaN / Inf
        const size_t S = (size_t)g.S;
        if (g64_18) {
            cpx<double> *o = (cpx<double> *)g64_18 + ((size_t)(p * 4 + mu) * 9) * S + i;
#pragma unroll
            for (int k = 0; k < 9; ++k) o[k * S] = m[k];
        }
        if (g64_12) {
            cpx<double> *o = (cpx<double> *)g64_12 + ((size_t)(p * 4 + mu) * 6) * S + i;
#pragma unroll
            for (int k = 0; k < 6; ++k) o[k * S] = m[k];
        }
        if (g32_12) {
            float4 *o = (float4 *)g32_12 + ((size_t)(p * 4 + mu) * 3) * S + i;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                o[k * S] = make_float4((float)m[2 * k].x, (float)m[2 * k].y, (float)m[2 * k + 1].x,
                                       (float)m[2 * k + 1].y);
        }
        if (g16_12) {
            struct alignas(8) h4 { _Float16 a, b, c, d; };
            h4 *o = (h4 *)g16_12 + ((size_t)(p * 4 + mu) * 3) * S + i;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                h4 v;
                v.a = (_Float16)m[2 * k].x;
                v.b = (_Float16)m[2 * k].y;
                v.c = (_Float16)m[2 * k + 1].x;
                v.d = (_Float16)m[2 * k + 1].y;
                o[k * S] = v;
            }
        }
    }
    // block max, then one atomic max on the (monotone for dev >= 0) bit pattern
    __shared__ double red[256];
    red[threadIdx.x] = dev;
    __syncthreads();
    for (int w = blockDim.x >> 1; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0)
        atomicMax(maxdev, (unsigned long long)__double_as_longlong(red[0]));
}

// Canonical complex128 [nrhs][V][4][3] <-> packed, ns consecutive checkerboard sites of one
// parity and all rhs per block.  The canonical side moves a site's 192 bytes in
// consecutive lanes, the packed side (rhs innermost) consecutive (site, rhs), and the
// spinors change layout in LDS.  Packing also clears the padding sites behind Vh;
// unpacking leaves the sites of the other parity untouched.  Bound by memory.  With one
// lane per (site, rhs) on both sides every canonical access touched a cache line per lane,
// a lane-varying parity made the packed accesses loop over descriptors, and a fill of the
// whole field went before: 20 x 18 x 14 x 30, 5 rhs, FP32 50 us (and 22 us of fills) to pack, 78 us
// to unpack; now 52 and 40 us (145 MB canonical, 75 MB packed).
constexpr int kSpinorLanes = 256;              // most (site, rhs) of a block
constexpr int kSpinorBatch = 6;                // canonical loads of a lane in flight
constexpr int kSpinorPitch = 13;               // elements per (site, rhs) in LDS: no bank conflicts

struct SpinorTiles {
    int ns, nblk;
    uint32_t tiles;   // per parity block
    FastDiv run, rhs; // ns * 12, nrhs
};

template <SpinorFmt F, bool PACK>
__global__ void __launch_bounds__(kSpinorLanes)
    spinor_layout_kernel(const Geom g, const SpinorTiles ts, void *packed, cpx<double> *canon,
                         int nrhs, int parity, size_t block_bytes) {
    using R = typename SpinorT<F>::real;
    __shared__ cpx<R> m[kSpinorLanes * kSpinorPitch];
    __shared__ uint32_t site[kSpinorLanes];
    const uint32_t V = 2u * (uint32_t)g.Vh, lanes = (uint32_t)(ts.ns * nrhs), tid = threadIdx.x;
    const uint32_t total = ts.tiles * (uint32_t)ts.nblk;
    for (uint32_t b = blockIdx.x; b < total; b += gridDim.x) {
        // both parities of a site range in turn: they share cache lines of the canonical field
        const uint32_t tile = ts.nblk == 2 ? b >> 1 : b, blk = ts.nblk == 2 ? b & 1u : 0u;
        const int p = parity >= 0 ? parity : (int)blk;
        const uint32_t i0 = tile * (uint32_t)ts.ns;
        if (tid < (uint32_t)ts.ns) {
            int x[4];
            const uint32_t i = i0 + tid;
            site_coords(g, i, p, x);
            site[tid] = i < (uint32_t)g.Vh
                            ? (uint32_t)x[0] + (uint32_t)g.L[0] *
                                                   ((uint32_t)x[1] + (uint32_t)g.L[1] *
                                                    ((uint32_t)x[2] + (uint32_t)g.L[2] * (uint32_t)x[3]))
                            : 0xffffffffu;
        }
        const SpinorBlock<F> pk((char *)packed + blk * block_bytes, g.S, nrhs);
        const uint32_t il = fdiv(tid, ts.rhs), r = tid - il * (uint32_t)nrhs;
        const bool own = tid < lanes && i0 + il < (uint32_t)(PACK ? g.S : g.Vh);
        cpx<R> v[12];
        if constexpr (!PACK) {
            if (own) {
                pk.load(i0 + il, r, v);
#pragma unroll
                for (int c = 0; c < 12; ++c) m[tid * kSpinorPitch + c] = v[c];
            }
        }
        __syncthreads();
        // unit u of the canonical side: rhs u / (12 ns), site and component in order
#pragma unroll
        for (int k0 = 0; k0 < 12; k0 += kSpinorBatch) {
            cpx<double> w[kSpinorBatch];
            uint32_t at[kSpinorBatch];
#pragma unroll
            for (int k = 0; k < kSpinorBatch; ++k) {
                const uint32_t u = (uint32_t)((k0 + k) * kSpinorLanes) + tid;
                if (u >= lanes * 12u) continue;
                const uint32_t q = fdiv(u, ts.run), e = u - q * ts.run.d, l = e / 12u, c = e - l * 12u;
                at[k] = (l * (uint32_t)nrhs + q) * kSpinorPitch + c;
                const uint32_t sl = site[l];
                cpx<double> *const o = canon + ((size_t)q * V + sl) * 12 + c;
                if constexpr (PACK) {
                    w[k] = {0.0, 0.0};
                    if (sl != 0xffffffffu) w[k] = *o;
                } else {
                    const cpx<R> d = m[at[k]];
                    if (sl != 0xffffffffu) *o = {(double)d.x, (double)d.y};
                }
            }
            if constexpr (PACK) {
#pragma unroll
                for (int k = 0; k < kSpinorBatch; ++k)
                    if ((uint32_t)((k0 + k) * kSpinorLanes) + tid < lanes * 12u)
                        m[at[k]] = {(R)w[k].x, (R)w[k].y};
            }
        }
        if constexpr (PACK) {
            __syncthreads();
            if (own) {
#pragma unroll
                for (int c = 0; c < 12; ++c) v[c] = m[tid * kSpinorPitch + c];
                pk.store(i0 + il, r, v);
            }
        }
        __syncthreads();  // m and site are reused by the next pass
    }
}

int grid_for(size_t work, int block) {
    size_t g = (work + block - 1) / block;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

size_t spinor_block_bytes(const Geom &g, SpinorFmt f, int nrhs) {
    const size_t SR = (size_t)g.S * nrhs;
    switch (f) {
        case SpinorFmt::F64: return 12 * SR * 16;
        case SpinorFmt::F32: return 12 * SR * 8;
        default: return 12 * SR * 4 + SR * 4;
    }
}

}  // namespace

hipError_t launch_pack_gauge(const Geom &g, const void *U, bool packed, void *g64_18,
                             void *g64_12, void *g32_12, void *g16_12,
                             unsigned long long *maxdev, hipStream_t st) {
    const size_t work = (size_t)g.Vh * 2 * 4;
    const auto kernel = packed ? pack_gauge_kernel<true> : pack_gauge_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(grid_for(work, 256)), dim3(256), 0, st, g,
                       (const cpx<double> *)U, g64_18, g64_12, g32_12, g16_12, maxdev);
    return hipGetLastError();
}

namespace {

template <bool PACK>
hipError_t layout_spinor(const Geom &g, SpinorFmt f, void *packed, void *canon, int nrhs,
                         int parity, hipStream_t st) {
    if (nrhs < 1 || nrhs > kRedMaxWidth) return hipErrorInvalidValue;
    const size_t bb = spinor_block_bytes(g, f, nrhs);
    SpinorTiles ts{};
    ts.ns = kSpinorLanes / nrhs;
    ts.nblk = parity >= 0 ? 1 : 2;
    ts.tiles = (uint32_t)(((PACK ? g.S : g.Vh) + ts.ns - 1) / ts.ns);
    ts.run = make_fastdiv((uint32_t)(ts.ns * 12));
    ts.rhs = make_fastdiv((uint32_t)nrhs);
    const size_t blocks = (size_t)ts.tiles * ts.nblk;
    const dim3 gr((unsigned)(blocks > 65536 ? 65536 : blocks)), bl(kSpinorLanes);
    cpx<double> *c = (cpx<double> *)canon;
    switch (f) {
        case SpinorFmt::F64: hipLaunchKernelGGL((spinor_layout_kernel<SpinorFmt::F64, PACK>), gr, bl, 0, st, g, ts, packed, c, nrhs, parity, bb); break;
        case SpinorFmt::F32: hipLaunchKernelGGL((spinor_layout_kernel<SpinorFmt::F32, PACK>), gr, bl, 0, st, g, ts, packed, c, nrhs, parity, bb); break;
        case SpinorFmt::F16: hipLaunchKernelGGL((spinor_layout_kernel<SpinorFmt::F16, PACK>), gr, bl, 0, st, g, ts, packed, c, nrhs, parity, bb); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_pack_spinor(const Geom &g, SpinorFmt f, void *dst, const void *src, int nrhs,
                              int parity, hipStream_t st) {
    return layout_spinor<true>(g, f, dst, const_cast<void *>(src), nrhs, parity, st);
}

hipError_t launch_unpack_spinor(const Geom &g, SpinorFmt f, void *dst, const void *src, int nrhs,
                                int parity, hipStream_t st) {
    return layout_spinor<false>(g, f, const_cast<void *>(src), dst, nrhs, parity, st);
}

}  // namespace cola
