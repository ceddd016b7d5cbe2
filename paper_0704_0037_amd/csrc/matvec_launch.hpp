// Host side of the interaction-matrix product: picks, for each axis, the kernels specialized for
// its padded length when one exists (index arithmetic folds to constants) or the general ones.
// Included by one translation unit per precision.
#pragma once

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <utility>

#include "ctx.hpp"
#include "matvec_kernels.hpp"
#include "zcol.hpp"


namespace dda {

template <typename R> inline const cplx<R> *tw_of(const Ctx &c);
template <> inline const double2 *tw_of<double>(const Ctx &c) { return c.tw64; }
template <> inline const float2 *tw_of<float>(const Ctx &c) { return c.tw32; }
template <typename R> inline const cplx<R> *ghat_of(const Ctx &c);
template <> inline const double2 *ghat_of<double>(const Ctx &c) { return c.ghat; }
template <> inline const float2 *ghat_of<float>(const Ctx &c) { return c.ghat32; }

// blocks above 64 KiB of dynamic LDS must be allowed explicitly.  The attribute is the kernel's limit and
// stays as it was set last, while one kernel runs with several sizes (the column kernel's follow the grid
// and the number of vectors), so it is only ever raised: once per kernel, device and larger size, and
// launches recorded into a graph after an eager one of the same size make no attribute calls.
template <class K> inline void allow_lds(K kernel, size_t bytes) {
    if (bytes <= 64 * 1024) return;
    static std::mutex mu;
    static std::map<std::pair<const void *, int>, size_t> allowed;
    int dev = 0;
    (void)hipGetDevice(&dev);
    const void *f = reinterpret_cast<const void *>(kernel);
    std::lock_guard<std::mutex> lock(mu);
    size_t &most = allowed[{f, dev}];
    if (bytes <= most) return;
    most = bytes;
    (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// LAUNCH(L) for a length with specialized kernels, LAUNCH(0) (planned at run time) for the others
#define DDA_DISPATCH(LEN, LAUNCH)                     \
    switch (LEN) {                                    \
        DDA_SPECIALIZED_LENGTHS(DDA_CASE_##LAUNCH)    \
        default: LAUNCH(0) break;                     \
    }
#define DDA_CASE_fwd_x(L) case L: fwd_x(L) break;
#define DDA_CASE_fwd_y(L) case L: fwd_y(L) break;
#define DDA_CASE_inv_y(L) case L: inv_y(L) break;
#define DDA_CASE_inv_x(L) case L: inv_x(L) break;
#define DDA_CASE_zcol(L) case L: zcol_launch<R, L>(c, w.B2, gh, nrhs, tw, s, done); break;

// Block shape of the column kernel: up to four waves over opb octant columns, which take
// ceil(4 nrhs opb / (W CPW)) rounds.  The smallest opb whose estimate is not beaten by 10 %: turns of
// the grid over the resident blocks, times rounds (a tenth for staging the tensor), times a factor
// for the waves that share a compute unit.  A wave of 3, 5 or 7 columns needs several octant
// columns to fill its rounds (L = 160, one vector: opb 1, 3: 96, 75 us; L = 96: opb 1, 5: 28,
// 22 us), and small grids run faster with one block per compute unit.
struct ZShape {
    int W, opb;
};
template <typename R, int LC> inline ZShape zcol_shape(int noct, int nrhs) {
    using Z = ZCol<LC>;
    constexpr int kCUs = 256, kWaves = 4 * zcol_waves_per_simd<R>(LC);
    ZShape best{1, 1};
    double cost = 1e300;
    for (int opb = 1; opb <= 8; ++opb) {
        const int64_t items = (int64_t)4 * nrhs * opb;
        const int W = items > 2 * Z::CPW ? 4 : items > Z::CPW ? 2 : 1;
        const size_t lds = zcol_lds<R, LC>(opb, W);
        if (opb > 1 && lds > 80 * 1024) break;
        const int per_cu = std::min<int>(160 * 1024 / (int)lds, kWaves / W);
        const int64_t rounds = (items + W * Z::CPW - 1) / (W * Z::CPW), blocks = (noct + opb - 1) / opb;
        const int resident = W * (int)std::min<int64_t>(per_cu, (blocks + kCUs - 1) / kCUs);
        const double turns = (double)blocks / (kCUs * per_cu);
        const double t = (turns < 4 ? std::ceil(turns) : turns) * (rounds + 0.1) * (8 + resident);
        if (t < 0.9 * cost) {
            cost = t;
            best = {W, opb};
        }
    }
    return best;
}

template <typename R, int LC>
inline void zcol_launch(const Ctx &c, cplx<R> *B2, const cplx<R> *gh, int nrhs, const cplx<R> *tw, hipStream_t s,
                        const int *done) {
    const int noct = (c.Lx / 2 + 1) * (c.Ly / 2 + 1);
    const ZShape z = zcol_shape<R, LC>(noct, nrhs);
    const size_t lds = zcol_lds<R, LC>(z.opb, z.W);
    const int blocks = (noct + z.opb - 1) / z.opb;
    allow_lds(&k_zcol<R, LC>, lds);
    hipLaunchKernelGGL((k_zcol<R, LC>), dim3((blocks + 7) / 8 * 8), dim3(64 * z.W), lds, s, B2, gh, c.nz, c.Lx, c.Ly,
                       nrhs, z.opb, tw + c.pzf.tw_off, done);
}

// Transforms in precision R on the work buffers of precision R (the context's, or the
// intermediates B1 / B2 of `wk` when given); x, y, scale and dots in RX.  EXT: leave out the lines
// outside the planes' ranges of y.
template <typename R, typename RX, bool EXT>
dda_status matvec_passes(Ctx &c, const cplx<RX> *x, cplx<RX> *y, int nrhs, const cplx<RX> *scale, cplx<RX> *dots,
                         hipStream_t s, const int *done, hipEvent_t *ev, const Work<R> &w) {
    using C = cplx<R>;
    const C *tw = tw_of<R>(c);
    const C *gh = ghat_of<R>(c);
    const int ncomp = 3 * nrhs;
    const Tiles &tl = tiles_of<R>(c);
    const int nlx = tl.nl_x, nly = tl.nl_y;
    const int ytiles = (c.ny + nlx - 1) / nlx, ztiles = (c.nz + nly - 1) / nly;
    const size_t lx_bytes = (size_t)nlx * lds_line_stride(c.Lx) * sizeof(C);
    const size_t ly_bytes = (size_t)nly * lds_line_stride(c.Ly) * sizeof(C);
    const size_t lz_bytes = zmul_lds_elems(c.Lz) * sizeof(C);
    const int N = (int)c.N;
    const int2 *ext = c.rows + (size_t)c.ny * c.nz;
    const dim3 xg(ncomp * c.nz * ytiles), yg(ncomp * c.Lx * ztiles);
    if (ev) DDA_HIP_CHECK(hipEventRecord(ev[0], s));
#define fwd_x(L)                                                                                                     \
    allow_lds(&k_fwd_x<R, L, RX, EXT>, lx_bytes);                                                                    \
    hipLaunchKernelGGL((k_fwd_x<R, L, RX, EXT>), xg, dim3(nlx * c.pxf.tpl), lx_bytes, s, c.gmap, c.rows, ext,        \
                       c.gmap_stride, c.rows_stride, x, w.B1, c.nx, c.ny, c.nz, N, c.pxf, tw, tl.lnl_x, done);
    DDA_DISPATCH(c.Lx, fwd_x)
#undef fwd_x
    if (ev) DDA_HIP_CHECK(hipEventRecord(ev[1], s));
#define fwd_y(L)                                                                                                     \
    allow_lds(&k_fwd_y<R, L, EXT>, ly_bytes);                                                                        \
    hipLaunchKernelGGL((k_fwd_y<R, L, EXT>), yg, dim3(nly * c.pyf.tpl), ly_bytes, s, ext, c.rows_stride, w.B1, w.B2, \
                       c.ny, c.nz, c.Lx, ncomp, c.pyf, tw, tl.lnl_y, done);
    DDA_DISPATCH(c.Ly, fwd_y)
#undef fwd_y
    if (ev) DDA_HIP_CHECK(hipEventRecord(ev[2], s));
    const int zblocks = (c.Lx / 2 + 1) * (c.Ly / 2 + 1);  // one block per octant column
    switch (c.Lz) {
        DDA_SPECIALIZED_LENGTHS(DDA_CASE_zcol)
        default:
            allow_lds(&k_zmul<R>, lz_bytes);
            hipLaunchKernelGGL(k_zmul<R>, dim3((zblocks + 7) / 8 * 8), dim3(3 * zmul_ct(c.pzf)), lz_bytes, s, w.B2, gh,
                               c.nz, c.Lx, c.Ly, nrhs, c.pzf, c.pzi, tw, done);
            break;
    }
    if (ev) DDA_HIP_CHECK(hipEventRecord(ev[3], s));
#define inv_y(L)                                                                                                     \
    allow_lds(&k_inv_y<R, L, EXT>, ly_bytes);                                                                        \
    hipLaunchKernelGGL((k_inv_y<R, L, EXT>), yg, dim3(nly * c.pyi.tpl), ly_bytes, s, ext, c.rows_stride, w.B2, w.B1, \
                       c.ny, c.nz, c.Lx, ncomp, c.pyi, tw, tl.lnl_y, done);
    DDA_DISPATCH(c.Ly, inv_y)
#undef inv_y
    if (ev) DDA_HIP_CHECK(hipEventRecord(ev[4], s));
#define inv_x(L)                                                                                                     \
    allow_lds(&k_inv_x<R, L, RX, EXT>, lx_bytes);                                                                    \
    hipLaunchKernelGGL((k_inv_x<R, L, RX, EXT>), xg, dim3(nlx * c.pxi.tpl), lx_bytes, s, c.gmap, c.rows, ext,        \
                       c.gmap_stride, c.rows_stride, w.B1, x, y, c.nx, c.ny, c.nz, N, c.pxi, tw, tl.lnl_x, scale,    \
                       dots, done);
    DDA_DISPATCH(c.Lx, inv_x)
#undef inv_x
    if (ev) DDA_HIP_CHECK(hipEventRecord(ev[5], s));
    DDA_HIP_CHECK(hipGetLastError());
    return DDA_OK;
}

// Lines (y, z) outside a plane's range of y are zero before the x pass and unused after it.  From 256 MB
// of B1 on, the size of the last-level cache, they are left out of the x passes and of B1.  A sphere
// leaves out 21 %: x passes 757 + 980 -> 677 + 896 us, y 1708 + 1670 -> 1622 + 1592 (256^3, two vectors);
// 128^3, two vectors, 403 MB: 1166 -> 1150 us in all; a solve of a 64 x 64 x 64 grid's ellipsoid for 16
// beams (402 MB) 50.0 -> 45.6 ms.  Below, the range is one more load before the
// others: 48^3 72.3 -> 73.5, 160^3 in single precision (197 MB) 752 -> 759.
template <typename R, typename RX = R>
dda_status matvec_device_impl(Ctx &c, const cplx<RX> *x, cplx<RX> *y, int nrhs, const cplx<RX> *scale,
                              cplx<RX> *dots, hipStream_t s, const int *done, hipEvent_t *ev,
                              const Work<R> *wk = nullptr) {
    const Work<R> &w = wk ? *wk : work_of<R>(c);
    const size_t b1_bytes = (size_t)3 * nrhs * c.nz * c.Lx * row_pitch(c.ny) * sizeof(cplx<R>);
    return b1_bytes >= ((size_t)256 << 20)
               ? matvec_passes<R, RX, true>(c, x, y, nrhs, scale, dots, s, done, ev, w)
               : matvec_passes<R, RX, false>(c, x, y, nrhs, scale, dots, s, done, ev, w);
}

}  // namespace dda
