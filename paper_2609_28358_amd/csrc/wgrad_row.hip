// wgrad_row.hip -- a5 for 3-wide kernels with batch block 32: the kernel-row
// weight-gradient tile (wgrad_row.h), its launch planning and dispatch.
#include "mx_internal.h"

namespace mxc {

#include "wgrad_row.h"

namespace {

// Operand slots in flight (steps): as many as the registers beside the
// accumulators hold without scratch memory; deeper rings measured no faster.
template <int FA, int FB, int NB>
constexpr int wr_depth() { return NB == 2 && (FA == MXC_E4M3 || fmt_bits(FB) == 6) ? 3 : 4; }

template <int FA, int FB, int NB, int S>
__global__ __launch_bounds__(WRT, NB == 2 ? 1 : 2) void wgrad_row_kernel(WRArgs p) {
    __shared__ float red[4][32 * NB * 32 * NB];
    wgrad_row_tile<FA, FB, NB, S, wr_depth<FA, FB, NB>()>(p, blockIdx.x, gridDim.x, red);
}

// The column strides each tile side is built for: FP4 / FP6 take 64 x 64 tiles
// at column stride 1 only.
template <int FA, int FB>
int wr_launch(const WRArgs& a, int nb, int sw, dim3 gd, hipStream_t s) {
    if (nb == 1 && sw == 1)      hipLaunchKernelGGL((wgrad_row_kernel<FA, FB, 1, 1>), gd, dim3(WRT), 0, s, a);
    else if (nb == 1 && sw == 2) hipLaunchKernelGGL((wgrad_row_kernel<FA, FB, 1, 2>), gd, dim3(WRT), 0, s, a);
    else if (nb == 2 && sw == 1) hipLaunchKernelGGL((wgrad_row_kernel<FA, FB, 2, 1>), gd, dim3(WRT), 0, s, a);
    else if constexpr (FA == MXC_E4M3) {
        if (nb != 2 || sw != 2) return MXC_ERR_ARG;
        hipLaunchKernelGGL((wgrad_row_kernel<FA, FB, 2, 2>), gd, dim3(WRT), 0, s, a);
    } else {
        return MXC_ERR_ARG;
    }
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_HIP;
}

}  // namespace

// Tile shape and splits of the kernel-row weight gradient; false when the
// layer is outside it or better off with the 64 x 64 tile of one tap
// (wgrad_tile.h).  Measured for the whole gradient, reduction included:
//   one channel block on each side: always (stem at batch 32 59 -> 37 us,
//     16 -> 16 channels at 160 x 160, batch 64, 37 -> 22 us);
//   FP8: always, the decoded window saves two of three decodes; 64 x 64 tiles
//     where a wave walks at least 12 columns (256 -> 256 at 16 x 16, batch 128,
//     89 -> 53 us), else 32 x 32 ones (64 -> 64 at 56 x 56, batch 32, 27 -> 19);
//   64 x 64 tiles only where their grid takes nearly every CU, or a wave walks
//     at least 64 columns: with 192 workgroups (512 channels on a side) 32 x 32
//     ones are faster, and share a launch with the input gradient (MXFP8
//     512 -> 256 at 14x14, batch 32: 37 -> 26 us alone, 59 -> 47 with it; MXFP4
//     512 -> 512 at 10x10, batch 64: 32 -> 22 and 58 -> 40; MXFP8 512 -> 256 at
//     40x40, batch 32, 100 columns a wave: 64 x 64 ones win, 118 against 130);
//   FP4 / FP6 on more blocks: 64 x 64 tiles where a wave walks enough columns
//     to cover the larger epilogue, column stride 1 (256 -> 256 as above 40 ->
//     34; FP6 128 -> 128 at 40 x 40, batch 64, 33 -> 29); FP4 needs more of
//     them, since its one-tap tiles share a launch with the input gradient
//     (128 -> 128 at 40 x 40: 29 -> 27 alone, but 44 -> 47 us with it);
//     32 x 32 tiles where there are few columns in all (128 -> 256, stride 2,
//     at 28 x 28, batch 32: 17 -> 14), a one-tap tile's wave having hardly
//     any to walk.
bool wgrad_row_plan(const Conv& cv, WRPlan& q) {
    if (cv.x.bn != 32 || cv.kw != 3 || (cv.sw != 1 && cv.sw != 2)) return false;
    // 32-bit buffer offsets: codes below 2 GiB per launch.  A larger layer of one
    // channel block on each side takes its batch groups in several launches (3 ->
    // 16 at 640x640, batch 192, MXFP8: 807 us in one-tap tiles, 369 so); the others
    // have one-tap tiles for that size.
    const long gb = (long)cv.ho * cv.wo * cv.gy.cp * 4 * fmt_bits(cv.fa);    // of one group
    const long xb = (long)cv.h * cv.w * cv.x.cp * 4 * fmt_bits(cv.fb);
    const long fit = 0x7FFFFF00L / std::max(gb, xb);
    if (fit == 0) return false;
    // a row that does not exist is walked from WR_OOB on; its last column must
    // lie below 2^32 too (rows of many channels under wide padding reach past it)
    const long step = std::max((long)cv.gy.cp * 4 * fmt_bits(cv.fa), (long)cv.sw * cv.x.cp * 4 * fmt_bits(cv.fb));
    if ((cv.wo + 3) * step >= 0x7FFFF000L) return false;
    q.launches = (int)((cv.x.ng + fit - 1) / fit);
    q.groups = (cv.x.ng + q.launches - 1) / q.launches;
    if (q.launches > 1 && (cv.gy.ncb > 1 || cv.x.ncb > 1)) return false;
    q.nrp = (q.groups * cv.ho + 1) / 2;
    const long total = (long)q.nrp * cv.wo;                           // columns of a launch's row pairs
    const long part = (long)cv.gy.cp * cv.kh * 3 * cv.x.cp * 4;       // bytes of one partial result
    auto tiles = [&](int n) { return (long)cv.kh * ((cv.gy.ncb + n - 1) / n) * ((cv.x.ncb + n - 1) / n); };
    // one workgroup per CU on 64 x 64 tiles (a wave per SIMD by their
    // registers), two on 32 x 32 ones; a wave walks at least 6 columns; the
    // partial results stay within 16 MiB
    auto split = [&](int n) {
        return std::max(1L, std::min({(n == 2 ? 256 : 512) / tiles(n), total / (4 * 6), (16L << 20) / part / q.launches}));
    };
    q.nb = 1;
    if (cv.gy.ncb > 1 || cv.x.ncb > 1) {
        const long cols = cv.gy.ncb > 1 && cv.x.ncb > 1 ? total / (4 * split(2)) : 0;
        const bool fills = split(2) * tiles(2) >= 224 || cols >= 64;
        if (cv.fa == MXC_E4M3) q.nb = cols >= 12 && fills ? 2 : 1;
        else if (cv.sw == 1 && cols >= (fmt_bits(cv.fb) == 6 ? 16 : 24)) q.nb = fills ? 2 : 1;
        else if (total > 128) return false;
    }
    const long nt = tiles(q.nb);
    if (nt > 0x7FFFFFL) return false;
    q.ntiles = (int)nt;
    q.per = (int)split(q.nb);
    if ((long)q.per * q.launches > std::max(1L, (16L << 20) / part)) return false;
    q.splits = q.per * q.launches;
    return true;
}

int wgrad_row_splits(const Conv& cv) {
    WRPlan q;
    return wgrad_row_plan(cv, q) ? q.splits : 0;
}

int launch_wgrad_row(const Conv& cv, const void* gc, const uint8_t* gs, const void* xc, const uint8_t* xs, float* dst,
                     hipStream_t s) {
    WRPlan q;
    if (!wgrad_row_plan(cv, q)) return MXC_ERR_SHAPE;
    Conv part = cv;                                        // the batch groups of one launch
    for (int g0 = 0; g0 < cv.x.ng; g0 += q.groups) {
        const int l = g0 / q.groups;
        const size_t gpix = (size_t)g0 * cv.ho * cv.wo, xpix = (size_t)g0 * cv.h * cv.w;
        part.x.ng = part.gy.ng = std::min(q.groups, cv.x.ng - g0);
        WRArgs a;
        const dim3 gd((unsigned)wgrad_row_fill(part, q, (const uint8_t*)gc + gpix * cv.gy.cp * 4 * fmt_bits(cv.fa),
                                               gs + gpix * cv.gy.ncb, (const uint8_t*)xc + xpix * cv.x.cp * 4 * fmt_bits(cv.fb),
                                               xs + xpix * cv.x.ncb,
                                               dst + (size_t)l * q.per * cv.gy.cp * cv.kh * 3 * cv.x.cp, a));
        int rc = MXC_ERR_ARG;
        if (cv.fa == MXC_E4M3 && cv.fb == MXC_E4M3)      rc = wr_launch<MXC_E4M3, MXC_E4M3>(a, q.nb, cv.sw, gd, s);
        else if (cv.fa == MXC_E2M1 && cv.fb == MXC_E2M1) rc = wr_launch<MXC_E2M1, MXC_E2M1>(a, q.nb, cv.sw, gd, s);
        else if (cv.fa == MXC_E2M3 && cv.fb == MXC_E2M3) rc = wr_launch<MXC_E2M3, MXC_E2M3>(a, q.nb, cv.sw, gd, s);
        else if (cv.fa == MXC_E2M1 && cv.fb == MXC_E3M2) rc = wr_launch<MXC_E2M1, MXC_E3M2>(a, q.nb, cv.sw, gd, s);
        if (rc) return rc;
    }
    return MXC_OK;
}

}  // namespace mxc
