// conv_lean_bwd.hip -- a layer's input gradient and batch-block-32 weight
// gradient in one launch (conv_lean_bwd_kernel, conv_lean_kern.h).
#include "conv_lean_kern.h"

namespace mxc {

namespace {

struct WArgs {                // the weight gradient's arguments, by its tile
    WLArgs l;
    WRArgs r;
};

template <int F, int KW, int PW, bool DG2, int NB, int NRB = 2, bool KR = false>
int bwd_launch(const LeanArgs& a, const WArgs& w, int nl, bool dgf, int grid, size_t lds, hipStream_t s) {
    const BwdWArgs<KW, NB>* q;
    if constexpr (KW == 3 && NB == 1) q = &w.r;
    else                              q = &w.l;
    static std::atomic<uint64_t> devs{0};
    if (raise_lds(conv_lean_bwd_kernel<F, KW, PW, DG2, NB, NRB, KR>, devs, lds)) return MXC_ERR_HIP;
    hipLaunchKernelGGL((conv_lean_bwd_kernel<F, KW, PW, DG2, NB, NRB, KR>), dim3(grid), dim3(LT), lds, s, a, *q, nl, dgf ? 1 : 0);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_HIP;
}

template <int F, int NB>
int bwd_launch_nb(const LeanArgs& a, const WArgs& q, int nl, bool dgf, int grid, size_t lds, bool dg2, int kw, int pw, bool kr,
                  hipStream_t s) {
    if constexpr (F == MXC_E2M1) {
        if (pw == NARROW_PW) {
            if (kw == 3 && kr)
                return dg2 ? bwd_launch<F, 3, NARROW_PW, true, NB, 1, true>(a, q, nl, dgf, grid, lds, s)
                           : bwd_launch<F, 3, NARROW_PW, false, NB, 1, true>(a, q, nl, dgf, grid, lds, s);
            if (dg2) return kw == 3 ? bwd_launch<F, 3, NARROW_PW, true, NB, 1>(a, q, nl, dgf, grid, lds, s)
                                    : bwd_launch<F, 1, NARROW_PW, true, NB, 1>(a, q, nl, dgf, grid, lds, s);
            return kw == 3 ? bwd_launch<F, 3, NARROW_PW, false, NB, 1>(a, q, nl, dgf, grid, lds, s)
                           : bwd_launch<F, 1, NARROW_PW, false, NB, 1>(a, q, nl, dgf, grid, lds, s);
        }
    }
    if (dg2) {
        if (kw == 3) return pw == 1 ? bwd_launch<F, 3, 1, true, NB>(a, q, nl, dgf, grid, lds, s) : bwd_launch<F, 3, 2, true, NB>(a, q, nl, dgf, grid, lds, s);
        return pw == 1 ? bwd_launch<F, 1, 1, true, NB>(a, q, nl, dgf, grid, lds, s) : bwd_launch<F, 1, 2, true, NB>(a, q, nl, dgf, grid, lds, s);
    }
    if (kw == 3) return pw == 1 ? bwd_launch<F, 3, 1, false, NB>(a, q, nl, dgf, grid, lds, s) : bwd_launch<F, 3, 2, false, NB>(a, q, nl, dgf, grid, lds, s);
    return pw == 1 ? bwd_launch<F, 1, 1, false, NB>(a, q, nl, dgf, grid, lds, s) : bwd_launch<F, 1, 2, false, NB>(a, q, nl, dgf, grid, lds, s);
}

template <int F>
int bwd_launch_f(const LeanArgs& a, const WArgs& q, int nl, bool dgf, int grid, size_t lds, bool dg2, int kw, int pw, bool kr,
                 bool nb1, hipStream_t s) {
    return nb1 ? bwd_launch_nb<F, 1>(a, q, nl, dgf, grid, lds, dg2, kw, pw, kr, s)
               : bwd_launch_nb<F, 2>(a, q, nl, dgf, grid, lds, dg2, kw, pw, kr, s);
}

}  // namespace

// Input gradient (dcv) and weight gradient (wcv, `splits` ways into wdst) of
// one layer in one launch; returns 1 when the layer or its formats are
// outside the grouped kernel (the caller then launches the two separately).
int launch_lean_bwd(const Conv& dcv, const void* wc, const uint8_t* ws, const void* gc, const uint8_t* gs,
                    float* gx, int layout, const Conv& wcv, const void* xc, const uint8_t* xs, float* wdst,
                    int splits, hipStream_t s) {
    const int f = dcv.fa;
    if ((f != MXC_E4M3 && f != MXC_E2M1) || dcv.fb != f || wcv.fa != f || wcv.fb != f) return 1;
    LeanPlan P;
    const int prc = lean_plan(dcv, true, wc, ws, gc, gs, gx, layout, nullptr, nullptr, nullptr, P);
    if (prc) return prc;
    if (P.rb == 1 && P.pw != NARROW_PW) return 1;        // a narrow shape this kernel is not built for
    WArgs q;
    WRPlan wr;
    const bool row = wgrad_row_plan(wcv, wr);
    if (row && (wr.nb != 1 || wr.launches > 1)) return 1;   // one wave per SIMD, or 2 GiB of codes: launches of its own
    const bool nb1 = row || (wgrad_single_block(wcv) && wcv.kw == 1);
    if (!row && !nb1 && wgrad_single_block(wcv)) return 1;
    const long wg = row ? wgrad_row_fill(wcv, wr, gc, gs, xc, xs, wdst, q.r)
                        : wgrad_lean_fill(wcv, gc, gs, xc, xs, wdst, splits, nullptr, nullptr, q.l);
    if (wg < 0) return MXC_ERR_SHAPE;
    LeanArgs& a = P.a;
    const long nl = ((long)(P.dg2 ? a.pofs[4] : a.ntiles) + 7) / 8 * 8;
    if (nl + wg > 0x7FFFFFFFL) return MXC_ERR_SHAPE;
    // ring depth for the combined grid, every workgroup holding at least the
    // LDS the weight-gradient tile sums its four waves through (64 KB, or
    // 16 KB on 32 x 32 tiles)
    const long red = nb1 ? 16384 : 65536;
    const long per_cu = (nl + wg + 255) / 256;
    int nbuf = 2;
    for (int b = 4; b > 2; b--) {
        const long need = (long)b * a.stage_bytes > red ? (long)b * a.stage_bytes : red;
        if (per_cu * need <= LDS_MAX) { nbuf = b; break; }
    }
    a.nbuf = nbuf;
    const int used = nbuf < P.nstage ? nbuf : P.nstage;
    size_t lds = lean_lds(a, used);
    if (lds < (size_t)red) lds = (size_t)red;
    const int grid = (int)(nl + wg);
    // The longer workgroups are dispatched first: an input-gradient tile runs
    // its taps times G_Y's channel blocks, a wave of the kernel-row tile its
    // columns.  Between the two orders (us, weight gradient first, then last):
    // MXFP8 512 -> 512 at 7x7, batch 32, stride 2, 36 steps against 2: 30 and 21.5;
    // 256 -> 512 at 14x14, stride 2, 36 against 7: 31.7 and 23.6; MXFP4 512 -> 256
    // at 20x20, batch 64, 72 against 100: 49 and 61.  The line lies where they
    // cross, at 2.5 steps a column.  One-tap tiles, whose workgroups are about
    // as long, go first.
    const long steps = (long)dcv.kh * dcv.kw * dcv.gy.ncb;                  // stride 2: a quarter, on average
    const bool dgf = row && 2 * steps >= 5L * q.r.spw * (P.dg2 ? 4 : 1);
    return f == MXC_E4M3 ? bwd_launch_f<MXC_E4M3>(a, q, (int)nl, dgf, grid, lds, P.dg2, dcv.kw, P.pw, P.krow, nb1, s)
                         : bwd_launch_f<MXC_E2M1>(a, q, (int)nl, dgf, grid, lds, P.dg2, dcv.kw, P.pw, P.krow, nb1, s);
}
}  // namespace mxc
