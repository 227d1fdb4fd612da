// wgrad_row.h -- the weight-gradient tile of 3-wide kernels with batch block
// 32 (a5): all three taps of one kernel row at once, walking along output
// rows so that an X column is loaded once for every tap that reads it.
// Included inside namespace mxc by .hip files only.
#pragma once

namespace {

constexpr int WRT = 256;

struct WRArgs {
    const uint8_t* gc;
    const uint8_t* gs;
    const uint8_t* xc;
    const uint8_t* xs;
    float* dst;
    int direct;                    // 1: dst is G_W (OIHW); 0: partial tiles
    int cout, cin, kh, sh, ph, pw, ho, wo, h, w;
    int gy_ncb, x_ncb, gy_cp, x_cp, ntot;
    uint32_t gbytes, xbytes;       // code bytes of G_Y and X (each below 2^31)
    int nrows, nrp;                // output rows (all batch groups), row pairs: ceil(nrows / 2)
    int cot, cit, ntiles;          // tiles along Cout and Cin, tiles in all (kernel rows x cot x cit)
    int spw;                       // pixel columns (of a row pair) per wave
    int nsplit;
};

// A fragment's registers (N of a row's bits / 4).  A vector, not an array: the
// compiler joined the six words of an E2M3 fragment and the two behind them
// into one 8-word read, which kept a slot of the ring in scratch memory (64
// bytes a lane at column stride 2; MXFP6 32 -> 32 at 10x10, batch 32, stride
// 2: 8.5 -> 7.4 us; 256 -> 256 at 28x28 27.9 -> 21.5).
template <int N> struct WRFrag {
    enum { n = N };
    int d __attribute__((ext_vector_type(N)));
};
template <int N> struct WRCol {
    enum { n = N };
    int d[N];
};
template <typename T> constexpr int wr_words = std::remove_reference_t<T>::n;

// Any offset past the tensor: a buffer load there returns zeros.
constexpr uint32_t WR_OOB = 0x80000000u;
__device__ __attribute__((aligned(16))) uint8_t g_zero_scale[16];

// What bounds the product on 64 x 64 tiles per tap is the operand stream: four
// fragment loads for four MFMAs.  Here a wave accumulates NB x NB blocks of
// 32 x 32 for the three taps of a kernel row.  Its two K blocks are the same
// column of two output rows, i and i + nrp of the list of all rows (so only
// the last pair of an odd count is half empty), and it walks the columns of
// that row pair: a column step loads the G_Y fragments of one column and the
// X fragments of S new columns (S: column stride), and multiplies the G_Y
// fragment with the window of three X columns it keeps in registers -- at
// NB = 2 and S = 1 four loads for twelve MFMAs.  A row pair starts with
// PR steps that only fill the window.  Loads run D steps ahead of the
// products (a ring of D operand slots).  Everything but a column's validity
// is fixed per row pair: rows outside the input, and columns outside it, load
// from past the end of the buffer descriptor, which returns zeros.  The E8M0
// scales of a step come with one byte load per new X column: the lanes of a
// quad fetch G_Y's and X's two blocks each and broadcast them by DPP.
template <int FA, int FB, int NB, int S, int D>
__device__ __forceinline__ void wgrad_row_tile(const WRArgs& p, int bid, int nblk, float (*red)[32 * NB * 32 * NB]) {
    constexpr int NI = NB, NJ = NB;
    static_assert((FA == MXC_E4M3) == (FB == MXC_E4M3), "FP8 pairs only with FP8");
    static_assert((NB == 1 || NB == 2) && (S == 1 || S == 2), "tile shape");
    constexpr bool X8 = FA == MXC_E4M3;
    constexpr int NP = X8 ? 2 : 1;                // rows a lane reads: both (FP8), or its half's own
    constexpr int PR = S == 1 ? 2 : 1;            // window-filling steps of a row pair
    constexpr int RBA = 32 * fmt_bits(FA) / 8, RBB = 32 * fmt_bits(FB) / 8;
    constexpr int TBA = 32 * RBA, TBB = 32 * RBB;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // each XCD takes a contiguous range of (split, tile): the tiles that read
    // the same pixels share its L2
    const int per_xcd = (nblk + 7) / 8;
    const int lin = (bid % 8) * per_xcd + bid / 8;
    if (lin >= p.ntiles * p.nsplit) return;
    const int tile = lin % p.ntiles, split = lin / p.ntiles;
    const int th = tile / (p.cot * p.cit);
    const int rc = tile % (p.cot * p.cit);
    const int cob = (rc / p.cit) * NI, cib = (rc % p.cit) * NJ;   // first channel blocks
    const int r = lane & 31, hf = lane >> 5;

    // A tile's second block that does not exist reads the first one: its
    // products land in rows or columns that are not written.
    const uint32_t gblk[2] = {(uint32_t)cob * TBA, (uint32_t)min(cob + 1, p.gy_ncb - 1) * TBA};
    const uint32_t xblk[2] = {(uint32_t)cib * TBB, (uint32_t)min(cib + 1, p.x_ncb - 1) * TBB};
    // a lane whose channel row is padding reads row 0 of its block, a line
    // the real rows fetch anyway.  Its products are not zero: where the layer
    // is split they reach the padding entries of the partial sums, which the
    // reduction must not read (it stops at cout and drops ci >= cin).
    const uint32_t la = (cob * 32 + r < p.cout ? r * RBA : 0) + (X8 ? 16 * hf : 0);
    const uint32_t lb = (cib * 32 + r < p.cin ? r * RBB : 0) + (X8 ? 16 * hf : 0);
    const uint32_t gpix = (uint32_t)p.gy_ncb * TBA, xpix = (uint32_t)p.x_ncb * TBB;
    const auto grs = __builtin_amdgcn_make_buffer_rsrc((void*)p.gc, (short)0, (int)p.gbytes, 0x00020000);
    const auto xrs = __builtin_amdgcn_make_buffer_rsrc((void*)p.xc, (short)0, (int)p.xbytes, 0x00020000);
    // scale bytes: lane l % 4 = 0, 1: G_Y's blocks, 2, 3: X's
    const bool sc_x = lane & 2;
    const int sc_blk = sc_x ? min(cib + (lane & 1), p.x_ncb - 1) : min(cob + (lane & 1), p.gy_ncb - 1);

    // fragments in the registers they need (4, 6 or 8), widened at the MFMA
    constexpr int FRA = fmt_bits(FA), FRB = fmt_bits(FB);
    using FragA = WRFrag<FRA>;
    using FragB = WRFrag<FRB>;
    auto wide = [](const auto& f) {
        constexpr int N = wr_words<decltype(f)>;
        v8i o;
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = e < N ? f.d[e < N ? e : 0] : 0;
        return o;
    };
    struct Slot {
        FragA a[NI];
        FragB b[S][NJ];
        int sc[S];
    };
    Slot sl[D];
    v16f acc[3][NI][NJ];
#pragma unroll
    for (int t = 0; t < 3; t++)
#pragma unroll
        for (int i = 0; i < NI; i++)
#pragma unroll
            for (int j = 0; j < NJ; j++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[t][i][j][e] = 0.0f;

    // the wave's columns [q0, q1) of the flattened (row pair, column) list
    const int total = p.nrp * p.wo;
    const int q0 = min((split * 4 + wave) * p.spw, total), q1 = min(q0 + p.spw, total);
    const int i0 = q0 / p.wo, x0 = q0 - i0 * p.wo;
    const int nstream = q1 > q0 ? q1 - q0 + PR * ((q1 - 1) / p.wo - i0 + 1) : 0;   // steps with the window fills

    // ---- load cursor: stream step ls of row pair li; G_Y column ls - PR, X
    // columns ls - pw (S = 1) or 2 ls - 1 - pw and 2 ls - pw (S = 2)
    int li = i0, ls = x0, ln = 0;
    int lmin = x0 + PR;                           // first step of the row pair with a product
    int rg[2], ry[2];                             // group and output row of the pair's two rows
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int row = li + k * p.nrp;
        rg[k] = row / p.ho;
        ry[k] = row - rg[k] * p.ho;
    }
    // a pointer to zero scales, held in registers (its address would be
    // loaded again at every use)
    const uint8_t* zs = g_zero_scale;
    asm("" : "+s"(zs));
    const uint8_t* const sbase = (sc_x ? p.xs : p.gs) + sc_blk;
    const uint32_t sncb = sc_x ? p.x_ncb : p.gy_ncb, sadd = sc_x ? S * p.x_ncb : p.gy_ncb;
    uint32_t vg[NP], vx[NP];                      // lane offsets of the cursor's columns
    const uint8_t* sp;                            // the lane's scale of the cursor's (first) column
    uint32_t sstep;                               // 0: the lane's row does not exist
    auto set_row = [&]() {
        uint32_t go[2], xo[2], pix[2];
        bool sv[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int row = li + k * p.nrp;
            const int iy = ry[k] * p.sh + th - p.ph;
            const int v = (int)(row < p.nrows) & (int)(li < p.nrp);
            const int xv = v & (int)(iy >= 0) & (int)(iy < p.h);
            const uint32_t gp = (uint32_t)row * (uint32_t)p.wo + (uint32_t)(ls - PR);
            const uint32_t xp = ((uint32_t)rg[k] * (uint32_t)p.h + (uint32_t)iy) * (uint32_t)p.w +
                                (uint32_t)(S == 1 ? ls - p.pw : 2 * ls - 1 - p.pw);
            go[k] = v ? gp * gpix : WR_OOB;
            xo[k] = xv ? xp * xpix : WR_OOB;
            pix[k] = sc_x ? xp : gp;              // may be one or two before the tensor: not read then
            sv[k] = sc_x ? xv : v;
        }
        if (X8) {
#pragma unroll
            for (int k = 0; k < NP; k++) { vg[k] = go[k]; vx[k] = xo[k]; }
        } else {
            vg[0] = hf ? go[1] : go[0];
            vx[0] = hf ? xo[1] : xo[0];
        }
        const bool v = hf ? sv[1] : sv[0];
        const int64_t at = (int64_t)(int32_t)(hf ? pix[1] : pix[0]) * (int64_t)sncb;
        sp = v ? sbase + at : zs;
        sstep = v ? sadd : 0u;
    };
    set_row();

    auto frag = [&](auto& o, auto rs, const uint32_t* v, uint32_t blk) {
        constexpr int N = wr_words<decltype(o)>;
        const v4i u = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, v[0], blk, 0));
#pragma unroll
        for (int e = 0; e < 4; e++) o.d[e] = u[e];
        if constexpr (N == 8) {
            const v4i w = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, v[NP - 1], blk, 0));
#pragma unroll
            for (int e = 0; e < 4; e++) o.d[4 + e] = w[e];
        } else if constexpr (N == 6) {
            const v2i w = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(rs, v[0] + 16, blk, 0));
            o.d[4] = w[0];
            o.d[5] = w[1];
        }
    };

    // issue the loads of the cursor's step and move along the row; next_row
    // follows when the row pair is done
    auto load = [&](Slot& o) {
        const bool live = ln < nstream;
        const bool gl = live & (ls >= lmin);
        uint32_t ga[NP];
#pragma unroll
        for (int k = 0; k < NP; k++) ga[k] = (gl ? vg[k] : WR_OOB) + la;
#pragma unroll
        for (int i = 0; i < NI; i++) frag(o.a[i], grs, ga, gblk[i]);
#pragma unroll
        for (int c = 0; c < S; c++) {
            const int col = S == 1 ? ls - p.pw : 2 * ls - 1 - p.pw + c;
            const bool xl = live & (col >= 0) & (col < p.w);
            uint32_t xa[NP];
#pragma unroll
            for (int k = 0; k < NP; k++) xa[k] = (xl ? vx[k] + c * xpix : WR_OOB) + lb;
#pragma unroll
            for (int j = 0; j < NJ; j++) frag(o.b[c][j], xrs, xa, xblk[j]);
            const uint8_t* q = gl ? sp : zs;
            const uint8_t* qx = xl ? sp + (c && sstep ? sncb : 0u) : zs;
            o.sc[c] = *(const __attribute__((address_space(1))) uint8_t*)(sc_x ? qx : q);
        }
        ln++;
        ls++;
#pragma unroll
        for (int k = 0; k < NP; k++) { vg[k] += gpix; vx[k] += S * xpix; }
        sp += sstep;
    };
    auto next_row = [&]() {
        if (ls != p.wo + PR) return;
        ls = 0;
        lmin = PR;
        li++;
#pragma unroll
        for (int k = 0; k < 2; k++)
            if (++ry[k] == p.ho) { ry[k] = 0; rg[k]++; }
        set_row();
    };
    // quad broadcast: the scale that lane Q of each quad fetched
    auto bc = [](int s, auto q) -> int {
        constexpr int Q = decltype(q)::fn;
        return __builtin_amdgcn_mov_dpp(s, Q * 0x55, 0xF, 0xF, true);
    };

    // the window: per X column the fragments (FP8: decoded to bf16) and scales
    constexpr int WR = X8 ? 16 : FRB;
    using ColF = WRCol<WR>;
    struct Col {
        ColF f[NJ];
        int s[NJ];
    };
    Col c0, c1;                                   // S = 1: columns -2 and -1 of the step; S = 2: c1 is column -1
#pragma unroll
    for (int j = 0; j < NJ; j++) {
#pragma unroll
        for (int e = 0; e < WR; e++) c0.f[j].d[e] = c1.f[j].d[e] = 0;
        c0.s[j] = c1.s[j] = 0;
    }
    // both K blocks' scale codes in every lane (FP8 lanes hold both K blocks)
    auto decode = [&](const auto& f, int s, int* out) {
        const auto t = __builtin_amdgcn_permlane32_swap(s, s, false, false);
        e4m3_decode32(wide(f), (int)t[0], (int)t[1], (uint32_t*)out);
    };
    auto column = [&](Col& c, const FragB* f, int sc) {
#pragma unroll
        for (int j = 0; j < NJ; j++) {
            c.s[j] = j == 0 ? bc(sc, FnTag<2>{}) : bc(sc, FnTag<3>{});
            if constexpr (X8) decode(f[j], c.s[j], c.f[j].d);
            else {
#pragma unroll
                for (int e = 0; e < WR; e++) c.f[j].d[e] = f[j].d[e];
            }
        }
    };

    int cs = x0, cmin = x0 + PR;                  // compute cursor: step of the row pair, its first product
    // One step: the products of slot o, and the loads that refill slot n (the
    // one the step before used up).  FP4 / FP6 on 2 x 2 blocks: straight-line
    // code, so that the loads' address arithmetic is interleaved with the
    // products (at one wave per SIMD nothing else fills the cycles a product
    // keeps the matrix core busy); a step without a product multiplies G_Y's
    // zeros with X under a zero scale, since X's own might be NaN.  FP8, whose
    // products take four times as long and whose decoded window may hold NaN,
    // and the smaller tiles, which run several waves per SIMD, branch.
    auto step = [&](const Slot& o, Slot& n, bool live) {
        int sa[NI];
        int ad[NI][X8 ? 16 : 1];
        auto tap = [&](int t, const Col& c) {
#pragma unroll
            for (int i = 0; i < NI; i++)
#pragma unroll
                for (int j = 0; j < NJ; j++) {
                    if constexpr (X8)
                        acc[t][i][j] = mfma_x8((const uint32_t*)ad[i], (const uint32_t*)c.f[j].d, acc[t][i][j]);
                    else
                        acc[t][i][j] = mfma_mx<FA, FB>(wide(o.a[i]), wide(c.f[j]), acc[t][i][j], sa[i],
                                                       NI * NJ < 4 || live ? c.s[j] : 0);
                }
        };
        auto scales = [&]() {
#pragma unroll
            for (int i = 0; i < NI; i++) {
                sa[i] = i == 0 ? bc(o.sc[0], FnTag<0>{}) : bc(o.sc[0], FnTag<1>{});
                if constexpr (X8) decode(o.a[i], sa[i], ad[i]);
            }
        };
        if constexpr (X8 || NI * NJ < 4) {
            if (live) {
                scales();
                tap(0, S == 1 ? c0 : c1);
                if constexpr (S == 1) tap(1, c1);
            }
            load(n);
            // a new column is decoded after the products of the column it replaces
            Col w;
            column(w, o.b[0], o.sc[0]);
            if (live) tap(S == 1 ? 2 : 1, w);
            if constexpr (S == 1) { c0 = c1; c1 = w; }
            else {
                column(c1, o.b[1], o.sc[1]);
                if (live) tap(2, c1);
            }
        } else {
            scales();
            load(n);
            Col w;
            column(w, o.b[0], o.sc[0]);
            tap(0, S == 1 ? c0 : c1);
            tap(1, S == 1 ? c1 : w);
            if constexpr (S == 1) {
                tap(2, w);
                c0 = c1;
                c1 = w;
            } else {
                column(c1, o.b[1], o.sc[1]);
                tap(2, c1);
            }
#pragma unroll
            for (int m = 0; m < 12; m++) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // a product
                __builtin_amdgcn_sched_group_barrier(0x006, 6, 0);    // vector / scalar arithmetic
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);    // a load
            }
        }
    };

#pragma unroll
    for (int b = 0; b < D - 1; b++) { load(sl[b]); next_row(); }
    // Whole rings without a test in them, then the steps that are left: a walk
    // ends with its last step (short ones lost up to D - 1 empty steps: MXFP4
    // 192 -> 384 at 10x10, batch 64, stride 2, 9.9 -> 9.0 us), and one block holds
    // a whole ring, so its steps overlap (against a test before each step: MXFP8
    // 320 -> 320 at 7x7, batch 128, 26.4 -> 24.5 us; MXFP4 3 -> 16 at 640x640, batch
    // 32, 37.2 -> 35.7).  Loads past the end bring nothing.
    auto slot = [&](int b) {
        step(sl[b], sl[(b + D - 1) % D], cs >= cmin);
        next_row();
        if (++cs == p.wo + PR) { cs = 0; cmin = PR; }
    };
    int ks = 0;
    for (; ks + D <= nstream; ks += D) {
#pragma unroll
        for (int b = 0; b < D; b++) slot(b);
    }
#pragma unroll
    for (int b = 0; b < D - 1; b++)
        if (ks + b < nstream) slot(b);

    // ---- per tap: sum the four waves' tiles, then write
    constexpr int RI = 32 * NI, RJ = 32 * NJ;
#pragma unroll
    for (int t = 0; t < 3; t++) {
        if (t > 0) __syncthreads();                   // the previous tap's sums are read
#pragma unroll
        for (int i = 0; i < NI; i++)
#pragma unroll
            for (int j = 0; j < NJ; j++)
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const int row = 32 * i + 8 * (e >> 2) + 4 * hf + (e & 3);
                    red[wave][row * RJ + 32 * j + r] = acc[t][i][j][e];
                }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < RI * RJ / WRT; k++) {
            const int idx = tid + WRT * k;
            const int row = idx / RJ, col = idx % RJ;
            const float v = (red[0][idx] + red[1][idx]) + (red[2][idx] + red[3][idx]);
            const int co = cob * 32 + row, ci = cib * 32 + col;
            if (p.direct) {
                if (co < p.cout && ci < p.cin) p.dst[(((size_t)co * p.cin + ci) * p.kh + th) * 3 + t] = v;
            } else if (co < p.gy_cp && ci < p.x_cp) {
                p.dst[((size_t)split * p.gy_cp + co) * p.ntot + (size_t)(th * 3 + t) * p.x_cp + ci] = v;
            }
        }
    }
}

// The tile arguments for one launch of a layer (cv: its batch groups; dst: G_W
// with one split in all, else this launch's partial tiles); returns the
// workgroup count, a multiple of 8.
inline long wgrad_row_fill(const Conv& cv, const WRPlan& q, const void* gc, const uint8_t* gs, const void* xc,
                           const uint8_t* xs, float* dst, WRArgs& a) {
    a.gc = (const uint8_t*)gc; a.gs = gs; a.xc = (const uint8_t*)xc; a.xs = xs;
    a.dst = dst;
    a.direct = q.splits == 1;
    a.cout = cv.cout; a.cin = cv.cin; a.kh = cv.kh; a.sh = cv.sh; a.ph = cv.ph; a.pw = cv.pw;
    a.ho = cv.ho; a.wo = cv.wo; a.h = cv.h; a.w = cv.w;
    a.gy_ncb = cv.gy.ncb; a.x_ncb = cv.x.ncb; a.gy_cp = cv.gy.cp; a.x_cp = cv.x.cp;
    a.ntot = cv.kh * 3 * cv.x.cp;
    a.gbytes = (uint32_t)((long)cv.gy.ng * cv.ho * cv.wo * cv.gy.cp * 4 * fmt_bits(cv.fa));
    a.xbytes = (uint32_t)((long)cv.x.ng * cv.h * cv.w * cv.x.cp * 4 * fmt_bits(cv.fb));
    a.nrows = cv.x.ng * cv.ho;
    a.nrp = (a.nrows + 1) / 2;
    a.cot = (cv.gy.ncb + q.nb - 1) / q.nb;
    a.cit = (cv.x.ncb + q.nb - 1) / q.nb;
    a.ntiles = q.ntiles;
    const long total = (long)a.nrp * cv.wo, waves = 4L * q.per;
    a.spw = (int)((total + waves - 1) / waves);
    a.nsplit = q.per;
    return ((long)q.ntiles * q.per + 7) / 8 * 8;
}

}  // namespace
