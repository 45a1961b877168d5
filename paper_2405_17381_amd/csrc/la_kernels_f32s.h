// fp32 path: the block loop of Alg. 5 / Alg. 6 with every contraction on the bf16 matrix cores,
// at fp32 accuracy, d = 64 and d = 128; blocks of BK = 32 rows.
//
// What bounds it.  In fp32 the path is bound by its contractions, not by memory: 160
// v_mfma_f32_32x32x2_f32 of 64 cycles per wave and block at d = 128, 4.3 us of matrix-core time
// for 48 KB of tiles.  A bf16 MFMA does sixteen times the work per cycle, and an fp32 number is
// exactly the sum of three bf16 numbers,
//     x = h + m + l,   h = bf16(x), m = bf16(x - h), l = x - h - m     (8 + 8 + 8 significant bits)
// so every product of two fp32 numbers is the sum of nine bf16 products, each exact in fp32.  The
// six of them that reach 2^-18 of the product are computed (hh, hm, mh, hl, lh, mm); the other three
// are below 2^-26 of it, a quarter of an fp32 rounding.  120 MFMAs of 32 cycles remain, and some
// 1100 vector instructions, most of them splits; counters show a SIMD issuing 64 % of the time, so
// what is left is the dependent chain of a block (four barriers, LDS round trips) that two waves per
// SIMD do not cover entirely.
// Accuracy.  Small products go to an accumulator of their own (or first into a common one) and meet
// the large ones in a single addition, and a block's contribution to the state is summed from zero
// and added once, so long sums see fewer roundings than the fp32 instruction gives them.
// Measured against v_mfma_f32_32x32x2_f32 (d = 128) and FMA (d = 64) kernels, la_fwd + la_bwd, with the
// relative 2-norm error against 64-bit arithmetic: 8 x 16 scans of 2048 tokens at d = 128, 1.26 -> 0.93 ms,
// 5.2e-7 -> 1.7e-7; two scans of 256 tokens at d = 64, 300 -> 71 us, 2.1e-7 -> 0.9e-7.
//
// One workgroup of D/32 wavefronts per (scan, segment), two workgroups per compute unit (72 KB of
// LDS each); ownership and fragment layouts are those of la_kernels_bf16_dma.h: wave w owns value
// features [32w, 32w+32) of Out and of the state, which stays in its accumulator registers in fp32.
// Tiles are split once, by the thread that fetched them, into three row-major bf16 tiles per operand
// (same row pitch and chunk swizzle as there); row reads serve the contractions over the features and
// transposing reads those over the tokens.  The score tile's feature sum is split over the waves (each
// wave would otherwise spend 48 MFMAs instead of 12 on it) and combined through the A tile's storage.
// The next block's tiles are prefetched into registers.
//
// Range.  The split needs |x| well below the largest bf16 number, and an infinite operand times a zero
// part would give NaN where fp32 arithmetic gives infinity.  A workgroup that meets a tile entry of
// 2^28 or more or NaN (or such an entering state, of 2^87 or more) runs that block and all that follow
// on v_mfma_f32_32x32x2_f32 instead; below those bounds nothing can overflow in the split form
// (n < 2^30: state < 2^87, result < 2^122).
#pragma once
#include "la_kernels_bf16_dma.h"

template <int D>
struct F32sCfg {
    static constexpr int BK = 32, NW = D / 32, NT = 64 * NW;
    static constexpr int PITCH = 2 * D, CPR = D / 8;
    static constexpr int PART = BK * D * 2;                  // one bf16 part of a tile: 8192 at D = 128
    static constexpr int OPER = 3 * PART;                    // an operand's h, m, l tiles
    // decay tables: rising, lambda^k at BK + k (k = -BK .. BK, zero for k < 0), falling, lambda^(BK - k) at
    // k (k = 0 .. 2 BK, zero for k > BK); and the flag "a block out of range was met"
    static constexpr int TABLE = 4 * (2 * (2 * BK + 1) + 2);
    static constexpr size_t lds_bytes(bool state_only) { return (size_t)(state_only ? 2 : 3) * OPER + TABLE; }
    // fp32 form (same storage): row-major tiles with row stride D + 1, partial scores
    static constexpr int LD = D + 1, LSP = BK + 1;
    static_assert(4 * (3 * BK * LD + NW * BK * LSP) <= 3 * OPER && 8 * BK * LD <= 2 * OPER, "fp32 form fits");
    static_assert(NW * 4096 <= OPER, "partial scores fit in the A tiles");
};

constexpr float kF32sTileMax = 268435456.0f;                 // 2^28
constexpr float kF32sStateMax = 1.5474250491067253e26f;      // 2^87

__device__ __forceinline__ f32x16_t mfma_f32(float a, float b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// The three bf16 parts of two fp32 numbers, packed.  The residuals x - bf16(x) come from the dot
// product of the packed pair with (-1, 0) or (0, -1), one instruction each where unpacking and
// subtracting takes two; they are exactly representable, so its rounding does not matter.
// neg_lo, neg_hi: those two constants in scalar registers (see F32sNeg).
struct F32sNeg {
    uint32_t lo, hi;
};
__device__ __forceinline__ float f32s_residual(uint32_t pair, uint32_t neg, float x)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pair), __builtin_bit_cast(bf16x2_t, neg), x, false);
}
__device__ __forceinline__ void f32s_split2(const F32sNeg &neg, float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    h = pack2_bf16(a, b);
    const float ra = f32s_residual(h, neg.lo, a), rb = f32s_residual(h, neg.hi, b);
    m = pack2_bf16(ra, rb);
    l = pack2_bf16(f32s_residual(m, neg.lo, ra), f32s_residual(m, neg.hi, rb));
}
// x * w where a zero weight gives zero whatever x is (a masked score may be NaN)
__device__ __forceinline__ float f32s_mask(float x, float w)
{
    float r;
    asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(w));
    return r;
}

// operand fragment in three parts, and the six products: the large one onto `big`, the others onto `small`
struct F32sFrag {
    U4 h, m, l;
};
__device__ __forceinline__ void f32s_mfma(const F32sFrag &a, const F32sFrag &b, f32x16_t &big, f32x16_t &small)
{
    small = mfma32(a.l, b.h, small);
    big = mfma32(a.h, b.h, big);
    small = mfma32(a.h, b.l, small);
    small = mfma32(a.m, b.m, small);
    small = mfma32(a.m, b.h, small);
    small = mfma32(a.h, b.m, small);
}

// Nothing moves across the end of a step: the scheduler would otherwise lift the splits and the
// fragment reads of many steps at once and run out of registers.  Each step reads the next one's
// fragments, so the LDS latency hides behind six MFMAs.
#define LA_F32S_STEP() __builtin_amdgcn_sched_barrier(0)
// Within a step: N times one MFMA followed by M vector instructions, so that the split of the next
// step's operand issues while the matrix core works on this one's.
template <int N, int M>
__device__ __forceinline__ void f32s_mix()
{
    if constexpr (N > 0) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, M, 0);
        f32s_mix<N - 1, M>();
    }
}
#define LA_F32S_MIX(N, M) f32s_mix<N, M>()

// max(big, |a|, |b|), NaN if any of them is
__device__ __forceinline__ float f32s_max3(float big, float a, float b)
{
    asm("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(big) : "v"(a), "v"(b));
    return big;
}

// REBUILD: short pieces whose workgroups first walk the blocks before their piece with the state update
// alone, for launches that would leave most of the chip idle (see la_scan_bf16_dma).
template <int D, bool STATE_ONLY, bool REBUILD = false>
__global__ __launch_bounds__(2 * D, 2) void la_scan_f32s(ScanLaunch launch, LaLambdas lams)
{
    using Cfg = F32sCfg<D>;
    constexpr int BK = Cfg::BK, NW = Cfg::NW, NT = Cfg::NT, PITCH = Cfg::PITCH, CPR = Cfg::CPR;
    constexpr int PART = Cfg::PART, OPER = Cfg::OPER, LD = Cfg::LD, LSP = Cfg::LSP;
    constexpr int KS_D = D / 16, KS_B = BK / 16, MT_D = D / 32;
    constexpr int SW8 = dma_swz<D>(8);
    constexpr int OFF_B = STATE_ONLY ? 0 : OPER, OFF_C = OFF_B + OPER;

    extern __shared__ __align__(16) unsigned char smem_f32s[];
    unsigned char *sA = smem_f32s, *sB = smem_f32s + OFF_B, *sC = smem_f32s + OFF_C;
    float *sPw = reinterpret_cast<float *>(smem_f32s + OFF_C + OPER) + BK;
    float *sFall = sPw + BK + 1;                             // sFall[k] = lambda^(BK - k)
    // (a plain LDS access: through a generic pointer it would wait for the result stores in flight)
    volatile __attribute__((address_space(3))) int *sFlag = (volatile __attribute__((address_space(3))) int *)(sFall + 2 * BK + 1);

    const int tid = threadIdx.x;
    const int l = tid & 63;
    int l32 = l & 31, g = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Pre-passes (one or two independent ones in a launch) follow one another in the grid; the block
    // scans of a backward pass (up to three roles) interleave, the workgroups of an item on one XCD.
    int role = 0, item = (int)blockIdx.x;
    if (STATE_ONLY) {
        if (launch.nroles == 2) {
            role = (int)(blockIdx.x / launch.items);
            item = (int)(blockIdx.x % launch.items);
        }
    } else if (launch.nroles > 1) {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        role = slot % launch.nroles;
        item = (slot / launch.nroles) * 8 + xcd;
        if (item >= launch.items) return;
    }
    const ScanArgs &a = launch.r[role];
    const bool rev = a.rev != 0;
    const int seg = item % a.S;
    int scan = item / a.S;
    if (STATE_ONLY) {
        const int b = scan % a.B, hd = scan / a.B;           // heads in dispatch order
        scan = b * a.H + lams.order[hd];
        if (!rev && seg == a.S - 1) return;                  // never consumed
        if (rev && seg == 0) return;
    }
    const float lam = lams.v[scan % a.H], lg = lams.lg2[scan % a.H];
    int seg_lo = seg * a.L;
    int seg_hi = min(a.n, seg_lo + a.L);
    int nwarm = 0;                             // leading blocks that only update the state
    bool from_start = true;                    // ... and whether they begin where the scan does
    if (REBUILD) {
        const int before = rev ? a.n - seg_hi : seg_lo;
        int rows = before;
        if (a.skip_bits > 0.f && lg < 0.f) {
            const float reach = a.skip_bits / -lg;
            if (reach < (float)before) rows = min(before, ((int)(reach / BK) + 2) * BK);
        }
        from_start = rows == before;
        nwarm = (rows + BK - 1) / BK;
        if (rev) seg_hi += rows;
        else seg_lo -= rows;
    }
    const int nblk = (seg_hi - seg_lo + BK - 1) / BK;

    const int bi = scan / a.H, hi = scan % a.H;
    const float *gA = (const float *)a.A + (size_t)bi * a.lA.bs + (size_t)hi * a.lA.hs;
    const float *gB = (const float *)a.Bm + (size_t)bi * a.lB.bs + (size_t)hi * a.lB.hs;
    const float *gC = (const float *)a.C + (size_t)bi * a.lC.bs + (size_t)hi * a.lC.hs;
    float *gO = (float *)a.Out + (size_t)bi * a.lO.bs + (size_t)hi * a.lO.hs;
    const float *gE = (a.act & LA_ACT_OUT) ? (const float *)a.E + (size_t)bi * a.lE.bs + (size_t)hi * a.lE.hs : gA;
    const int ldA = a.lA.ld, ldB = a.lB.ld, ldC = a.lC.ld, ldO = a.lO.ld, ldE = a.lE.ld;

    // lambda^k in double (binary powering: a relative error of a few 2^-53), rounded once; zero for
    // k < 0, so that the weight lambda^(m-1-r) of a row r >= m of a partial block needs no clamp
    for (int k = tid - BK; k <= BK; k += NT) {
        double p = 1.0, b = (double)lam;
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            if ((k >> e) & 1) p *= b;
            b *= b;
        }
        const float pk = k < 0 ? 0.0f : (float)p;
        sPw[k] = pk;
        sFall[BK - k] = pk;
    }
    if (tid == 0) *sFlag = 0;
    F32sNeg neg = {0x0000bf80u, 0xbf800000u};                // bf16 pairs (-1, 0) and (0, -1)
    // (opaque: the compiler would encode the first as the inline constant -1.0, which reads as (-1.0f)'s
    // 32 bits, i.e. as (0, -1))
    asm("" : "+s"(neg.lo), "+s"(neg.hi));

    // ---- per-lane addressing (see la_kernels_bf16_dma.h) ---------------------------------
    int ro_base = l32 * PITCH, ro_sw = dma_swz<D>(l32) ^ g;
    const int a4 = l & 3, b4 = (l >> 2) & 3, h16 = (l >> 4) & 1;
    int tr_base = (4 * g + b4) * PITCH + 8 * (a4 & 1);
    int tr_sw = (2 * h16 + (a4 >> 1)) ^ dma_swz<D>(4 * g + b4);
    auto row_frag = [&](const unsigned char *s, int ks) -> F32sFrag {
        const unsigned char *p = s + ro_base + (((2 * ks) ^ ro_sw) << 4);
        return F32sFrag{*(const U4 *)p, *(const U4 *)(p + PART), *(const U4 *)(p + 2 * PART)};
    };
    auto tr_part = [&](const unsigned char *s, int ks, int mt) -> U4 {
        const unsigned char *p = s + tr_base + 16 * ks * PITCH;
        const U2 lo = lds_read_tr(p + (((4 * mt) ^ tr_sw) << 4));
        const U2 hi2 = lds_read_tr(p + 8 * PITCH + (((4 * mt) ^ tr_sw ^ SW8) << 4));
        return U4{lo[0], lo[1], hi2[0], hi2[1]};
    };
    auto tr_frag = [&](const unsigned char *s, int ks, int mt) -> F32sFrag {
        return F32sFrag{tr_part(s, ks, mt), tr_part(s + PART, ks, mt), tr_part(s + 2 * PART, ks, mt)};
    };
    // staging: this thread's chunks of eight features, (row srow + 16 u, chunk sch), u = 0, 1
    int srow = tid / CPR, sch = tid % CPR;

    // ---- running state St[i][j], j = 32 w + l32, in accumulator layout ---------------------
    f32x16_t st[MT_D];
    const float *gIn = STATE_ONLY ? nullptr
                       : REBUILD  ? (!rev && from_start && a.st_in ? a.st_in + (size_t)scan * (D * D) : nullptr)
                                  : la_entering_state(a, scan, seg, rev, lg, D * D);
    float amax = 0.0f;
#pragma unroll
    for (int mt = 0; mt < MT_D; ++mt) st[mt] = f32x16_t{0};
    if (gIn) {                                               // (all loads of the state in flight at once)
        const float *p = gIn + (a.transpose_init ? (32 * w + l32) * D + 4 * g : 4 * g * D + 32 * w + l32);
        const int di = a.transpose_init ? 1 : D;             // distance of one state row
#pragma unroll
        for (int mt = 0; mt < MT_D; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) st[mt][v] = p[(32 * mt + 8 * (v >> 2) + (v & 3)) * di];
#pragma unroll
        for (int mt = 0; mt < MT_D; ++mt)
#pragma unroll
            for (int v = 0; v < 16; v += 2) amax = f32s_max3(amax, st[mt][v], st[mt][v + 1]);
    }
    const bool want_final = !STATE_ONLY && !rev && a.st_out != nullptr && seg == a.S - 1;

    int ib0 = 0;     // pre-pass: skip blocks whose decay weights are below 2^-skip_bits
    if (STATE_ONLY && a.skip_bits > 0.f && lam < 1.0f) {
        const float reach = a.skip_bits / -lg;
        if (reach < (float)(nblk * BK)) ib0 = max(0, nblk - ((int)(reach / BK) + 2));
    }
    __syncthreads();                                         // table and flag ready
    if (!(amax < kF32sStateMax)) *sFlag = 1;

    // ---- global -> registers (rows past the segment end read the last row and are zeroed when
    // the block is staged) ---------------------------------------------------------------------
    float4 ra[2][2], rb[2][2], rc[2][2];
    auto load_block = [&](int blk, bool lead = false) {      // lead: no A tile
        const int t0 = seg_lo + blk * BK;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const size_t row = (size_t)min(t0 + srow + 16 * u, seg_hi - 1);
            const float4 *pb = (const float4 *)(gB + row * ldB + 8 * sch);
            const float4 *pc = (const float4 *)(gC + row * ldC + 8 * sch);
            rb[u][0] = pb[0]; rb[u][1] = pb[1];
            rc[u][0] = pc[0]; rc[u][1] = pc[1];
            if (!STATE_ONLY && !(REBUILD && lead)) {
                const float4 *pa = (const float4 *)(gA + row * ldA + 8 * sch);
                ra[u][0] = pa[0]; ra[u][1] = pa[1];
            }
        }
    };
    // zero padding of a partial block (exact)
    auto pad_block = [&](int t0) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (t0 + srow + 16 * u >= seg_hi) {
                const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
                rb[u][0] = rb[u][1] = rc[u][0] = rc[u][1] = z;
                if (!STATE_ONLY) ra[u][0] = ra[u][1] = z;
            }
    };
    // Swish of the operands that are pre-activations (phi(0) = 0: the padding stays zero)
    auto act_block = [&]() {
        auto act4 = [](float4 &x) { x = make_float4(la_swish(x.x), la_swish(x.y), la_swish(x.z), la_swish(x.w)); };
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (a.act & LA_ACT_BM) act4(rb[u][e]);
                if (a.act & LA_ACT_C) act4(rc[u][e]);
                if (!STATE_ONLY && (a.act & LA_ACT_A)) act4(ra[u][e]);
            }
    };
    auto unpack = [](const float4 (&r)[2], float (&x)[8]) {
        x[0] = r[0].x; x[1] = r[0].y; x[2] = r[0].z; x[3] = r[0].w;
        x[4] = r[1].x; x[5] = r[1].y; x[6] = r[1].z; x[7] = r[1].w;
    };
    // registers -> LDS, split; returns the largest magnitude staged by this thread
    auto stage_split = [&](bool lead = false) -> float {
        float big = 0.0f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = srow + 16 * u;
            const int off = r * PITCH + ((sch ^ dma_swz<D>(r)) << 4);
            auto put = [&](const float4 (&rr)[2], unsigned char *dst) {
                float x[8];
                unpack(rr, x);
                F32sFrag f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t h, m, lo;
                    f32s_split2(neg, x[2 * e], x[2 * e + 1], h, m, lo);
                    f.h[e] = h; f.m[e] = m; f.l[e] = lo;
                    big = f32s_max3(big, x[2 * e], x[2 * e + 1]);
                }
                *(U4 *)(dst + off) = f.h;
                *(U4 *)(dst + off + PART) = f.m;
                *(U4 *)(dst + off + 2 * PART) = f.l;
                LA_F32S_STEP();
            };
            put(rb[u], sB);
            put(rc[u], sC);
            if (!STATE_ONLY && !(REBUILD && lead)) put(ra[u], sA);
        }
        return big;
    };
    // ... and unsplit, for the fp32 form: [A][B][C] (pre-pass: [B][C]), row stride LD
    float *pA = reinterpret_cast<float *>(smem_f32s);
    float *pB = pA + (STATE_ONLY ? 0 : BK * LD), *pC = pB + BK * LD;
    float *pS = pC + BK * LD;                                // [NW][BK][LSP]
    auto stage_plain = [&]() {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = srow + 16 * u;
            auto put = [&](const float4 (&rr)[2], float *dst) {
                float x[8];
                unpack(rr, x);
#pragma unroll
                for (int e = 0; e < 8; ++e) dst[r * LD + 8 * sch + e] = x[e];
            };
            put(rb[u], pB);
            put(rc[u], pC);
            if (!STATE_ONLY) put(ra[u], pA);
        }
    };
    // result of row t, features 32 w + col .. + 3
    auto store4 = [&](int t, int col, float4 o) {
        if (a.act & LA_ACT_OUT) {                            // phi' of the pre-activation tile
            const float4 e = *(const float4 *)(gE + (size_t)t * ldE + 32 * w + col);
            o.x *= la_swish_grad(e.x); o.y *= la_swish_grad(e.y);
            o.z *= la_swish_grad(e.z); o.w *= la_swish_grad(e.w);
        }
        float4 *dst = (float4 *)(gO + (size_t)t * ldO + 32 * w + col);
        if (a.act & LA_ACT_ACC) {                            // add to what is there
            const float4 e = *dst;
            o.x += e.x; o.y += e.y; o.z += e.z; o.w += e.w;
        }
        *dst = o;
    };

    const auto blk_of = [&](int ib) { return rev ? (nblk - 1 - ib) : ib; };
    // the state handed back is the one after the last real row: the final, partial block of m rows is
    // weighted lambda^(m-1-r) and decays the old state by lambda^m
    const auto rows_of = [&](int t0) { return (want_final && t0 + BK > seg_hi) ? seg_hi - t0 : BK; };
    const bool any_act = (a.act & (LA_ACT_A | LA_ACT_BM | LA_ACT_C)) != 0;
    // REBUILD: the state entering a multiple of saved_L, to the slot where la_entering_state looks for it
    const int own_lo = seg_lo + (REBUILD && !rev ? nwarm * BK : 0);
    const bool state_due = REBUILD && !rev && launch.saved != nullptr && own_lo % launch.saved_L == 0;
    auto save_state = [&]() {
        const int s0 = own_lo / launch.saved_L;
        const bool chain_free = a.skip_bits > 0.f && -lg * (float)launch.saved_L >= a.skip_bits;
        if (chain_free && s0 == 0) return;
        float *p = launch.saved + ((size_t)scan * launch.saved_S + (chain_free ? s0 - 1 : s0)) * (size_t)(D * D) +
                   4 * g * D + 32 * w + l32;
#pragma unroll
        for (int mt = 0; mt < MT_D; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) p[(32 * mt + 8 * (v >> 2) + (v & 3)) * D] = st[mt][v];
    };
    int ib = ib0;
    if (ib < nblk) load_block(blk_of(ib), ib < nwarm);
    for (; ib < nblk; ++ib) {
        const bool lead = REBUILD && ib < nwarm;
        if (REBUILD && state_due && ib == nwarm) save_state();
        const int t0 = seg_lo + blk_of(ib) * BK, m_rows = rows_of(t0);
        // the lane's address terms are derived anew in every block (an XOR or an add each) instead of
        // living in a register per address for the whole loop, which would leave none for the prefetch
        asm volatile("" : "+v"(l32), "+v"(g), "+v"(ro_base), "+v"(ro_sw), "+v"(tr_base), "+v"(tr_sw), "+v"(srow), "+v"(sch));
        if (t0 + BK > seg_hi) pad_block(t0);
        if (any_act) act_block();
        if (!(stage_split(lead) < kF32sTileMax)) *sFlag = 1;
        __syncthreads();                                     // tiles staged
        if (__builtin_amdgcn_readfirstlane(*sFlag) != 0) break;
        if (ib + 1 < nblk) load_block(blk_of(ib + 1), ib + 1 < nwarm);
        f32x16_t x = {0};
        if (!STATE_ONLY && !lead) {
            // ---- this wave's share of the scores: S^T (lane = q, registers = keys) over 32 features
            f32x16_t s = {0};
            {
                f32x16_t sc = {0};
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const F32sFrag fa = row_frag(sA, 2 * w + k), fb = row_frag(sB, 2 * w + k);
                    f32s_mfma(fb, fa, s, sc);
                    LA_F32S_STEP();
                }
                s += sc;
            }
            LA_F32S_STEP();
            // ---- inter block: x^T = (St^T A^T) * scale(q); state operand from the accumulators, the
            // lane halves exchanging the rows they lack
            f32x16_t xc = {0};
            auto state_frag = [&](int ks) -> F32sFrag {
                const int mt = ks >> 1, h8 = 8 * (ks & 1);
                F32sFrag so;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    uint32_t xh, xm, xl, yh, ym, yl;
                    f32s_split2(neg, st[mt][h8 + 2 * e], st[mt][h8 + 2 * e + 1], xh, xm, xl);
                    f32s_split2(neg, st[mt][h8 + 4 + 2 * e], st[mt][h8 + 5 + 2 * e], yh, ym, yl);
                    const auto rh = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
                    const auto rm = __builtin_amdgcn_permlane32_swap(xm, ym, false, false);
                    const auto rl = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
                    so.h[e] = rh[0]; so.h[2 + e] = rh[1];
                    so.m[e] = rm[0]; so.m[2 + e] = rm[1];
                    so.l[e] = rl[0]; so.l[2 + e] = rl[1];
                }
                return so;
            };
            F32sFrag fn = row_frag(sA, 0), sn = state_frag(0);
            LA_F32S_STEP();
#pragma unroll
            for (int ks = 0; ks < KS_D; ++ks) {
                const F32sFrag fa = fn, so = sn;
                if (ks + 1 < KS_D) {
                    fn = row_frag(sA, ks + 1);
                    sn = state_frag(ks + 1);
                }
                f32s_mfma(so, fa, x, xc);
                LA_F32S_MIX(6, 9);
                LA_F32S_STEP();
            }
            const float rsq = sPw[rev ? BK - l32 : l32 + 1];
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = (x[v] + xc[v]) * rsq;
            __syncthreads();                             // every wave is done with the A tiles
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4)
                *(float4 *)(sA + ((v4 * NW + w) * 64 + l) * 16) =
                    make_float4(s[4 * v4], s[4 * v4 + 1], s[4 * v4 + 2], s[4 * v4 + 3]);
            __syncthreads();                             // partial scores complete
            // ---- P = S * mask, split in registers: already the operand of the intra product
            xc = f32x16_t{0};
            // lambda^|q - key| of keys 4 g, 4 g + 1, ..; zero beyond the diagonal
            const float *mask_tab = (rev ? sPw - l32 : sFall + BK - l32) + 4 * g;
            auto score_frag = [&](int ks) -> F32sFrag {
                F32sFrag pk;
#pragma unroll
                for (int v4 = 0; v4 < 2; ++v4) {
                    float4 t = *(const float4 *)(sA + (((2 * ks + v4) * NW) * 64 + l) * 16);
#pragma unroll
                    for (int ww = 1; ww < NW; ++ww) {
                        const float4 y = *(const float4 *)(sA + (((2 * ks + v4) * NW + ww) * 64 + l) * 16);
                        t.x += y.x; t.y += y.y; t.z += y.z; t.w += y.w;
                    }
                    float p[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        p[e] = f32s_mask(p[e], mask_tab[16 * ks + 8 * v4 + e]);
                    }
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        uint32_t h, m, lo;
                        f32s_split2(neg, p[2 * e], p[2 * e + 1], h, m, lo);
                        pk.h[2 * v4 + e] = h; pk.m[2 * v4 + e] = m; pk.l[2 * v4 + e] = lo;
                    }
                }
                return pk;
            };
            // ---- intra block: Out^T += C^T P^T
            const F32sFrag c0 = tr_frag(sC, 0, w), p0 = score_frag(0);
            LA_F32S_STEP();
            const F32sFrag c1 = tr_frag(sC, 1, w), p1 = score_frag(1);
            f32s_mfma(c0, p0, x, xc);
            LA_F32S_MIX(6, 15);
            LA_F32S_STEP();
            f32s_mfma(c1, p1, x, xc);
            auto store_row = [&]() {
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4)
                    store4(t0 + l32, 8 * v4 + 4 * g,
                           make_float4(x[4 * v4] + xc[4 * v4], x[4 * v4 + 1] + xc[4 * v4 + 1],
                                       x[4 * v4 + 2] + xc[4 * v4 + 2], x[4 * v4 + 3] + xc[4 * v4 + 3]));
            };
            // (two forms, so that the compiler can count the stores of a full block and does not make the
            // next block's staging wait for them along with its loads)
            if (t0 + BK <= seg_hi) {
                store_row();
            } else {
                if (t0 + l32 < seg_hi) store_row();
                __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
            }
        }
        // ---- state update: St = lambda^BK St + Bm^T (w C) ------------------------------------
        {
            const float decay = sPw[m_rows];
            const float *w_tab = (rev ? sPw : sFall + 1 + BK - m_rows) + 4 * g;   // weight of rows 4 g, ..
            F32sFrag cw[KS_B];
#pragma unroll
            for (int ks = 0; ks < KS_B; ++ks) {
                const F32sFrag c = tr_frag(sC, ks, w);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int key = 16 * ks + (e < 2 ? 0 : 8) + 2 * (e & 1);   // slot 2 e's row, less 4 g
                    const float w0 = w_tab[key], w1 = w_tab[key + 1];
                    uint32_t h, m, lo;
                    f32s_split2(neg, ((bf16_lo(c.h[e]) + bf16_lo(c.m[e])) + bf16_lo(c.l[e])) * w0,
                                ((bf16_hi(c.h[e]) + bf16_hi(c.m[e])) + bf16_hi(c.l[e])) * w1, h, m, lo);
                    cw[ks].h[e] = h; cw[ks].m[e] = m; cw[ks].l[e] = lo;
                }
                LA_F32S_STEP();
            }
            // one accumulator per tile, the small products first, so that the block's contribution
            // sees the rounding of two additions, and the state that of one
            F32sFrag b0 = tr_frag(sB, 0, 0), b1 = tr_frag(sB, 1, 0);
#pragma unroll
            for (int mt = 0; mt < MT_D; ++mt) {
                f32x16_t u = {0};
                u = mfma32(b0.l, cw[0].h, u);
                u = mfma32(b0.m, cw[0].m, u);
                u = mfma32(b0.h, cw[0].l, u);
                u = mfma32(b1.l, cw[1].h, u);
                u = mfma32(b1.m, cw[1].m, u);
                u = mfma32(b1.h, cw[1].l, u);
                u = mfma32(b0.m, cw[0].h, u);
                u = mfma32(b0.h, cw[0].m, u);
                u = mfma32(b1.m, cw[1].h, u);
                u = mfma32(b1.h, cw[1].m, u);
                u = mfma32(b0.h, cw[0].h, u);
                u = mfma32(b1.h, cw[1].h, u);
                if (mt + 1 < MT_D) {
                    b0 = tr_frag(sB, 0, mt + 1);
                    b1 = tr_frag(sB, 1, mt + 1);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) st[mt][v] = fmaf(decay, st[mt][v], u[v]);
                LA_F32S_STEP();
            }
        }
        __syncthreads();                                     // every tile of this block is dead
    }
    // ---- the fp32 form, from the first block out of range on (v_mfma_f32_32x32x2_f32: A operand
    // A[l%32][l/32], B operand B[l/32][l%32]), single floats from row-major tiles; register v of a
    // state tile pairs rows i and i + 4
    // (a leading block that meets its end here has its result computed too, and not stored)
    if (ib < nblk) load_block(blk_of(ib));
    for (int first = ib; ib < nblk; ++ib) {
        const bool lead = REBUILD && ib < nwarm;
        if (REBUILD && state_due && ib == nwarm && ib > first) save_state();
        const int t0 = seg_lo + blk_of(ib) * BK, m_rows = rows_of(t0);
        if (t0 + BK > seg_hi) pad_block(t0);
        if (any_act) act_block();
        stage_plain();
        if (ib + 1 < nblk) load_block(blk_of(ib + 1));
        __syncthreads();
        f32x16_t acc = {0};
        if (!STATE_ONLY) {
            f32x16_t s = {0};
#pragma unroll 4
            for (int k = 0; k < 16; ++k) {               // partial scores S[q][key] over 32 features
                const int f = 32 * w + 2 * k + g;
                s = mfma_f32(pA[l32 * LD + f], pB[l32 * LD + f], s);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) pS[(w * BK + 8 * (v >> 2) + 4 * g + (v & 3)) * LSP + l32] = s[v];
#pragma unroll
            for (int mt = 0; mt < MT_D; ++mt) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    acc = mfma_f32(pA[l32 * LD + 32 * mt + 8 * (v >> 2) + 4 * g + (v & 3)], st[mt][v], acc);
                LA_F32S_STEP();
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int q = 8 * (v >> 2) + 4 * g + (v & 3);
                acc[v] *= rev ? sPw[BK - q] : sPw[q + 1];
            }
            __syncthreads();                             // partial score tiles complete
#pragma unroll 4
            for (int k = 0; k < 16; ++k) {
                const int key = 2 * k + g, q = l32;
                float p = 0.f;
#pragma unroll
                for (int ww = 0; ww < NW; ++ww) p += pS[(ww * BK + q) * LSP + key];
                const int dist = rev ? key - q : q - key;
                acc = mfma_f32(dist >= 0 ? p * sPw[dist] : 0.f, pC[key * LD + 32 * w + l32], acc);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = t0 + 8 * (v >> 2) + 4 * g + (v & 3);
                if (t < seg_hi && !lead) {
                    float o = acc[v];
                    if (a.act & LA_ACT_OUT) o *= la_swish_grad(gE[(size_t)t * ldE + 32 * w + l32]);
                    if (a.act & LA_ACT_ACC) o += gO[(size_t)t * ldO + 32 * w + l32];
                    gO[(size_t)t * ldO + 32 * w + l32] = o;
                }
            }
        }
        const float decay = sPw[m_rows];
#pragma unroll
        for (int mt = 0; mt < MT_D; ++mt) {
            f32x16_t s = st[mt];
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] *= decay;
#pragma unroll 4
            for (int k = 0; k < 16; ++k) {
                const int r = 2 * k + g;
                const float wr = rev ? sPw[r] : sPw[m_rows - 1 - r];
                s = mfma_f32(wr * pB[r * LD + 32 * mt + l32], pC[r * LD + 32 * w + l32], s);
            }
            st[mt] = s;
            LA_F32S_STEP();
        }
        __syncthreads();                                     // every tile of this block is dead
    }

    if (STATE_ONLY || want_final) {
        float *dst = STATE_ONLY ? a.states + ((size_t)scan * a.S + seg) * (size_t)(D * D)
                                : a.st_out + (size_t)scan * (D * D);
#pragma unroll
        for (int mt = 0; mt < MT_D; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = 32 * mt + 8 * (v >> 2) + 4 * g + (v & 3);
                dst[(size_t)i * D + 32 * w + l32] = st[mt][v];
            }
    }
}
