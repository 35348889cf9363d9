// Large fp32 layers on the bf16 matrix cores (gfx950): the whole layer in one
// kernel, its fp32 GEMM operands split exactly into three bf16 terms.
//
// v_mfma_f32_16x16x4_f32 runs at 1/16 of the rate of v_mfma_f32_16x16x32_bf16.
// A fp32 value's 24 significand bits are exactly h + m + l, three bf16 values
// of 8 bits each (h and m cut off or rounded, l what is left).  u*v is then the
// sum of nine products, of which the six largest,
//     hh + hm + mh + hl + mm + lh,
// leave an error below 2^-21 |u v| (the dropped ml + lm + ll; about 2^-24 on
// average), no more than fp32 accumulation over the channels adds.  Six
// products at 16 times the rate are 2.67 times the fp32 matrix rate.
//
// Operand layout.  A reduction slot pair of the instruction (one dword of an
// operand) holds two terms of one channel, so 16 channels make one K = 32
// instruction: X = (m, h) and Y = (h, l) (low half first) of four consecutive
// channels are a lane's 16-byte operands, and three instructions give all six
// products:
//     X_u . X_v = mm + hh,   X_u . Y_v = mh + hl,   Y_u . X_v = hm + lh.
#include "wino_device.h"

namespace wino {

// ------------------------------------------------------------------ split U
// (X, Y) of one value as split3 gives them (for the inputs), but with h and m
// rounded to nearest (h only where that cannot overflow): m and l then have either
// sign, so that the dropped products of the filters' terms with an input's
// cut-off ones average out.
__device__ __forceinline__ void split3_rounded(float v, uint32_t& X, uint32_t& Y) {
    const uint32_t vb = __float_as_uint(v);
    const uint32_t hb = (vb & 0x7f800000u) < 0x7f000000u ? vb + 0x8000u : vb;
    const float r1 = v - __uint_as_float(hb & kHi16);               // exact
    const uint32_t rb = __float_as_uint(r1);
    const uint32_t mb = (rb & 0x7f800000u) < 0x7f000000u ? rb + 0x8000u : rb;
    const float r2 = r1 - __uint_as_float(mb & kHi16);              // exact, at most 8 bits
    X = __builtin_amdgcn_perm(hb, mb, 0x07060302u);
    Y = __builtin_amdgcn_perm(__float_as_uint(r2), hb, 0x07060302u);
}

// U [KB][CQ][T/4][64][4] fp32 -> US [KB][C16][T]{[64][16 bytes] X, [64][8
// bytes] l}: lane q*16 + k%16 of (kb, c16, t) holds channels c16*16 + 4q .. +3.
// The kernel puts Y together from l and X's high halves: the filters stream
// through L2 and L1 once per workgroup, so their bytes are what counts.
// Channels past C are zero (padding of U, or quads past CQ).  A thread does
// four positions.
__global__ __launch_bounds__(256) void k_usplit(const float* __restrict__ U, char* __restrict__ US, int CQ,
                                                int C16, int TG, long n) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int lane = (int)(i & 63), q = lane >> 4;
    const long w = i >> 6;                        // (kb * C16 + c16) * TG + tg
    const int tg = (int)(w % TG);
    const long kc = w / TG;
    const int c16 = (int)(kc % C16);
    const long kb = kc / C16;
    const int cq = c16 * 4 + q;
    f32x4 u[4];
#pragma unroll
    for (int d = 0; d < 4; ++d)
        u[d] = cq < CQ ? *(const f32x4*)(U + (((kb * CQ + cq) * TG + tg) * 64 + d * 16 + (lane & 15)) * 4)
                       : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t X[4], Y[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) split3_rounded(u[d][e] * kSplitScale, X[d], Y[d]);
        char* o = US + ((kc * TG + tg) * 4 + e) * kUsBytes;
        *(uint4*)(o + lane * 16) = make_uint4(X[0], X[1], X[2], X[3]);
        *(uint2*)(o + 1024 + lane * 8) = make_uint2(__builtin_amdgcn_perm(Y[1], Y[0], 0x07060302u),
                                                    __builtin_amdgcn_perm(Y[3], Y[2], 0x07060302u));
    }
}

// ------------------------------------------------------------------ the layer
// A workgroup of 8 waves (one per CU: 144 or 128 accumulators and 110 other
// registers per lane) owns 64 filters x 32 consecutive tiles (alpha = 6) or 64
// tiles (alpha = 4) at all T positions.  Per 16 channels:
//   - each wave transforms the regions of 16 tiles x 4 channels (x to registers,
//     loaded after the previous step's products), splits the T values and
//     writes them to LDS as MFMA operands (147 KB: one stage, so transforms and
//     products alternate between two barriers);
//   - wave (position quarter wp, filter half wf) multiplies 32 filters x all
//     tiles at its HN x HN quarter of the positions: with 32 x 32 products per
//     wave every LDS operand is read by two waves only, and each filter operand
//     by one wave, once for all tiles, straight to registers.
// What bounds it (timestamps, N = 64 256-channel 56x56 layer, cycles per step of
// 9600): products 6000 (3460 of MFMA issue; the address units are busy for 3460
// with the filters' 221 KB, 64 B a cycle, and about 1500 with x), transforms and
// splits 3400 (VALU and MFMA hardly overlap), barriers 600; per workgroup 9000
// before the first step and 13000 of epilogue.  What that measured on the way
// there (this layer): 8-byte filter elements (X and Y) 650 us, 6-byte ones 595,
// the outer region columns from the neighbouring lanes instead of by loads of
// their own 540.  2^16 in B^T and 2^-32 and the check in the epilogue cost 1-2%
// (582 -> 590, N = 32 64-channel 224x224 354 -> 363).
// Against fp32 MFMA kernels, both timed in turn: N = 32 64-channel 224x224 536 ->
// 375 us, N = 32 128-channel 112x112 417 -> 310, N = 64 256-channel 56x56 645 -> 560,
// N = 32 5x5 48 -> 64 at 35x35 50 -> 39.
template <int MT, int R>
struct Bf3Shape {
    static constexpr int A = MT + R - 1, T = A * A, HN = A / 2, NP = HN * HN, PAD = (R - 1) / 2;
    static constexpr int FB = 2, TB = A == 6 ? 2 : 4;        // 16-filter / 16-tile blocks of a wave
    static constexpr int KGW = 4;                            // filter blocks of a workgroup
    static constexpr int UN = TB * 4 / 8;                    // transform units of a wave per step
    static constexpr int VB = T * TB * 2048;                 // LDS bytes: X and Y of a 16-channel step
    static constexpr int D = NP % 3 == 0 ? 3 : 4;            // filter ring: positions in flight
    static constexpr int NC = FB * TB, OWN = NC / 4;         // (fb, tb) blocks of a wave; owned in the epilogue
    static constexpr int NO = MT * MT;
    static constexpr int RB = 2 * 4 * 3 * OWN * NO * 256;    // bytes one filter slot's exchange takes
    static constexpr int RS = VB / RB >= 4 ? 4 : VB / RB >= 2 ? 2 : 1;   // filter slots per exchange
    // Row of the last transform unit after which the ring's position p is loaded.
    static constexpr int ring_row(int p) { return D == 3 ? (p == 0 ? 2 : p == 1 ? 4 : 5) : p * A / D; }
    static_assert(NP % D == 0, "the ring wraps onto the next step's slots");
};

// B^T of 4 and of 6 points, 12 operations for the latter; SC: times kSplitScale
// (powers of two, so the rounding is the same), 2 or 3 operations more.
template <bool SC>
__device__ __forceinline__ void bf3_bt(const float (&a)[4], float (&r)[4]) {
    if constexpr (SC) {
        constexpr float S = kSplitScale;
        const float s1 = S * a[1], s2 = S * a[2];
        r[0] = __builtin_fmaf(S, a[0], -s2);
        r[1] = s1 + s2;
        r[2] = s2 - s1;
        r[3] = __builtin_fmaf(-S, a[3], s1);
    } else {
        bt_1d(a, r);
    }
}
template <bool SC>
__device__ __forceinline__ void bf3_bt(const float (&a)[6], float (&r)[6]) {
    constexpr float S = SC ? kSplitScale : 1.0f;
    const float s3 = S * a[3], s4 = S * a[4], s5 = S * a[5];
    const float d31 = __builtin_fmaf(-S, a[1], s3), d42 = __builtin_fmaf(-S, a[2], s4);
    const float p = __builtin_fmaf(-4.0f * S, a[2], s4), q = __builtin_fmaf(-4.0f * S, a[1], s3);
    r[0] = __builtin_fmaf(4.0f * S, a[0], __builtin_fmaf(-5.0f * S, a[2], s4));    //  4a0 - 5a2 + a4
    r[1] = p + q;                                                                  // -4a1 - 4a2 + a3 + a4
    r[2] = p - q;                                                                  //  4a1 - 4a2 - a3 + a4
    r[3] = __builtin_fmaf(2.0f, d31, d42);                                         // -2a1 - a2 + 2a3 + a4
    r[4] = __builtin_fmaf(-2.0f, d31, d42);                                        //  2a1 - a2 - 2a3 + a4
    r[5] = __builtin_fmaf(4.0f * S, a[1], __builtin_fmaf(-5.0f * S, a[3], s5));    //  4a1 - 5a3 + a5
}

template <int MT, int R, bool RAG>
__global__ __launch_bounds__(512) void k_bf3(const float* __restrict__ x, const char* __restrict__ US,
                                             const float* __restrict__ U, float* __restrict__ y, Geom g,
                                             FusedTiling ft, int relu, int vec_ok, int nts) {
    using S = Bf3Shape<MT, R>;
    constexpr int A = S::A, T = S::T, HN = S::HN, NP = S::NP, FB = S::FB, TB = S::TB, D = S::D, UN = S::UN, PAD = S::PAD;
    __shared__ uint4 vs[S::VB / 16];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int item = (blockIdx.x & 7) * ft.per + (blockIdx.x >> 3);
    if (item >= ft.nt * ft.nkg) return;
    const int kgi = item % ft.nkg, tp = item / ft.nkg;      // filter group fastest
    const int wp = wave & 3, wf = wave >> 2;
    const int nsteps = ft.nsteps;

    // ---- transform units: unit id = wave + 8j is (tile block id % TB, quad id / TB)
    const int utb = wave % TB, uq0 = wave / TB;
    const int p0 = (tp * TB + utb) * 16;
    const TileCoord tc = decode_tile(p0 + (lane & 15), g);
    const int cl = lane >> 4;
    const int n0 = __builtin_amdgcn_readfirstlane(min(p0, g.P - 1) / (g.th * g.tw));
    // x as a buffer that starts pad rows before image n0, so that a region's
    // offsets count from its first row: row u is a uniform u * W further, and a
    // lane needs one offset.  Rows outside the image and channels past C take
    // an offset past the buffer's end, which reads as zero; the others lie
    // inside x.
    const size_t img = (size_t)g.C * g.H * g.W;
    const int64_t left = (int64_t)(((size_t)g.N - n0) * img + (size_t)PAD * g.W) * 4;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(x + (size_t)n0 * img - (size_t)PAD * g.W), (short)0,
        (int)(left < (int64_t)kInvalid ? left : (int64_t)kInvalid), kRsrcWord3);
    const uint32_t plane_b = (uint32_t)g.H * g.W * 4;
    const uint32_t reg0 = ((uint32_t)(tc.n - n0) * g.C + cl) * plane_b + ((uint32_t)tc.ti * g.W + tc.tj) * (MT * 4);
    bool rv[A];
#pragma unroll
    for (int u = 0; u < A; ++u) {
        const int rr = tc.ti * MT - PAD + u;
        rv[u] = tc.valid && rr >= 0 && rr < g.H;
    }
    // A lane loads the MT middle columns of its region (the tile's own); the
    // PAD columns to either side are middle columns of the neighbouring tiles,
    // in the neighbouring lanes, except at the ends of the 16 tiles: lane 0
    // loads its left columns, lane 15 its right ones.  Loads cost more than
    // these moves: the filters keep the address units busy.
    const bool has_l = tc.tj > 0 && tc.valid, has_r = tc.tj + 1 < g.tw && tc.valid;
    const int e16 = lane & 15;
    const bool eok = (e16 == 0 && has_l) || (e16 == 15 && has_r);
    const uint32_t edge0 = e16 == 15 ? reg0 + MT * 4 : reg0 - PAD * 4;
    bool cv[MT];                                    // RAG: the tile's columns inside the image
#pragma unroll
    for (int v = 0; v < MT; ++v) cv[v] = tc.tj * MT + v < g.W;
    const bool ev = tc.tj * MT + MT + 1 < g.W || e16 != 15;    // RAG, PAD = 2: lane 15's second column
    typedef float fm __attribute__((ext_vector_type(MT)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    fm dm[UN][A];                                   // middle columns
    float de[UN][A][PAD];                           // lanes 0 and 15: their outer columns
    // Load n of the NX loads of step s's regions: row by row, middle and edge.
    constexpr int NX = UN * A * 2;
    auto load_x = [&](int s, auto nc) {
        constexpr int n = decltype(nc)::value, j = n / (A * 2), u = n / 2 % A;
        const int c0 = s * 16 + (uq0 + j * (8 / TB)) * 4;
        const bool ok = rv[u] && c0 + cl < g.C;
        const int so = __builtin_amdgcn_readfirstlane(c0 * (int)plane_b + u * g.W * 4);
        if constexpr (n % 2 == 0) {
            const int o = (int)(ok ? reg0 : kInvalid);
            if constexpr (MT == 4) dm[j][u] = __builtin_bit_cast(fm, __builtin_amdgcn_raw_buffer_load_b128(xr, o, so, 0));
            else dm[j][u] = __builtin_bit_cast(fm, __builtin_amdgcn_raw_buffer_load_b64(xr, o, so, 0));
        } else {
            const int o = (int)(ok && eok ? edge0 : kInvalid);
            if constexpr (PAD == 1) {
                de[j][u][0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, o, so, 0));
            } else {
                const f32x2 q = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(xr, o, so, 0));
                de[j][u][0] = q[0];
                de[j][u][1] = q[1];
            }
        }
    };
    // Row u of unit j's region from the loaded columns.
    auto region_row = [&](int j, int u, float (&r)[A]) {
        float m[MT], e[PAD];
#pragma unroll
        for (int v = 0; v < MT; ++v) m[v] = !RAG || cv[v] ? dm[j][u][v] : 0.0f;
#pragma unroll
        for (int v = 0; v < PAD; ++v) e[v] = !RAG || v == 0 || ev ? de[j][u][v] : 0.0f;
        auto dpp = [](float old, float v, auto ctrl) {
            return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(old), __float_as_uint(v),
                                                               decltype(ctrl)::value, 0xf, 0xf, false));
        };
#pragma unroll
        for (int v = 0; v < PAD; ++v) {
            const float l = dpp(e[v], m[MT - PAD + v], IC<0x111>{});       // row_shr:1: from lane - 1
            const float h = dpp(e[v], m[v], IC<0x101>{});                  // row_shl:1: from lane + 1
            r[v] = has_l ? l : 0.0f;
            r[PAD + MT + v] = has_r ? h : 0.0f;
        }
#pragma unroll
        for (int v = 0; v < MT; ++v) r[PAD + v] = m[v];
    };
    // Transform and split unit j and write it to LDS [t][tb][X|Y][64 lanes][16
    // bytes]: lane (tile i, channel quad*4 + d) writes dword d of lane quad*16 + i.
    uint32_t* const vdst = (uint32_t*)vs + utb * 512 + (lane & 15) * 4 + cl;
    // after_row(u) runs after row u (the next step's filter loads go there, into
    // the registers that the finished rows free).
    auto transform = [&](int j, auto&& after_row) {
        float d[A][A], t1[A][A];
#pragma unroll
        for (int u = 0; u < A; ++u) region_row(j, u, d[u]);
#pragma unroll
        for (int v = 0; v < A; ++v) {
            float c[A], r[A];
#pragma unroll
            for (int u = 0; u < A; ++u) c[u] = d[u][v];
            bf3_bt<true>(c, r);
#pragma unroll
            for (int u = 0; u < A; ++u) t1[u][v] = r[u];
        }
        uint32_t* const o = vdst + (uq0 + j * (8 / TB)) * 64;
#pragma unroll
        for (int u = 0; u < A; ++u) {
            float r[A];
            bf3_bt<false>(t1[u], r);
#pragma unroll
            for (int v = 0; v < A; ++v) {
                uint32_t X, Y;
                split3(r[v], X, Y);
                o[(u * A + v) * TB * 512] = X;
                o[(u * A + v) * TB * 512 + 256] = Y;
            }
            after_row(u);
        }
    };

    // ---- filters: ring of D positions of FB blocks, X and Y
    const size_t us_b = (size_t)g.KB * nsteps * T * kUsBytes;
    const __amdgpu_buffer_rsrc_t ur = __builtin_amdgcn_make_buffer_rsrc(
        (void*)US, (short)0, (int)(us_b < 0x7fffffffu ? us_b : 0x7fffffffu), kRsrcWord3);
    const uint32_t l16 = (uint32_t)lane * 16u;
    const int t0 = (wp >> 1) * HN * A + (wp & 1) * HN;      // first position of this wave's HN x HN quarter
    uint32_t ub[FB];
#pragma unroll
    for (int f = 0; f < FB; ++f) {
        const int kb = min(kgi * S::KGW + wf * FB + f, g.KB - 1);
        ub[f] = __builtin_amdgcn_readfirstlane(((uint32_t)kb * nsteps * T + t0) * kUsBytes);
    }
    const uint32_t l8 = 1024u + (uint32_t)lane * 8u;
    uint4 uX[D][FB];
    uint2 uL[D][FB];
    // load k (X, l of filter block k / 2) of position p of step s
    auto load_u1 = [&](int s, auto pc, auto kc) {
        constexpr int p = decltype(pc)::value, pt = (p / HN) * A + p % HN, k = decltype(kc)::value, f = k / 2;
        const int so = (int)(ub[f] + (uint32_t)s * T * kUsBytes) + pt * kUsBytes;
        if constexpr (k % 2 == 0)
            uX[p % D][f] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ur, (int)l16, so, 0));
        else
            uL[p % D][f] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(ur, (int)l8, so, 0));
    };
    auto load_u = [&](int s, auto pc) { static_for<0, 2 * FB>([&](auto kc) { load_u1(s, pc, kc); }); };

    f32x4 acc[FB][TB][NP];
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int p = 0; p < NP; ++p) acc[f][b][p] = f32x4{0.f, 0.f, 0.f, 0.f};

    const uint4* const vsrc = vs + t0 * TB * 128 + lane;
    static_for<0, NX>([&](auto nc) { load_x(0, nc); });
    // Transform the loaded regions, and load the ring's first filters of step s.
    auto transform_all = [&](int s) {
#pragma unroll
        for (int j = 0; j < UN; ++j)
            transform(j, [&](int u) {
                if (j + 1 < UN) return;
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, D>([&](auto pc) {
                    constexpr int p = decltype(pc)::value;
                    if (u == S::ring_row(p)) load_u(s, pc);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
    };
    transform_all(0);
    wait_vm_lds<63>();
    wg_barrier();
    for (int s = 0; s < nsteps; ++s) {
        const bool more = s + 1 < nsteps;
        // groups (position, tile block) in order, each group's V one group ahead
        uint4 vX[2], vY[2];
        auto load_v = [&](auto ic) {
            constexpr int i = decltype(ic)::value, p = i / TB, pt = (p / HN) * A + p % HN;
            vX[i & 1] = vsrc[(pt * TB + i % TB) * 128];
            vY[i & 1] = vsrc[(pt * TB + i % TB) * 128 + 64];
        };
        uint4 uY[FB];
        // The filters that take position p-1's place in the ring load one at a time
        // between the products of position p (four at once held a wave at issue
        // for 250-480 cycles).
        auto slot = [&](auto pc, auto kc) {
            constexpr int p = decltype(pc)::value, k = decltype(kc)::value, NS = 3 * TB;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (p >= 1 && p - 1 + D < NP && k * 2 * FB / NS < (k + 1) * 2 * FB / NS)
                load_u1(s, IC<p - 1 + D>{}, IC<k * 2 * FB / NS>{});
            __builtin_amdgcn_sched_barrier(0);
        };
        load_v(IC<0>{});
        static_for<0, NP * TB>([&](auto ic) {
            constexpr int i = decltype(ic)::value, p = i / TB, b = i % TB;
            if constexpr (i + 1 < NP * TB) load_v(IC<i + 1>{});
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < FB; ++f) acc[f][b][p] = mfma16x16x32<2>(uX[p % D][f], vY[i & 1], acc[f][b][p]);
            if constexpr (b == 0) {
#pragma unroll
                for (int f = 0; f < FB; ++f) {
                    uY[f] = us_y(uX[p % D][f], uL[p % D][f]);
                }
            }
            slot(IC<p>{}, IC<3 * b>{});
#pragma unroll
            for (int f = 0; f < FB; ++f) acc[f][b][p] = mfma16x16x32<2>(uY[f], vX[i & 1], acc[f][b][p]);
            slot(IC<p>{}, IC<3 * b + 1>{});
#pragma unroll
            for (int f = 0; f < FB; ++f) acc[f][b][p] = mfma16x16x32<2>(uX[p % D][f], vX[i & 1], acc[f][b][p]);
            slot(IC<p>{}, IC<3 * b + 2>{});
        });
        if (more) {
            // Not between the products: loads return in order, so the filters' waits
            // would wait for x from HBM too (N = 64 256-channel 56x56 layer 705
            // against 596 us).
            static_for<0, NX>([&](auto nc) { load_x(s + 1, nc); });
            wait_vm_lds<63>();
            wg_barrier();                          // every wave is done with this step's V
            __builtin_amdgcn_sched_barrier(0);
            transform_all(s + 1);
            wait_vm_lds<63>();
            wg_barrier();                          // the next step's V is written
        }
    }

    // ---- epilogue: this wave's part of A^T M A from its HN x HN quarter of
    // the positions; the four quarters of a (fb, tb) block are summed through
    // LDS, RS filter slots at a time; wave wp owns blocks wp*OWN .. +OWN-1.
    constexpr int OWN = S::OWN, NO = S::NO, RS = S::RS;
    const bool rl = relu != 0, vo = vec_ok != 0;
    TileCoord ot[OWN];
#pragma unroll
    for (int c = 0; c < OWN; ++c) ot[c] = decode_tile((tp * TB + (wp * OWN + c) % TB) * 16 + (lane & 15), g);
    float* const ex = (float*)vs;
    float chk[OWN] = {};                           // NaN once an output of the block is not finite
    auto slot = [&](int owner, int idx, int c, int rr) -> float* {
        return ex + (((((wf * 4 + owner) * 3 + idx) * OWN + c) * RS + rr) * NO) * 64;
    };
#pragma unroll
    for (int r0 = 0; r0 < 4; r0 += RS) {
        __syncthreads();                           // V, or the last slots' exchange, is consumed
        float own[RS][OWN][MT][MT];
        auto part = [&](auto wc) {
            constexpr int W = decltype(wc)::value, X0 = (W >> 1) * HN, N0 = (W & 1) * HN;
#pragma unroll
            for (int rr = 0; rr < RS; ++rr)
#pragma unroll
                for (int c = 0; c < S::NC; ++c) {
                    float h[MT][HN];
#pragma unroll
                    for (int v = 0; v < HN; ++v) {
                        float a[HN], r[MT];
#pragma unroll
                        for (int u = 0; u < HN; ++u) a[u] = acc[c / TB][c % TB][u * HN + v][r0 + rr];
                        AtRows<MT, X0, HN>::f(a, r);
#pragma unroll
                        for (int i = 0; i < MT; ++i) h[i][v] = r[i];
                    }
                    float o[MT][MT];
#pragma unroll
                    for (int i = 0; i < MT; ++i) AtRows<MT, N0, HN>::f(h[i], o[i]);
                    if (c / OWN == W) {
#pragma unroll
                        for (int i = 0; i < MT; ++i)
#pragma unroll
                            for (int k = 0; k < MT; ++k) own[rr][c % OWN][i][k] = o[i][k];
                    } else {
                        float* e = slot(c / OWN, (W - c / OWN + 3) & 3, c % OWN, rr) + lane * 4;
#pragma unroll
                        for (int k = 0; k < NO / 4; ++k)
                            *(f32x4*)(e + k * 256) = f32x4{o[(4 * k) / MT][(4 * k) % MT], o[(4 * k + 1) / MT][(4 * k + 1) % MT],
                                                           o[(4 * k + 2) / MT][(4 * k + 2) % MT], o[(4 * k + 3) / MT][(4 * k + 3) % MT]};
                    }
                }
        };
        with_ic(wp, part, std::make_integer_sequence<int, 4>{});
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < RS; ++rr)
#pragma unroll
            for (int c = 0; c < OWN; ++c) {
                float o[MT][MT];
#pragma unroll
                for (int k = 0; k < NO / 4; ++k) {
                    f32x4 q = {own[rr][c][(4 * k) / MT][(4 * k) % MT], own[rr][c][(4 * k + 1) / MT][(4 * k + 1) % MT],
                               own[rr][c][(4 * k + 2) / MT][(4 * k + 2) % MT], own[rr][c][(4 * k + 3) / MT][(4 * k + 3) % MT]};
#pragma unroll
                    for (int i = 0; i < 3; ++i) q += *(const f32x4*)(slot(wp, i, c, rr) + lane * 4 + k * 256);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[(4 * k + e) / MT][(4 * k + e) % MT] = q[e] * kSumScale;
                }
#pragma unroll
                for (int i = 0; i < NO; ++i) chk[c] = __builtin_fmaf(o[i / MT][i % MT], 0.0f, chk[c]);
                const int k = (kgi * S::KGW + wf * FB + (wp * OWN + c) / TB) * 16 + 4 * cl + r0 + rr;
                if (nts) store_block<MT, true>(y, g, ot[c], k, o, rl, vo);
                else store_block<MT, false>(y, g, ot[c], k, o, rl, vo);
            }
    }
    // An operand that is infinite or NaN has no split: every result it enters is
    // NaN here.  Such blocks (and those whose sums overflow) run once more on
    // fp32 MFMA, which gives the infinities and NaNs of the other kernels.
#pragma unroll 1
    for (int c = 0; c < OWN; ++c) {
        const int b = wp * OWN + c, kb = kgi * S::KGW + wf * FB + b / TB;
        if (kb >= g.KB || !__any(OWN == 1 || c == 0 ? chk[0] != chk[0] : chk[OWN - 1] != chk[OWN - 1])) continue;
        const int q0 = (tp * TB + b % TB) * 16;
        const TileCoord qt = decode_tile(q0 + (lane & 15), g);
        f32x4 m[T];
        fp32_products<MT, R>(x, U, g, q0, kb, lane, m);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float m1[T], o[MT][MT];
#pragma unroll
            for (int t = 0; t < T; ++t) m1[t] = m[t][r];
            output_tf<MT, R>(m1, o);
            store_block<MT, false>(y, g, qt, kb * 16 + 4 * cl + r, o, rl, vo);
        }
    }
}

// ------------------------------------------------------------------ host
hipError_t launch_usplit(const float* U, void* US, const Geom& g, hipStream_t s) {
    const int c16 = (g.CQ + 3) / 4, tg = g.T / 4;
    const long n = (long)g.KB * c16 * tg * 64;
    if ((n + 255) / 256 > 0x7fffffffL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_usplit, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, U, (char*)US, g.CQ, c16, tg, n);
    return hipGetLastError();
}

size_t bf3_workspace(const Geom& g) { return us_bytes(g); }

long bf3_items(const Geom& g) {
    const long nb = ((long)g.P + 15) / 16, tb = g.A == 6 ? 2 : 4;
    return (nb + tb - 1) / tb * ((g.KB + 3) / 4);
}

bool bf3_takes(const Geom& g) {
    // NCHW "same" layers: the neighbouring lanes hold a region's outer columns
    if (g.nhwc || g.axis != 0 || g.pad != (g.r - 1) / 2) return false;
    // 32-bit offsets: into x over the images that 16 tiles span (channels past
    // C, up to two steps on, add theirs to kInvalidOffset), and into the filters
    const int64_t span = 16 / ((int64_t)g.th * g.tw) + 2, plane_b = (int64_t)g.H * g.W * 4;
    const int64_t c16 = (g.CQ + 3) / 4;
    if (span * g.C * plane_b + 2 * g.pad * (int64_t)g.W * 4 >= (int64_t)kInvalidOffset) return false;
    if ((int64_t)kInvalidOffset + (c16 + 2) * 16 * plane_b + 8 * (int64_t)g.W * 4 >= ((int64_t)1 << 32)) return false;
    return bf3_workspace(g) <= 0x7fffffffu && bf3_items(g) < (1L << 28);
}

// One workgroup per CU: rounds of a fixed part (first loads and transform,
// exchange, stores) and the 16-channel steps, as measured (F(4x4): 7 rounds of
// 16 steps 560 us, 13 of 4 375 us; F(2x2,5x5): two of 3 39 us; F(2x2): one of
// 32 steps 121 us), after the filters' split.  889 layers took 84-112% of it in 90
// of 100.
double bf3_ns(const Geom& g) {
    const double steps = (g.CQ + 3) / 4, rounds = (double)((bf3_items(g) + 255) / 256);
    const double split = 3000.0 + 10.0 * 256.0 * g.T * g.KB * steps / 5000.0;
    return split + rounds * (g.A == 6 ? (g.r == 5 ? 7500.0 : 10800.0) + 4100.0 * steps : 7700.0 + 3500.0 * steps);
}

template <int MT, int R>
static hipError_t bf3_instance(const float* x, const float* U, float* y, void* ws, const Geom& g, bool relu,
                               hipStream_t s) {
    using S = Bf3Shape<MT, R>;
    const int c16 = (g.CQ + 3) / 4;
    const hipError_t e = launch_usplit(U, ws, g, s);
    if (e != hipSuccess) return e;
    FusedTiling ft{};
    const int nb = (int)(((long)g.P + 15) / 16);
    ft.nt = (nb + S::TB - 1) / S::TB;
    ft.nkg = (g.KB + S::KGW - 1) / S::KGW;
    ft.per = (int)(((long)ft.nt * ft.nkg + 7) / 8);
    ft.nsteps = c16;
    const dim3 grid((unsigned)(8 * ft.per)), block(512);
    const int vec_ok = (g.Wo % MT == 0) && aligned(y, 4 * MT);
    if (g.W % MT == 0)
        hipLaunchKernelGGL((k_bf3<MT, R, false>), grid, block, 0, s, x, (const char*)ws, U, y, g, ft, (int)relu, vec_ok,
                           split_stream_stores(g));
    else
        hipLaunchKernelGGL((k_bf3<MT, R, true>), grid, block, 0, s, x, (const char*)ws, U, y, g, ft, (int)relu, vec_ok,
                           split_stream_stores(g));
    return hipGetLastError();
}

hipError_t launch_bf3(const float* x, const float* U, float* y, void* ws, const Geom& g, bool relu, hipStream_t s) {
    if (g.r == 5) return g.m == 2 ? bf3_instance<2, 5>(x, U, y, ws, g, relu, s) : hipErrorInvalidValue;
    if (g.r != 3) return hipErrorInvalidValue;
    if (g.m == 2) return bf3_instance<2, 3>(x, U, y, ws, g, relu, s);
    if (g.m == 4) return bf3_instance<4, 3>(x, U, y, ws, g, relu, s);
    return hipErrorInvalidValue;
}

}  // namespace wino
