// The T per-position GEMMs, M_t = U_t^T V_t, of large fp32 layers on the bf16
// matrix cores (gfx950): U and V as words of three bf16 terms in memory (the
// filters' split and the input transforms write them), the six largest products
// summed by v_mfma_f32_16x16x32_bf16 (wino_bf3.hip says why that is as exact as
// fp32 products, and how X and Y operands give six products in three
// instructions), M in fp32.
#include "wino_device.h"

namespace wino {

// A workgroup of 8 waves owns four positions x 128 filters x 128 tiles; wave
// (position, filter half) multiplies 64 filters x 128 tiles at its position
// (128 accumulators a lane).  A step is 16 channels: V comes by DMA into a ring
// of three 48 KB LDS stages, two steps ahead, one barrier a step; a wave's
// filters (no other wave uses them) straight to registers, one step ahead.
// V is split in memory and not here because vector and matrix instructions of
// a SIMD hardly overlap: splitting V's fp32 words on the way into LDS cost as
// much as the products (step of this size 4800 cycles, 2200 of them products).
// The layer, against the split algorithm on fp32 MFMA, both timed in turn: N = 32
// 512-channel 14x14 F(2x2) 140 -> 104 us, N = 32 512-channel 28x28 F(4x4) 328 -> 250;
// channel-last N = 16 456 -> 512 at 28x28 against the three stages 160 -> 126.
constexpr int kG3K = 8, kG3P = 8;                      // filter and tile blocks of a workgroup

// B^T of 4 and of 6 points by rows.
__device__ const float kBt4[4][4] = {{1, 0, -1, 0}, {0, 1, 1, 0}, {0, -1, 1, 0}, {0, 1, 0, -1}};
__device__ const float kBt6[6][6] = {{4, 0, -5, 0, 1, 0}, {0, -4, -4, 1, 1, 0}, {0, 4, -4, -1, 1, 0},
                                     {0, -2, -1, 2, 1, 0}, {0, 2, -1, -2, 1, 0}, {0, 4, 0, -5, 0, 1}};

// M of (tile block pb, filter blocks kb .. kb+FB-1) at position t on fp32 MFMA,
// straight from x and U.  Only the region elements that B^T weighs are read: a
// zero times an infinity would be NaN.
template <int FB>
__device__ __forceinline__ void fp32_position(const float* __restrict__ x, const float* __restrict__ U, const Geom& g,
                                              int pb, int kb, int t, int lane, float* __restrict__ M) {
    const int A = g.A, xi = t / A, nu = t % A, cl = lane >> 4;
    const float* const bx = A == 4 ? kBt4[xi] : kBt6[xi];
    const float* const bn = A == 4 ? kBt4[nu] : kBt6[nu];
    const TileCoord tc = decode_tile(pb * 16 + (lane & 15), g);
    const int r0 = tc.ti * g.m - g.pad, c0 = tc.tj * g.m - g.pad;
    const size_t chan = g.nhwc ? 1 : (size_t)g.H * g.W, pix = g.nhwc ? g.C : 1;
    f32x4 acc[FB];
#pragma unroll
    for (int f = 0; f < FB; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int cq = 0; cq < g.CQ; ++cq) {
        const int c = cq * 4 + cl;
        const bool ok = tc.valid && c < g.C;
        const float* const xc = x + (size_t)tc.n * g.C * g.H * g.W + (ok ? c : 0) * chan;
        float v = 0.0f;
        for (int i = 0; i < A; ++i) {
            if (bx[i] == 0.0f) continue;
            float s = 0.0f;
            for (int j = 0; j < A; ++j) {
                if (bn[j] == 0.0f) continue;
                const int row = r0 + i, col = c0 + j;
                const bool in = ok && (unsigned)row < (unsigned)g.H && (unsigned)col < (unsigned)g.W;
                s = __builtin_fmaf(bn[j], in ? xc[((size_t)row * g.W + col) * pix] : 0.0f, s);
            }
            v = __builtin_fmaf(bx[i], s, v);
        }
#pragma unroll
        for (int f = 0; f < FB; ++f) {
            const size_t k = min(kb + f, g.KB - 1);
            acc[f] = mfma16x16x4(U[(((k * g.CQ + cq) * (g.T / 4) + t / 4) * 64 + lane) * 4 + t % 4], v, acc[f]);
        }
    }
#pragma unroll
    for (int f = 0; f < FB; ++f)
        if (kb + f < g.KB) *(f32x4*)(M + (((size_t)pb * g.KB + kb + f) * g.T + t) * 256 + lane * 4) = acc[f];
}

__global__ __launch_bounds__(512) void k_gemm3(const char* __restrict__ US, const char* __restrict__ V3,
                                               const float* __restrict__ x, const float* __restrict__ U,
                                               float* __restrict__ M, Geom g) {
    constexpr int FB = kG3K / 2, PB = kG3P, BLK = 4 * kUsBytes;   // BLK: a tile block's four positions
    __shared__ uint4 st0[PB * BLK / 16], st1[PB * BLK / 16], st2[PB * BLK / 16];
    const int T = g.T, TG = T / 4;
    const int nkg = (g.KB + kG3K - 1) / kG3K, npg = (g.PB + PB - 1) / PB;
    // Items (position group, tile group, filter group), filter group fastest,
    // each XCD a contiguous range: a position group's U stays in its L2, and
    // the filter groups that share V run together.
    const long nitems = (long)TG * npg * nkg, per = (nitems + 7) / 8;
    const long item = (long)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (item >= nitems) return;
    const int kb0 = (int)(item % nkg) * kG3K;
    const long rest = item / nkg;
    const int pb0 = (int)(rest % npg) * PB, tg = (int)(rest / npg);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int we = wave & 3, kbw = kb0 + (wave >> 2) * FB;
    const int nsteps = (g.CQ + 3) / 4;

    // V: wave w brings tile block w's four positions of a step, 6 KB in six
    // loads (blocks past P and steps past the last read zero).
    const uint32_t vstride = (uint32_t)nsteps * T * kUsBytes;
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(V3 + (size_t)pb0 * vstride), (short)0, (int)((uint32_t)min(g.PB - pb0, PB) * vstride), kRsrcWord3);
    const uint32_t l16 = (uint32_t)lane * 16u;
    auto stage = [&](auto rc) -> uint4* {
        constexpr int R = decltype(rc)::value % 3;
        if constexpr (R == 0) return st0;
        else if constexpr (R == 1) return st1;
        else return st2;
    };
    auto load_v = [&](auto rc, int s, auto ic) {
        constexpr int i = decltype(ic)::value;
        const uint32_t so = __builtin_amdgcn_readfirstlane((uint32_t)wave * vstride + ((uint32_t)s * T + tg * 4) * kUsBytes + i * 1024u);
        lds_dma<16>(vr, (float*)(stage(rc) + wave * (BLK / 16) + i * 64), s < nsteps ? l16 : 0x80000000u, so);
    };
    // The filters of position tg*4 + we: X and l of FB blocks.
    const size_t us_b = (size_t)g.KB * vstride;
    const __amdgpu_buffer_rsrc_t ur = __builtin_amdgcn_make_buffer_rsrc(
        (void*)US, (short)0, (int)(us_b < 0x7fffffffu ? us_b : 0x7fffffffu), kRsrcWord3);
    uint4 aX[2][FB], aY[FB];                           // sets of even and odd steps
    uint2 aL[2][FB];
    auto load_u = [&](int s, auto rc, auto kc) {       // load k of 2*FB: X, l of block k / 2
        constexpr int R = decltype(rc)::value % 2, k = decltype(kc)::value, f = k / 2;
        const int kb = min(kbw + f, g.KB - 1);
        const int so = __builtin_amdgcn_readfirstlane(
            (((uint32_t)kb * nsteps + min(s, nsteps - 1)) * T + tg * 4 + we) * kUsBytes);
        if constexpr (k % 2 == 0)
            aX[R][f] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ur, (int)l16, so, 0));
        else
            aL[R][f] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(ur, 1024 + lane * 8, so, 0));
    };

    f32x4 acc[FB][PB];
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int b = 0; b < PB; ++b) acc[f][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    static_for<0, 6>([&](auto ic) { load_v(IC<0>{}, 0, ic); });
    static_for<0, 6>([&](auto ic) { load_v(IC<1>{}, 1, ic); });
    static_for<0, 2 * FB>([&](auto kc) { load_u(0, IC<0>{}, kc); });
    // A step issues 2*FB filter loads and then six V loads (in that order,
    // between the products), so V of step s, which step s-2 asked for last, has
    // landed when at most the 2*FB + 6 loads of step s-1 are outstanding.
    constexpr int WAITN = 6 + 2 * FB;
    auto step = [&](auto rc, int s) {                  // s % 6 == R
        constexpr int R = decltype(rc)::value;
        wait_vm_lds<WAITN>();
        wg_barrier();                                  // the step's V is in LDS; the step before is done
        const char* sv = (const char*)stage(rc) + we * kUsBytes;
        uint4 bX[2];
        uint2 bL[2];
        bX[0] = *(const uint4*)(sv + lane * 16);
        bL[0] = *(const uint2*)(sv + 1024 + lane * 8);
#pragma unroll
        for (int f = 0; f < FB; ++f) aY[f] = us_y(aX[R % 2][f], aL[R % 2][f]);
        auto slot = [&](auto kc) {
            constexpr int k = decltype(kc)::value;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (k < 2 * FB) load_u(s + 1, IC<R + 1>{}, IC<k>{});
            else if constexpr (k - 2 * FB < 6) load_v(IC<R + 2>{}, s + 2, IC<k - 2 * FB>{});
            __builtin_amdgcn_sched_barrier(0);
        };
        static_for<0, PB>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            if constexpr (b + 1 < PB) {
                bX[(b + 1) & 1] = *(const uint4*)(sv + (b + 1) * BLK + lane * 16);
                bL[(b + 1) & 1] = *(const uint2*)(sv + (b + 1) * BLK + 1024 + lane * 8);
            }
            __builtin_amdgcn_sched_barrier(0);
            const uint4 bY = us_y(bX[b & 1], bL[b & 1]);
#pragma unroll
            for (int f = 0; f < FB; ++f) acc[f][b] = mfma16x16x32<2>(aX[R % 2][f], bY, acc[f][b]);
            slot(IC<3 * b>{});
#pragma unroll
            for (int f = 0; f < FB; ++f) acc[f][b] = mfma16x16x32<2>(aY[f], bX[b & 1], acc[f][b]);
            slot(IC<3 * b + 1>{});
#pragma unroll
            for (int f = 0; f < FB; ++f) acc[f][b] = mfma16x16x32<2>(aX[R % 2][f], bX[b & 1], acc[f][b]);
            slot(IC<3 * b + 2>{});
        });
    };
    for (int s = 0; s < nsteps; s += 6) {
        step(IC<0>{}, s);
        if (s + 1 < nsteps) step(IC<1>{}, s + 1);
        if (s + 2 < nsteps) step(IC<2>{}, s + 2);
        if (s + 3 < nsteps) step(IC<3>{}, s + 3);
        if (s + 4 < nsteps) step(IC<4>{}, s + 4);
        if (s + 5 < nsteps) step(IC<5>{}, s + 5);
    }
    __builtin_amdgcn_s_waitcnt(0);                     // no load outlives the loop
    uint32_t redo = 0;                                 // bit b: a product of tile block b is not finite
#pragma unroll
    for (int b = 0; b < PB; ++b) {
        float chk = 0.0f;                              // NaN once a product is not finite
#pragma unroll
        for (int f = 0; f < FB; ++f) {
#pragma unroll
            for (int r = 0; r < 4; ++r) chk = __builtin_fmaf(acc[f][b][r], 0.0f, chk);
            if (kbw + f < g.KB && pb0 + b < g.PB)
                *(f32x4*)(M + (((size_t)(pb0 + b) * g.KB + kbw + f) * T + tg * 4 + we) * 256 + lane * 4) = acc[f][b] * kSumScale;
        }
        if (__any(chk != chk)) redo |= 1u << b;
    }
    // An operand that is infinite or NaN has no split: every product it enters is
    // NaN here.  Such tile blocks (and those whose sums overflow) run once more
    // on fp32 MFMA, straight from x and U, which gives the other kernels'
    // infinities and NaNs.
#pragma unroll 1
    for (; redo; redo &= redo - 1) {
        const int pb = pb0 + __builtin_ctz(redo);
        if (pb < g.PB) fp32_position<FB>(x, U, g, pb, kbw, tg * 4 + we, lane, M);
    }
}

// Bytes of the split filters and of the split transformed input: the layer's K,
// P and C in whole blocks and steps.
size_t us_bytes(const Geom& g) { return (size_t)g.KB * ((g.CQ + 3) / 4) * g.T * kUsBytes; }
size_t v3_bytes(const Geom& g) { return (size_t)g.PB * ((g.CQ + 3) / 4) * g.T * kUsBytes; }

bool gemm3_takes(const Geom& g) {
    // 32-bit offsets into the filters and into eight tile blocks (two steps past C)
    return us_bytes(g) <= 0x7fffffffu && (size_t)kG3P * ((g.CQ + 3) / 4 + 2) * g.T * kUsBytes < 0x7fffffffu;
}

long gemm3_items(const Geom& g) {
    return (long)(g.T / 4) * ((g.PB + kG3P - 1) / kG3P) * ((g.KB + kG3K - 1) / kG3K);
}

hipError_t launch_gemm3(const void* US, const void* V3, const float* x, const float* U, float* M, const Geom& g,
                        hipStream_t s) {
    const long wgs = (gemm3_items(g) + 7) / 8 * 8;
    if (wgs > 0x7fffffffL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_gemm3, dim3((unsigned)wgs), dim3(512), 0, s, (const char*)US, (const char*)V3, x, U, M, g);
    return hipGetLastError();
}

}  // namespace wino
