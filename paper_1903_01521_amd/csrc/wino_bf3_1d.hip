// 1-D fp32 layers (1 x r and r x 1 filters, T = 8) in one kernel on the bf16
// matrix cores (gfx950), their operands split exactly into three bf16 terms
// (wino_bf3.hip says why that is as exact as fp32 products).
#include "wino_device.h"

namespace wino {

// A workgroup of four waves, two workgroups per CU, owns 32 consecutive tiles x
// up to 128 filters at all 8 positions; wave w multiplies 32 filters x the 32
// tiles (128 accumulators a lane), so a wave holds every position of its
// (filter, tile) pairs and the output transform needs no exchange.  Per 16
// channels a wave transforms and splits two units of 16 tiles x 4 channels into
// one of two 32 KB LDS stages while the other is multiplied: one barrier a step.
// Each filter operand is read by one wave, once for all tiles, straight to
// registers, four positions ahead.
// What bounds it: a step of two workgroups takes about 4 us, of which products
// 1.3 us, transforms, splits and operand words about 1 us (VALU and MFMA hardly
// overlap), filters (96 KB a workgroup) 1.3 us of the address units.  One
// workgroup per CU with the filters eight positions ahead was slower at every
// size (its accumulators move between the two register files: 39 -> 68 us on
// the first layer below), and so was one with 64 tiles (99 us).  Two 16-byte
// loads of the 8 inputs along W instead of eight of 4 bytes: 302 -> 279 us on the
// second.  Against the three stages (fp32 GEMMs), both timed in turn: N = 32 1x7
// 192 -> 160 at 17x17 48 -> 37 us (7x1 42), N = 64 1x3 512 -> 512 at 28x28 415 -> 282,
// N = 16 1x7 64 -> 64 at 112x112 192 -> 87, N = 32 1x5 256 -> 256 at 28x28 98 -> 57.
constexpr int kL1FB = 2, kL1TB = 2, kL1Waves = 4;

// bt8 times kSplitScale (powers of two: the same rounding), 3 operations more.
__device__ __forceinline__ void bt8_scaled(const float (&d)[8], float (&v)[8]) {
    constexpr float S = kSplitScale;
    const float s5 = S * d[5], s6 = S * d[6], s7 = S * d[7];
    v[0] = __builtin_fmaf(5.25f * S, d[2] - d[4], __builtin_fmaf(-S, d[0], s6));
    v[7] = __builtin_fmaf(5.25f * S, d[3] - d[5], __builtin_fmaf(-S, d[1], s7));
    const float s15 = __builtin_fmaf(S, d[1], s5), s26 = __builtin_fmaf(S, d[2], s6);
    v[1] = __builtin_fmaf(-4.25f * S, d[3] + d[4], s15 + s26);
    v[2] = __builtin_fmaf(4.25f * S, d[3] - d[4], s26 - s15);
    const float o3 = __builtin_fmaf(0.5f * S, d[1], __builtin_fmaf(-2.5f * S, d[3], 2.0f * s5));
    const float e3 = __builtin_fmaf(0.25f * S, d[2], __builtin_fmaf(-1.25f * S, d[4], s6));
    v[3] = e3 + o3;
    v[4] = e3 - o3;
    const float o5 = __builtin_fmaf(2.0f * S, d[1], __builtin_fmaf(-2.5f * S, d[3], 0.5f * s5));
    const float e5 = __builtin_fmaf(4.0f * S, d[2], __builtin_fmaf(-5.0f * S, d[4], s6));
    v[5] = e5 + o5;
    v[6] = e5 - o5;
}

template <int MT, int AX>
__global__ __launch_bounds__(256, 2) void k_bf3_1d(const float* __restrict__ x, const char* __restrict__ US,
                                                   const float* __restrict__ U, float* __restrict__ y, Geom g, int nkg,
                                                   int kgw, int items, int per, int relu, int vec2) {
    constexpr int T = 8, FB = kL1FB, TB = kL1TB, D = 4, UN = TB * 4 / kL1Waves;
    __shared__ uint4 vs[2 * T * TB * 128];             // [stage][t][tile block][X | Y][64 lanes]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Items (tile blocks, filter group), filter group fastest, each XCD a
    // contiguous range: the groups that share x run together.
    const int item = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (item >= items) return;
    const int kgi = item % nkg, tp = item / nkg;
    const int kbw = kgi * kgw + wave * FB;             // this wave's first filter block
    const bool work = kbw < min(g.KB, (kgi + 1) * kgw);
    const int nsteps = (g.CQ + 3) / 4;

    // ---- transform units: tile block wave % 2, quads wave / 2 and wave / 2 + 2
    const int utb = wave % TB, uq = wave / TB;                // unit j: quad uq + j * (4 / TB)
    const int p0 = (tp * TB + utb) * 16;
    const TileCoord tc = decode_tile(p0 + (lane & 15), g);
    const int cl = lane >> 4;
    const int n0 = __builtin_amdgcn_readfirstlane(min(p0, g.P - 1) / (g.th * g.tw));
    const size_t img = (size_t)g.C * g.H * g.W;
    // The buffer starts 8 inputs before image n0, so that no offset is negative.
    const size_t left = ((size_t)g.N - n0) * img * 4 + 32;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(x + (size_t)n0 * img - 8), (short)0, (int)(left < kInvalid ? left : kInvalid), kRsrcWord3);
    const uint32_t plane_b = (uint32_t)g.H * g.W * 4;
    // The lane's 8 inputs along the axis, `step` bytes apart from off0; in[u]: inside the
    // image (outside it, and for tiles past P, they are zero).
    const int r0 = AX == 1 ? tc.ti : tc.ti * MT - g.pad, c0 = AX == 1 ? tc.tj * MT - g.pad : tc.tj;
    uint32_t in = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int row = AX == 1 ? r0 : r0 + u, col = AX == 1 ? c0 + u : c0;
        in |= (tc.valid && (unsigned)row < (unsigned)g.H && (unsigned)col < (unsigned)g.W ? 1u : 0u) << u;
    }
    const uint32_t off0 = 32u + ((uint32_t)(tc.n - n0) * g.C + cl) * plane_b + (uint32_t)(r0 * g.W + c0) * 4u;
    const uint32_t ustep = AX == 1 ? 4u : (uint32_t)g.W * 4u;
    // Along W the 8 inputs are contiguous: two 16-byte loads, whose dwords outside
    // the row transform() drops.  Only in the first image's first rows and
    // channel can they begin before x itself: a wave that has such tiles loads its
    // first step's inputs one at a time, as all do along H.
    const bool wide0 = n0 != 0 || !__any(in != 0 && off0 < 32u);
    float xd[UN][8];
    auto load_x = [&](int s) {                         // channels past C read as zero
#pragma unroll
        for (int j = 0; j < UN; ++j) {
            const int c = s * 16 + (uq + j * (4 / TB)) * 4;
            const bool ok = c + cl < g.C;
            const int so = __builtin_amdgcn_readfirstlane((int)((uint32_t)c * plane_b));
            if (AX == 1 && (s > 0 || wide0)) {
                const uint32_t o = ok && in ? off0 : kInvalid;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 q = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(o + 16u * h), so, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) xd[j][4 * h + e] = q[e];
                }
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    xd[j][u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                   xr, (int)(ok && (in >> u & 1) ? off0 + u * ustep : kInvalid), so, 0));
            }
        }
    };
    // lane (tile i, channel quad*4 + d) writes dword d of lane quad*16 + i
    uint32_t* const vdst = (uint32_t*)vs + utb * 512 + (lane & 15) * 4 + cl;
    auto transform = [&](int stage) {
#pragma unroll
        for (int j = 0; j < UN; ++j) {
            float d[8], v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) d[u] = AX == 2 || (in >> u & 1) ? xd[j][u] : 0.0f;
            bt8_scaled(d, v);
            uint32_t* const o = vdst + stage * (T * TB * 512) + (uq + j * (4 / TB)) * 64;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                uint32_t X, Y;
                split3(v[t], X, Y);
                o[t * TB * 512] = X;
                o[t * TB * 512 + 256] = Y;
            }
        }
    };

    // ---- filters: ring of D positions
    const size_t us_b = (size_t)g.KB * nsteps * T * kUsBytes;
    const __amdgpu_buffer_rsrc_t ur = __builtin_amdgcn_make_buffer_rsrc(
        (void*)US, (short)0, (int)(us_b < 0x7fffffffu ? us_b : 0x7fffffffu), kRsrcWord3);
    const int l16 = lane * 16, l8 = 1024 + lane * 8;
    uint4 uX[D][FB];
    uint2 uL[D][FB];
    auto load_u = [&](int s, auto pc) {                // position p of step s; steps past the last read the last
        constexpr int p = decltype(pc)::value;
#pragma unroll
        for (int f = 0; f < FB; ++f) {
            const int kb = min(kbw + f, g.KB - 1);
            const int so = __builtin_amdgcn_readfirstlane(
                (int)((((uint32_t)kb * nsteps + min(s, nsteps - 1)) * T + p) * kUsBytes));
            uX[p % D][f] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ur, l16, so, 0));
            uL[p % D][f] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(ur, l8, so, 0));
        }
    };

    f32x4 acc[FB][TB][T];
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int p = 0; p < T; ++p) acc[f][b][p] = f32x4{0.f, 0.f, 0.f, 0.f};

    load_x(0);
    if (work) static_for<0, D>([&](auto pc) { load_u(0, pc); });
    transform(0);
    load_x(1);
    wait_vm_lds<63>();
    wg_barrier();
    for (int s = 0; s < nsteps; ++s) {
        if (s + 1 < nsteps) {
            transform((s + 1) & 1);
            load_x(s + 2);
        }
        if (work) {
            const uint4* const sv = vs + (s & 1) * (T * TB * 128) + lane;
            uint4 vX[2][TB], vY[2][TB];
            auto load_v = [&](auto pc) {
                constexpr int p = decltype(pc)::value;
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    vX[p & 1][b] = sv[(p * TB + b) * 128];
                    vY[p & 1][b] = sv[(p * TB + b) * 128 + 64];
                }
            };
            load_v(IC<0>{});
            static_for<0, T>([&](auto pc) {
                constexpr int p = decltype(pc)::value;
                if constexpr (p + 1 < T) load_v(IC<p + 1>{});
                __builtin_amdgcn_sched_barrier(0);
                uint4 uY[FB];
#pragma unroll
                for (int f = 0; f < FB; ++f) uY[f] = us_y(uX[p % D][f], uL[p % D][f]);
#pragma unroll
                for (int f = 0; f < FB; ++f)
#pragma unroll
                    for (int b = 0; b < TB; ++b) acc[f][b][p] = mfma16x16x32<2>(uX[p % D][f], vY[p & 1][b], acc[f][b][p]);
#pragma unroll
                for (int f = 0; f < FB; ++f)
#pragma unroll
                    for (int b = 0; b < TB; ++b) acc[f][b][p] = mfma16x16x32<2>(uY[f], vX[p & 1][b], acc[f][b][p]);
#pragma unroll
                for (int f = 0; f < FB; ++f)
#pragma unroll
                    for (int b = 0; b < TB; ++b) acc[f][b][p] = mfma16x16x32<2>(uX[p % D][f], vX[p & 1][b], acc[f][b][p]);
                __builtin_amdgcn_sched_barrier(0);
                load_u(s + (p + D) / T, IC<(p + D) % T>{});
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        wait_vm_lds<63>();
        wg_barrier();          // the next step's V is written, this step's consumed
    }
    if (!work) return;

    // Outputs of the 16 filters of block kb from their products m, times scale;
    // true where one of them is not finite (before ReLU).
    auto store = [&](const TileCoord& ot, int kb, const f32x4 (&m)[T], float scale) -> bool {
        float chk = 0.0f;                              // NaN once an output is not finite
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = kb * 16 + 4 * cl + r;
            float a[8], o[MT];
#pragma unroll
            for (int t = 0; t < T; ++t) a[t] = m[t][r];
            at8<MT>(a, o);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                o[i] *= scale;
                chk = __builtin_fmaf(o[i], 0.0f, chk);
            }
            if (!ot.valid || k >= g.K) continue;
            float* yk = y + ((size_t)ot.n * g.K + k) * g.Ho * g.Wo;
#pragma unroll
            for (int i = 0; i < MT; ++i) o[i] = relu ? fmaxf(o[i], 0.0f) : o[i];
            if constexpr (AX == 1) {
                float* const row = yk + (size_t)ot.ti * g.Wo;
                const int col = ot.tj * MT;
#pragma unroll
                for (int i = 0; i < MT; i += 2) {
                    if (vec2 && col + i + 1 < g.Wo) {
                        store_out<false>(row + col + i, o[i], o[i + 1]);
                    } else {
                        if (col + i < g.Wo) row[col + i] = o[i];
                        if (col + i + 1 < g.Wo) row[col + i + 1] = o[i + 1];
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    if (ot.ti * MT + i < g.Ho) yk[(size_t)(ot.ti * MT + i) * g.Wo + ot.tj] = o[i];
            }
        }
        return chk != chk;
    };
    uint32_t redo = 0;                                 // bit b * FB + f: a block to run again
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        const TileCoord ot = decode_tile((tp * TB + b) * 16 + (lane & 15), g);
#pragma unroll
        for (int f = 0; f < FB; ++f)
            if (__any(store(ot, kbw + f, acc[f][b], kSumScale))) redo |= 1u << (b * FB + f);
    }
    // An operand that is infinite or NaN has no split: every result it enters is
    // NaN here.  Such blocks (and those whose sums overflow) run once more on
    // fp32 MFMA, which gives the infinities and NaNs of the three stages.
#pragma unroll 1
    for (int i = 0; i < TB * FB; ++i) {
        const int kb = kbw + i % FB;
        if (!(redo >> i & 1) || kb >= g.KB) continue;
        const TileCoord ot = decode_tile((tp * TB + i / FB) * 16 + (lane & 15), g);
        f32x4 m[T];
#pragma unroll
        for (int t = 0; t < T; ++t) m[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int q0 = AX == 1 ? ot.ti : ot.ti * MT - g.pad, q1 = AX == 1 ? ot.tj * MT - g.pad : ot.tj;
#pragma unroll 1
        for (int cq = 0; cq < g.CQ; ++cq) {
            const int c = cq * 4 + cl;
            const float* xc = x + ((size_t)ot.n * g.C + (c < g.C ? c : 0)) * g.H * g.W;
            float d[8], v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int row = AX == 1 ? q0 : q0 + u, col = AX == 1 ? q1 + u : q1;
                d[u] = ot.valid && c < g.C && (unsigned)row < (unsigned)g.H && (unsigned)col < (unsigned)g.W
                           ? xc[(size_t)row * g.W + col] : 0.0f;
            }
            bt8(d, v);
            const float* ug = U + ((size_t)kb * g.CQ + cq) * T * 64 + lane * 4;
#pragma unroll
            for (int g4 = 0; g4 < T / 4; ++g4) {
                const f32x4 u = *(const f32x4*)(ug + g4 * 256);
#pragma unroll
                for (int e = 0; e < 4; ++e) m[4 * g4 + e] = mfma16x16x4(u[e], v[4 * g4 + e], m[4 * g4 + e]);
            }
        }
        store(ot, kb, m, 1.0f);
    }
}

// ------------------------------------------------------------------ host
// Filter groups of at most 8 blocks, as even as whole waves (two blocks) allow.
static int l1_groups(const Geom& g) { return (g.KB + kL1Waves * kL1FB - 1) / (kL1Waves * kL1FB); }

long bf3_1d_items(const Geom& g) { return ((long)g.PB + kL1TB - 1) / kL1TB * l1_groups(g); }

bool bf3_1d_takes(const Geom& g) {
    // 32-bit offsets: into x over the images that 16 tiles span (channels past
    // C, up to three steps on, add theirs to kInvalidOffset), and into the filters
    const int64_t span = 16 / ((int64_t)g.th * g.tw) + 2, plane_b = (int64_t)g.H * g.W * 4;
    const int64_t c16 = (g.CQ + 3) / 4;
    if (g.axis == 0 || span * g.C * plane_b + 64 >= (int64_t)kInvalidOffset) return false;
    if ((int64_t)kInvalidOffset + (c16 + 3) * 16 * plane_b >= ((int64_t)1 << 32)) return false;
    if ((int64_t)g.CQ * 8192 >= (int64_t)kInvalidOffset) return false;   // what the stages' GEMM takes
    return us_bytes(g) <= 0x7fffffffu && bf3_1d_items(g) < (1L << 28);
}

hipError_t launch_bf3_1d(const float* x, const float* U, float* y, void* ws, const Geom& g, bool relu, hipStream_t s) {
    const hipError_t e = launch_usplit(U, ws, g, s);
    if (e != hipSuccess) return e;
    const int nkg = l1_groups(g), items = (int)bf3_1d_items(g), per = (items + 7) / 8;
    const int kgw = ((g.KB + nkg - 1) / nkg + kL1FB - 1) / kL1FB * kL1FB;
    const int vec2 = g.Wo % 2 == 0 && aligned(y, 8);
    const dim3 grid((unsigned)(8 * per)), block(256);
#define WINO_L1(MT, AX) \
    if (g.m == MT && g.axis == AX) { \
        hipLaunchKernelGGL((k_bf3_1d<MT, AX>), grid, block, 0, s, x, (const char*)ws, U, y, g, nkg, kgw, items, per, (int)relu, vec2); \
        return hipGetLastError(); \
    }
    WINO_L1(6, 1) WINO_L1(4, 1) WINO_L1(2, 1) WINO_L1(6, 2) WINO_L1(4, 2) WINO_L1(2, 2)
#undef WINO_L1
    return hipErrorInvalidValue;
}

// Estimated time, fitted to 1640 layers (74-121% of it in 90 of 100): the filters'
// split, the launches and the last workgroups' outputs (m along the axis, rows
// apart along H), then 1.6 us per step of every 256 workgroups (two of a CU
// overlap, but a step of the pair takes twice as long; one alone takes as long,
// its filter loads' latency) and their outputs.
double bf3_1d_ns(const Geom& g) {
    const double items = bf3_1d_items(g) / 256.0, rounds = items > 1.0 ? items : 1.0, steps = (g.CQ + 3) / 4;
    const double first = g.m == 6 ? 2800.0 : g.m == 4 ? 1100.0 : 0.0, more = g.m == 6 ? 4900.0 : g.m == 4 ? 3000.0 : 1300.0;
    return 8800.0 + first + (g.axis == 2 ? 800.0 : 0.0) + 1600.0 * rounds * steps + more * (rounds - 1.0);
}

}  // namespace wino
