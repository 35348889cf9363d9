// Device helpers shared by the kernel files: MFMA wrappers, tile geometry,
// region loads and output stores, waits and barriers, compile-time loops.
#pragma once

#include <type_traits>
#include <utility>

#include "wino_internal.h"
#include "wino_transforms.h"

namespace wino {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma16x16x4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// The 16-bit form: fp16 (PREC 1) or bf16 (PREC 2), eight reduction slots per
// lane in a 16-byte operand, fp32 accumulation.
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int PREC>
__device__ __forceinline__ f32x4 mfma16x16x32(uint4 a, uint4 b, f32x4 c) {
    if constexpr (PREC == 1)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b),
                                                       c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                        __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// ------------------------------------------------------------------ exact split
// A fp32 value as three bf16 terms, h + m + l, eight significand bits each: the
// operands of the kernels that run fp32 products on the bf16 matrix cores.  They
// split 2^16 times the value: bf16's smallest number is 2^-133, fp32's 2^-149, so
// that of unscaled values below 2^-110 l, and below 2^-118 m, would lose bits (x of
// 1e-36 gave errors of 3e-5).  Products carry 2^32, taken out of the sums.  At the
// other end values from 2^112 and sums from 2^96 overflow, which the check for
// results that are not finite catches.
constexpr uint32_t kHi16 = 0xffff0000u;
constexpr float kSplitScale = 65536.0f, kSumScale = 1.0f / (65536.0f * 65536.0f);

// (X, Y) of one value, h and m cut off towards zero; low half first:
// X = (m, h), Y = (h, l).
__device__ __forceinline__ void split3(float v, uint32_t& X, uint32_t& Y) {
    const uint32_t vb = __float_as_uint(v);
    const float r1 = v - __uint_as_float(vb & kHi16);               // exact
    const uint32_t rb = __float_as_uint(r1);
    const float r2 = r1 - __uint_as_float(rb & kHi16);              // exact, at most 8 bits
    X = __builtin_amdgcn_perm(vb, rb, 0x07060302u);                 // low half m, high half h
    Y = __builtin_amdgcn_perm(__float_as_uint(r2), vb, 0x07060302u);   // low half h, high half l
}

// 4 x 4 transpose of the wave's four rows of 16 lanes and four registers: r[k]
// in row e becomes r[e] of row k.
__device__ __forceinline__ void transpose_rows(uint32_t (&r)[4]) {
    auto swap32 = [](uint32_t& a, uint32_t& b) {       // rows 2, 3 of a with rows 0, 1 of b
        const auto q = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = q[0];
        b = q[1];
    };
    auto swap16 = [](uint32_t& a, uint32_t& b) {       // rows 1, 3 of a with rows 0, 2 of b
        const auto q = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = q[0];
        b = q[1];
    };
    swap32(r[0], r[2]);
    swap32(r[1], r[3]);
    swap16(r[0], r[1]);
    swap16(r[2], r[3]);
}

// Split filters in memory (k_usplit): per (filter block, 16 channels, position)
// the X words [64][16 bytes] and the l terms [64][8 bytes].
constexpr int kUsBytes = 1536;

// The same layout for transformed inputs, [tile block][C16][T]{X, l}: a wave
// that holds T values of (channel lane / 16 of quad q, tile lane % 16) stores
// them as operand words, four positions at a time (after the transpose a lane
// has the quad's four channels at position lane / 16).  blk: the (tile block, 16
// channels).  Whole columns of lanes (one tile's four) are active or not.
template <int T>
__device__ __forceinline__ void store_v3(char* __restrict__ blk, int q, int lane, const float (&v)[T]) {
    char* p = blk + (lane >> 4) * kUsBytes;
    const int i = q * 16 + (lane & 15);
#pragma unroll
    for (int g4 = 0; g4 < T / 4; ++g4) {
        uint32_t r[4], X[4], Y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = __float_as_uint(v[4 * g4 + e]);
        transpose_rows(r);
#pragma unroll
        for (int d = 0; d < 4; ++d) split3(__uint_as_float(r[d]) * kSplitScale, X[d], Y[d]);
        *(uint4*)(p + g4 * 4 * kUsBytes + i * 16) = make_uint4(X[0], X[1], X[2], X[3]);
        *(uint2*)(p + g4 * 4 * kUsBytes + 1024 + i * 8) = make_uint2(__builtin_amdgcn_perm(Y[1], Y[0], 0x07060302u),
                                                                     __builtin_amdgcn_perm(Y[3], Y[2], 0x07060302u));
    }
}

// A lane's Y = (h, l) words from its X = (m, h) words and l terms.
__device__ __forceinline__ uint4 us_y(uint4 X, uint2 L) {
    return make_uint4(__builtin_amdgcn_perm(L.x, X.x, 0x05040302u), __builtin_amdgcn_perm(L.x, X.y, 0x07060302u),
                      __builtin_amdgcn_perm(L.y, X.z, 0x05040302u), __builtin_amdgcn_perm(L.y, X.w, 0x07060302u));
}

// ------------------------------------------------------------------ helpers

__device__ __forceinline__ uint32_t fdiv(uint32_t n, FastDiv d) { return (__umulhi(n, d.m) + n) >> d.l; }

struct TileCoord {
    int n, ti, tj;
    bool valid;
};

__device__ __forceinline__ TileCoord decode_tile(int p, const Geom& g) {
    TileCoord t;
    t.valid = p < g.P;
    const int pp = t.valid ? p : 0;
    const int per = g.th * g.tw;
    t.n = pp / per;
    const int rem = pp - t.n * per;
    t.ti = rem / g.tw;
    t.tj = rem - t.ti * g.tw;
    return t;
}

// ---- region loads through a per-wave buffer resource -----------------------
// Offsets are 32-bit byte offsets from the first image a 16-tile block touches.
// Any offset >= kInvalid lies past the resource's record count, and the buffer
// unit returns 0 for it: a padded row, column, channel or tile is read as zero
// without a select.  The host guarantees that every valid offset is below
// kInvalid (the images one block spans hold < 1 GiB of input).
constexpr uint32_t kInvalid = kInvalidOffset;
constexpr int kRsrcWord3 = 0x00020000;   // raw (unformatted) 32-bit buffer

// Transformed filters as a raw buffer (the host keeps U below 2 GiB for the
// fused kernels).  A lane's 16-byte word of a U group sits at the constant
// per-lane offset lane*16 plus a wave-uniform group offset, so filter loads
// need no per-load address registers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t u_rsrc(const float* U, const Geom& g) {
    const size_t ub = (size_t)g.KB * g.CQ * g.T * 256;
    return __builtin_amdgcn_make_buffer_rsrc((void*)U, (short)0, (int)(ub < 0x7fffffffu ? ub : 0x7fffffffu),
                                             kRsrcWord3);
}
__device__ __forceinline__ f32x4 u_load(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t group_off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)group_off, 0));
}

// Regions of side A (MT + 2 for 3x3 filters, MT + 4 for 5x5) stepping by MT.
template <int MT, int A = MT + 2>
struct RegionPlan {
    __amdgpu_buffer_rsrc_t rsrc;     // wave-uniform
    uint32_t row[A];                 // lane's channel-plane + row byte offset, or kInvalid
    uint32_t col[A];                 // column byte offset, or kInvalid
    uint32_t plane_bytes;            // H*W*4: step between channels (soffset units)
};

// p0 = first tile of the wave's 16-tile block (wave-uniform); tc = lane's tile;
// cl = lane's channel within a quad.
template <int MT, int A = MT + 2>
__device__ __forceinline__ RegionPlan<MT, A> make_region_plan(const float* __restrict__ x, const Geom& g,
                                                              int p0, const TileCoord& tc, int cl) {
    RegionPlan<MT, A> rp;
    const int n0 = __builtin_amdgcn_readfirstlane(min(p0, g.P - 1) / (g.th * g.tw));
    const size_t img = (size_t)g.C * g.H * g.W;
    const size_t left = ((size_t)g.N - n0) * img * 4;
    rp.rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(x + (size_t)n0 * img), (short)0,
                                                (int)(left < kInvalid ? left : kInvalid), kRsrcWord3);
    rp.plane_bytes = (uint32_t)g.H * g.W * 4;
    const uint32_t plane = ((uint32_t)(tc.n - n0) * g.C + cl) * rp.plane_bytes;
    const int r0 = tc.ti * MT - g.pad, c0 = tc.tj * MT - g.pad;
#pragma unroll
    for (int u = 0; u < A; ++u) {
        const int row = r0 + u;
        rp.row[u] = (tc.valid && row >= 0 && row < g.H) ? plane + (uint32_t)row * g.W * 4 : kInvalid;
    }
#pragma unroll
    for (int v = 0; v < A; ++v) {
        const int col = c0 + v;
        rp.col[v] = (col >= 0 && col < g.W) ? (uint32_t)col * 4 : kInvalid;
    }
    return rp;
}

// d = the region of channel quad cq for this lane (channel cq*4 + cl), zero
// outside the image, past the last channel, and for tiles past P.
template <int MT, int A = MT + 2>
__device__ __forceinline__ void load_region(const RegionPlan<MT, A>& rp, const Geom& g, int cq, int cl,
                                            float (&d)[A][A]) {
    const uint32_t chan = (cq * 4 + cl < g.C) ? 0u : kInvalid;
    const int soff = __builtin_amdgcn_readfirstlane(cq * 4 * (int)rp.plane_bytes);
#pragma unroll
    for (int u = 0; u < A; ++u) {
        const uint32_t rowq = rp.row[u] + chan;
#pragma unroll
        for (int v = 0; v < A; ++v)
            d[u][v] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                          rp.rsrc, (int)(rowq + rp.col[v]), soff, 0));
    }
}

// Products of one (16-tile block at tile p0, filter block kb) at all T positions
// on fp32 MFMA, straight from x and U: what the kernels that split their
// operands in three run again where a result is not finite.  A lane gets the
// accumulator words of M (tile lane % 16, filters 4 * (lane / 16) .. +3).
template <int MT, int R>
__device__ __forceinline__ void fp32_products(const float* __restrict__ x, const float* __restrict__ U, const Geom& g,
                                              int p0, int kb, int lane, f32x4 (&acc)[(MT + R - 1) * (MT + R - 1)]) {
    constexpr int A = MT + R - 1, T = A * A;
    const int cl = lane >> 4;
    const TileCoord tc = decode_tile(p0 + (lane & 15), g);
    const RegionPlan<MT, A> rp = make_region_plan<MT, A>(x, g, p0, tc, cl);
    const __amdgpu_buffer_rsrc_t ur = u_rsrc(U, g);
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int cq = 0; cq < g.CQ; ++cq) {
        float d[A][A], v[T];
        load_region<MT, A>(rp, g, cq, cl, d);
        input_tf<A - 2>(d, v);
        const uint32_t grp = __builtin_amdgcn_readfirstlane((uint32_t)(kb * g.CQ + cq) * (T / 4) * 1024u);
#pragma unroll
        for (int g4 = 0; g4 < T / 4; ++g4) {
            const f32x4 u = u_load(ur, (uint32_t)lane * 16u, grp + g4 * 1024u);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * g4 + e] = mfma16x16x4(u[e], v[4 * g4 + e], acc[4 * g4 + e]);
        }
    }
}

// Output rows leave through streaming (non-temporal) stores where a kernel
// writes whole cache lines: y is not read back, so it need not displace cached
// inputs.  Where the lines of a row are completed by several store
// instructions (rows narrower than a line run, or not line-aligned), plain
// stores let L2 merge the pieces before they go to HBM; streaming stores of
// such pieces run at half the bandwidth or less.
template <bool NT>
__device__ __forceinline__ void store_out(float* p, float a, float b, float c, float d) {
    const f32x4 q = {a, b, c, d};
    if constexpr (NT) __builtin_nontemporal_store(q, (f32x4*)p);
    else *(f32x4*)p = q;
}
template <bool NT>
__device__ __forceinline__ void store_out(float* p, float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 q = {a, b};
    if constexpr (NT) __builtin_nontemporal_store(q, (f32x2*)p);
    else *(f32x2*)p = q;
}

// Write output row i (MT values) of the block of (tile tc, output channel k),
// cropped to Ho x Wo.
template <int MT, bool NT = true>
__device__ __forceinline__ void store_row(float* __restrict__ y, const Geom& g, const TileCoord& tc, int k,
                                          int i, const float (&o)[MT], bool relu, bool vec_ok) {
    const int oi = tc.ti * MT + i, oj0 = tc.tj * MT;
    if (!tc.valid || k >= g.K || oi >= g.Ho) return;
    float* row = y + (((size_t)tc.n * g.K + k) * (size_t)g.Ho + oi) * (size_t)g.Wo + oj0;
    float v[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) v[j] = relu ? fmaxf(o[j], 0.0f) : o[j];
    if (vec_ok && oj0 + MT <= g.Wo) {
        if constexpr (MT == 4) {
            store_out<NT>(row, v[0], v[1], v[2], v[3]);
        } else {
            store_out<NT>(row, v[0], v[1]);
        }
    } else {
        // Plain 4-byte stores, whatever NT says: they merge into whole lines
        // in L2, where non-temporal ones went out as partial-line writes
        // (25-30% of the split and fused calls on 26-30 pixel wide layers).
#pragma unroll
        for (int j = 0; j < MT; ++j)
            if (oj0 + j < g.Wo) row[j] = v[j];
    }
}

// Write the m x m output block of (tile tc, output channel k), cropped to Ho x Wo.
template <int MT, bool NT = true>
__device__ __forceinline__ void store_block(float* __restrict__ y, const Geom& g,
                                            const TileCoord& tc, int k,
                                            const float (&o)[MT][MT], bool relu, bool vec_ok) {
#pragma unroll
    for (int i = 0; i < MT; ++i) store_row<MT, NT>(y, g, tc, k, i, o[i], relu, vec_ok);
}

// Channel-last y [N][Ho][Wo][K]: the m x m outputs of (tile tc, output channels
// k0 .. k0+3), cropped to Ho x Wo and K; one 16-byte store per pixel when vec
// (K % 4 == 0 and y 16-byte aligned), streaming when NT.
template <int MT, bool NT = false>
__device__ __forceinline__ void store_tile_nhwc(float* __restrict__ y, const Geom& g, const TileCoord& tc, int k0,
                                                const float (&o)[4][MT][MT], bool relu, bool vec) {
    if (!tc.valid || k0 >= g.K) return;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            const int oi = tc.ti * MT + i, oj = tc.tj * MT + j;
            if (oi >= g.Ho || oj >= g.Wo) continue;
            float* py = y + (((size_t)tc.n * g.Ho + oi) * g.Wo + oj) * g.K + k0;
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = relu ? fmaxf(o[r][i][j], 0.0f) : o[r][i][j];
            if (vec && k0 + 4 <= g.K) {
                store_out<NT>(py, v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (k0 + r < g.K) py[r] = v[r];
            }
        }
}

// Store a lane's T transform-domain values into one (block, quad) group of the
// U/V layout [T/4][64][4]: one 16-byte store per group of four positions, the
// wave writing whole 1 KiB runs.  NT: streaming stores (measured: faster for
// the staged input transform, slower for the split path's).
template <int T, bool NT>
__device__ __forceinline__ void store_t4(float* __restrict__ blk, int lane, const float (&v)[T]) {
#pragma unroll
    for (int g4 = 0; g4 < T / 4; ++g4)
        store_out<NT>(blk + ((size_t)g4 * 64 + lane) * 4, v[4 * g4], v[4 * g4 + 1], v[4 * g4 + 2], v[4 * g4 + 3]);
}

// s_waitcnt immediate: vmcnt <= n, lgkmcnt = 0, expcnt unconstrained.
template <int n>
__device__ __forceinline__ void wait_vm_lds() {
    static_assert(n >= 0 && n < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (0 << 8) | (((n >> 4) & 3) << 14));
}

// Workgroup barrier without the release fence of __syncthreads(): that fence
// would also wait for the direct-to-LDS loads still in flight for later steps.
// Callers first wait for exactly the loads (vmcnt) and LDS operations
// (lgkmcnt) the other waves need; the memory clobber keeps the compiler from
// moving memory accesses across it.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// One direct-to-LDS buffer load of BYTES per lane (a device function: the
// host pass rejects the 16-byte form written directly in a kernel body).
template <int BYTES>
__device__ __forceinline__ void lds_dma(__amdgpu_buffer_rsrc_t r, float* lds, uint32_t off, uint32_t soff = 0) {
    static_assert(BYTES == 4 || BYTES == 16, "dword or 16-byte loads");
    if constexpr (BYTES == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, lds, 16, off, soff, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(r, lds, 4, off, soff, 0, 0);
}

template <int R> using IC = std::integral_constant<int, R>;

// f(IC<I>) for I = I0 .. I1-1, in order.
template <int I0, int I1, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I0 < I1) {
        f(IC<I0>{});
        static_for<I0 + 1, I1>(f);
    }
}

// f(IC<v>) for the runtime value v in [0, N) (wave-uniform): one instance per value.
template <typename F, int... I>
__device__ __forceinline__ void with_ic(int v, F&& f, std::integer_sequence<int, I...>) {
    ((v == I ? (f(IC<I>{}), 0) : 0), ...);
}

// ------------------------------------------------------------------ launch helpers
static inline bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

// The split path's GEMM kernel streams y only past half of the 256 MB
// last-level cache: below that, plain stores leave y there for the next
// layer and also finish sooner themselves (VGG-16 at N = 32: layers with
// 51-103 MB of output 2-9% faster per call, the stack 3%); at 205 MB streaming
// stays ahead (the 112x112 layers 3-6%, the channel-last N = 64 256-channel
// layer 2%).
constexpr size_t kSplitStreamBytes = 128u << 20;
static inline int split_stream_stores(const Geom& g) {
    return (size_t)g.N * g.K * g.Ho * g.Wo * sizeof(float) > kSplitStreamBytes ? 1 : 0;
}

}  // namespace wino
