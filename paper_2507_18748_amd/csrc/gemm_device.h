// Device-side building blocks shared by the GEMM kernels: matrix-instruction
// wrappers, buffer loads with hardware range checks, the implicit-GEMM gather
// state, LDS-direct loads and the one-pass epilogue.
#pragma once
#include "kernels.h"

#include <type_traits>

namespace ppipe {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int NUM_XCD = 8;

template <typename T> struct Mfma;
template <> struct Mfma<_Float16> {
    static __device__ __forceinline__ void step(const uint4& a, const uint4& b, floatx4& c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a),
                                                   __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
    }
};
template <> struct Mfma<__bf16> {
    static __device__ __forceinline__ void step(const uint4& a, const uint4& b, floatx4& c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                    __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
// fp32: a 16-byte vector holds 4 consecutive k; four K=4 MFMAs consume it.
// Lane group g supplies k = 4g + t to instruction t for both operands, so the
// pairing of A and B elements is the same as a plain dot product over k.
template <> struct Mfma<float> {
    static __device__ __forceinline__ void step(const uint4& a, const uint4& b, floatx4& c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    }
};

// The activation as one clamp (v_med3_f32): [-inf, inf], [0, inf] or [0, 6].
__device__ __forceinline__ float apply_act(float v, int act)
{
    const float lo = act == ACT_NONE ? -INFINITY : 0.0f;
    const float hi = act == ACT_RELU6 ? 6.0f : INFINITY;
    return __builtin_amdgcn_fmed3f(v, lo, hi);
}

// Load / store 4 consecutive elements of T as one vector access.
template <typename T> struct Vec4;
template <> struct Vec4<float> {
    static __device__ __forceinline__ float4 load(const float* p) { return *(const float4*)p; }
    static __device__ __forceinline__ void store(float* p, float4 v) { *(float4*)p = v; }
};
template <typename T> struct Vec4 {   // 16-bit types
    static __device__ __forceinline__ float4 load(const T* p)
    {
        uint2 u = *(const uint2*)p;
        T e[4];
        __builtin_memcpy(e, &u, 8);
        return make_float4((float)e[0], (float)e[1], (float)e[2], (float)e[3]);
    }
    static __device__ __forceinline__ void store(T* p, float4 v)
    {
        T e[4] = {(T)v.x, (T)v.y, (T)v.z, (T)v.w};
        uint2 u;
        __builtin_memcpy(&u, e, 8);
        *(uint2*)p = u;
    }
};

// Compile-time loop: f(std::integral_constant<int, I>) for I in [B, E).  Keeps
// register-ring indices constant so the ring never lands in scratch memory.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// Tile index -> (m tile, co tile) after spreading the 1-D grid over the XCDs
// in contiguous ranges (the hardware deals block b to XCD b % 8).
// bid, G: the block's index among the G blocks of this problem (a paired
// launch runs two problems in one grid).
__device__ __forceinline__ int3 tile_of_block(const ConvGemmArgs& a, int bid, int G)
{
    const int xcd = bid % NUM_XCD, slot = bid / NUM_XCD;
    const int per = G / NUM_XCD, rem = G % NUM_XCD;
    int lin = xcd * per + min(xcd, rem) + slot;
    const int tiles = a.tiles_m * a.tiles_co;
    const int split = a.splits > 1 ? fast_div(lin, a.div_tiles) : 0;
    lin -= split * tiles;
    const int fast = a.co_fastest ? a.tiles_co : a.tiles_m;
    const int q = fast_div(lin, a.div_fast), r = lin - q * fast;
    return a.co_fastest ? make_int3(q, r, split) : make_int3(r, q, split);   // (m tile, co tile, split)
}
__device__ __forceinline__ int3 tile_of_block(const ConvGemmArgs& a)
{
    return tile_of_block(a, (int)blockIdx.x, (int)gridDim.x);
}

// ---- buffer loads -------------------------------------------------------
// Operands are read through buffer resources: a lane whose byte offset is at
// or beyond the array size gets zeros from the hardware range check.  Zero
// padding taps, ragged tile rows and the K tail are therefore plain loads at
// offset OOB, with no branch and no select in the main loop.
constexpr uint32_t OOB = 0x80000000u;
constexpr int RSRC_FLAGS = 0x00020000;   // raw buffer, 32-bit data format

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                             RSRC_FLAGS);
}
__device__ __forceinline__ uint4 buf_load16(__amdgpu_buffer_rsrc_t r, uint32_t off, int soff = 0)
{
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}
// Position of a K step in (kh, kw, ci) order, wave-uniform, advanced by a
// fixed number of channels; steps never straddle a tap (C is a multiple of the
// step, or the window is 1x1 and the tail is cut by the channel test).
struct TapCursor {
    int ci, kw, kh;
    __device__ __forceinline__ void start(const ConvGemmArgs& a, int k0)
    {
        const int tap = fast_div(k0, a.div_c);
        ci = k0 - tap * a.C;
        kh = fast_div(tap, a.div_kw);
        kw = tap - kh * a.KW;
    }
    __device__ __forceinline__ void advance(int step, int C, int KW)
    {
        ci += step;
        if (ci >= C) {
            ci = 0;
            if (++kw == KW) {
                kw = 0;
                ++kh;
            }
        }
    }
};

// One output pixel (GEMM column) as seen by the gather: byte offset of its
// window origin and which kernel rows / columns fall inside the image.
struct PixelRow {
    int off;          // bytes of x[n][ho*s - p][wo*s - p][0] (may be negative)
    uint32_t hmask;   // bit kh set: 0 <= ho*s - p + kh < H
    uint32_t wmask;   // bit kw set: 0 <= wo*s - p + kw < W
};

// Byte offset of vector kv of a pixel's stage at tap (kh, kw), channel 0; OOB
// where the tap is outside the image or the vector past the channels that are
// left (cleft: those from the stage's first on).
template <int EPV>
__device__ __forceinline__ uint32_t tap_offset(const PixelRow& p, int kh, int kw, int kv, int tap_off,
                                               int cleft)
{
    const int in = (int)((p.hmask << (31 - kh)) & (p.wmask << (31 - kw)));   // sign: both bits set
    return in < 0 && kv * EPV < cleft ? (uint32_t)(p.off + tap_off + kv * 16) : OOB;
}

// Bits k of 0 .. n - 1 with 0 <= first + k < size.
__device__ __forceinline__ uint32_t tap_mask(int first, int n, int size)
{
    const int lo = max(-first, 0), hi = min(n, size - first);   // bits lo .. hi - 1
    return lo >= hi ? 0u : (0xffffffffu >> (32 - (hi - lo))) << lo;
}

__device__ __forceinline__ PixelRow pixel_row(const ConvGemmArgs& a, int m, int esz)
{
    PixelRow p{0, 0u, 0u};
    if (m >= a.M)
        return p;
    const int n = fast_div(m, a.div_hw), rm = m - n * (a.Ho * a.Wo);
    const int ho = fast_div(rm, a.div_w), wo = rm - ho * a.Wo;
    const int hi0 = ho * a.stride - a.pad, wi0 = wo * a.stride - a.pad;
    p.off = (((n * a.H + hi0) * a.W + wi0) * a.C) * esz;
    p.hmask = tap_mask(hi0, a.KH, a.H);
    p.wmask = tap_mask(wi0, a.KW, a.W);
    return p;
}

// Slot of 16-byte vector kv of stage row r: kv ^ dma_swz(r) (see the DMA-staged
// kernels: conflict-free MFMA fragment reads of 128-byte rows).
__device__ __forceinline__ int dma_swz(int r) { return r & 7; }

// One 16-byte load per lane from a buffer resource into LDS: lane L writes
// bytes [lds + 16 L, lds + 16 L + 16); lanes whose offset is beyond the
// resource range write zeros.  Written as inline assembly so that the compiler
// does not insert a full wait for all LDS loads before every LDS read; the
// kernel waits on the vector memory counter itself (dma_wait).  M0 carries the
// LDS address and needs one wait state before the load.
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(voff), "s"(r) : "memory");
}
// The same with a scalar offset added to every lane's (both count in the range
// check; soff must not exceed the resource's size).
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff,
                                      uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory");
}
// Workgroup barrier without the memory fence of __syncthreads (which waits
// for every outstanding LDS read first).  Used where the LDS data a barrier
// protects was written by LDS-direct loads each wave already waited for, and
// the only reads still in flight target a stage no load overwrites next.
__device__ __forceinline__ void bare_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Wait until at most N of this wave's vector memory operations are pending
// (they complete in issue order).
template <int N>
__device__ __forceinline__ void dma_wait()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// Wait until every LDS read this wave issued has returned its data.
__device__ __forceinline__ void lds_read_drain() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// ---- weight prefetch ------------------------------------------------------
// A block past a launch's own tiles reads its part of the next GEMM's weights
// through LDS-direct loads (the data lands in LDS and is dropped), which leaves
// them in the memory-side cache.  idx: this block among the added ones, lds:
// this wave's 1 KB of LDS.
__device__ __forceinline__ void prefetch_weights(const PrefetchArgs& p, int idx, int waves,
                                                 int wave, int lane, uint32_t lds)
{
    const auto src = make_rsrc(p.w, p.bytes);
    for (uint32_t o = (uint32_t)(idx * waves + wave) * 1024u; o < p.bytes;
         o += (uint32_t)(p.blocks * waves) * 1024u)
        dma16(src, o + lane * 16u, lds);
    dma_wait<0>();
}

// ---- prefetched single-pass epilogue (LDS-staged kernels) ----------------
// Dynamic LDS of a staged kernel: the stage ring, or the whole fp32
// [pixel][channel] accumulator tile (rows padded by 4 floats) when that is
// larger, so the epilogue stages the tile in one pass.
constexpr int gemm_lds_bytes(int BM, int BN, int NS)
{
    return NS * (BM + BN) * 128 > BN * (BM + 4) * 4 ? NS * (BM + BN) * 128 : BN * (BM + 4) * 4;
}

// Epilogue operands of one thread.  A thread finishes the same EPV channels
// (co0 + c, c fixed by the thread index) of NV pixel rows of the tile, so its
// scale, shift and residual vectors are all known when the K loop ends: their
// loads go out together, before the tile is staged, instead of one dependent
// chain per pass.
template <typename T, int BM, int BN, int NT>
struct EpiPre {
    static constexpr int ESZ = (int)sizeof(T);
    static constexpr int EPV = 16 / ESZ;
    static constexpr int VPR = BM / EPV;          // 16-byte vectors per staged pixel row
    static constexpr int NV = BN * VPR / NT;      // vectors per thread
    static_assert(NT % VPR == 0 && (BN * VPR) % NT == 0, "fixed channel group per thread");
    floatx4 sc[EPV / 4], bi[EPV / 4];
    uint4 res[NV];

    __device__ __forceinline__ void load(const ConvGemmArgs& a, int m0, int co0, int tid)
    {
        const int co = co0 + (tid % VPR) * EPV;
        const bool cok = co < a.Co;                // Co % EPV == 0: the whole vector is in range
        const auto sr = make_rsrc(a.scale, (uint32_t)a.Co * 4);
        const auto br = make_rsrc(a.bias, (uint32_t)a.Co * 4);
#pragma unroll
        for (int q = 0; q < EPV / 4; ++q) {
            sc[q] = __builtin_bit_cast(floatx4, buf_load16(sr, cok ? (uint32_t)(co + 4 * q) * 4 : OOB));
            bi[q] = __builtin_bit_cast(floatx4, buf_load16(br, cok ? (uint32_t)(co + 4 * q) * 4 : OOB));
        }
        if (a.res) {
            const auto rr = make_rsrc(a.res, (uint32_t)((size_t)a.M * a.Co * ESZ));
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const int m = m0 + (tid + k * NT) / VPR;
                res[k] = buf_load16(rr, cok && m < a.M ? (uint32_t)(((size_t)m * a.Co + co) * ESZ) : OOB);
            }
        }
    }

    // The tile is staged in ep ([pixel][channel] fp32, LROW floats a row).
    template <int LROW>
    __device__ __forceinline__ void finish(const ConvGemmArgs& a, const float* ep, int m0, int co0,
                                           int tid) const
    {
        const int c = (tid % VPR) * EPV, co = co0 + c;
        if (co >= a.Co)
            return;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int row = (tid + k * NT) / VPR, m = m0 + row;
            if (m >= a.M)
                break;                            // rows grow with k
            float o[EPV];
#pragma unroll
            for (int q = 0; q < EPV / 4; ++q) {
                const floatx4 x = *(const floatx4*)(ep + row * LROW + c + 4 * q);
#pragma unroll
                for (int j = 0; j < 4; ++j) o[4 * q + j] = x[j] * sc[q][j] + bi[q][j];
            }
            if (a.res) {
                T r[EPV];
                __builtin_memcpy(r, &res[k], 16);
#pragma unroll
                for (int j = 0; j < EPV; ++j) o[j] += (float)r[j];
            }
            T e[EPV];
#pragma unroll
            for (int j = 0; j < EPV; ++j) e[j] = (T)apply_act(o[j], a.act);
            uint4 u;
            __builtin_memcpy(&u, e, 16);
            *(uint4*)((T*)a.y + (size_t)m * a.Co + co) = u;
        }
    }
};

}  // namespace ppipe
