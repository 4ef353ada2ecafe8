// fp32 convolutions on the 16-bit matrix cores: every fp32 operand is the
// exact sum of three bf16 values.
//
// The fp32 matrix instruction runs at 1/16 of the bf16 rate (157 against 2500
// TFLOP/s), and the fp32 layers of a partition were bound by it.  A float has
// 24 significant bits and a bf16 eight, so x = x0 + x1 + x2 with
//     x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1
// (rounded to nearest even; both differences are exact, and x2 fits a bf16), the
// splitting of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype for Higher-Precision Computations" (ARITH 2019).
// A product of two such sums has nine terms; the three smallest (x1 w2, x2 w1,
// x2 w2) are left out and the other six are accumulated in fp32 by
// v_mfma_f32_16x16x32_bf16, whose 16-bit products are exact.  |x1| is at most
// 2^-8 and |x2| 2^-17 of |x|, so the terms left out stay below 2^-24 of |x w|,
// one rounding to fp32 (2^-28 on average); a product that fits fp32 has none of
// them.  Nothing is stored or summed in 16 bits: the planes together hold the
// fp32 value.  The fp32 accumulator is rounded six times per 32 k instead of
// at each of eight K = 4 instructions, and the error against 64-bit sums is no
// larger than the fp32 instruction's (figures at the dispatch rule).  Work per
// 32 k of a 16x16 tile: 6 x 16 cycles against 8 x 32.
//
// Weights are split once at create (launch_split_weights) into fragment order
// [16 channels][32 k][plane][lane][8 bf16] (lane l: channel l % 16, k = 4 (l / 16)
// .. + 4 and 16 + 4 (l / 16) .. + 4, the same order for both operands): a
// fragment is 1 KB contiguous in memory and in LDS.  Activations stay fp32 in
// memory and each wave splits the fragments it loads.  A wave owns 16 FM
// channels x 32 pixels, so that its split (56 vector instructions per 32 k)
// fits beside its 12 FM matrix instructions.
//
// Planes below the smallest normal bf16 (2^-126) are flushed, which an operand
// below 2^-102 would lose bits to.  Weights are therefore split after a
// multiplication by 2^24 (every fp32 value is a multiple of 2^-149, so every
// scaled plane is normal or zero) that the sums carry and the tile's end takes
// out.  Doing the same to the activations costs 3.6% (two more vector
// instructions per pair), so they stay as they are: flushes change a sum by
// less than 2^-124 of the filter's magnitude, which only a tiny sum can show.
// A block with a sum below 2^-98 of it (`tiny`, zero sums among them) looks its
// activations over, and one that finds a nonzero one below 2^-102 takes the
// fp32 path of the next paragraph.  (Checking the sums takes 0.1 to 0.2 us of a
// tile; maps of zeros, where every block looks, take 1.4 times as long.)
//
// Infinities, NaN, and magnitudes that round to an infinite bf16 (scaled
// weights or sums among them, from 2^104 on) leave a non-finite sum (inf - inf
// in the split), never a finite wrong one.  A block that finds one recomputes
// its tile with the fp32 instruction from the fp32 weights, so such inputs give
// what the fp32 kernels give.
#include "gemm_device.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace ppipe {

namespace {

struct SplitArgs {
    ConvGemmArgs a;
    const void* w3;    // weight planes in fragment order
    const float* tiny; // [Co]: scaled sums below it may have lost bits of tiny activations
    float tiny_max;    // the largest of them
};
constexpr float SPLIT_W_SCALE = 0x1p24f, SPLIT_UNSCALE = 0x1p-24f;
constexpr uint32_t SPLIT_X_MIN = (127u - 102u) << 23;   // 2^-102: every plane is normal

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float x, float y)   // nearest even
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){x, y}, bf16x2));
}
// v - (low / high half of p): one v_dot2_f32_bf16 with (-1, 0) or (0, -1); the
// difference of a float and its bf16 rounding is exact.  The unit comes from a
// register: as an inline constant the instruction takes -1.0 for (0, -1).
__device__ __forceinline__ float minus_half(float v, uint32_t p, uint32_t unit)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p),
                                           __builtin_bit_cast(bf16x2, unit), v, false);
}

// Two floats into the three planes of one 32-bit word each.
__device__ __forceinline__ void split2(float x, float y, uint32_t& p0, uint32_t& p1, uint32_t& p2)
{
    uint32_t LO = 0x0000bf80u, HI = 0xbf800000u;
    asm("" : "+s"(LO), "+s"(HI));
    p0 = pack_bf16(x, y);
    const float rx = minus_half(x, p0, LO), ry = minus_half(y, p0, HI);
    p1 = pack_bf16(rx, ry);
    p2 = pack_bf16(minus_half(rx, p1, LO), minus_half(ry, p1, HI));
}
// Eight consecutive k (two 16-byte vectors) into three fragment vectors.
__device__ __forceinline__ void split8(const uint4& lo, const uint4& hi, uint4 (&p)[3])
{
    const uint32_t v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    uint32_t o[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        split2(__uint_as_float(v[2 * i]), __uint_as_float(v[2 * i + 1]), o[0][i], o[1][i], o[2][i]);
#pragma unroll
    for (int q = 0; q < 3; ++q) p[q] = make_uint4(o[q][0], o[q][1], o[q][2], o[q][3]);
}

__device__ __forceinline__ uint4 scaled(const float4& v)
{
    return make_uint4(__float_as_uint(v.x * SPLIT_W_SCALE), __float_as_uint(v.y * SPLIT_W_SCALE),
                      __float_as_uint(v.z * SPLIT_W_SCALE), __float_as_uint(v.w * SPLIT_W_SCALE));
}

// One thread per (16-channel group, 32-k chunk, lane).
__global__ void __launch_bounds__(256)
split_weights_kernel(const float* __restrict__ w, uint4* __restrict__ w3, int Co, int Kpad,
                     int chunks, int groups)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    const int lane = i & 63;
    const uint32_t gc = i >> 6;                   // group * chunks + chunk
    if (gc >= (uint32_t)groups * chunks)
        return;
    const int c = gc % chunks, g = gc / chunks;
    const int row = g * 16 + (lane & 15), k = 32 * c + 4 * (lane >> 4);
    uint4 lo = make_uint4(0u, 0u, 0u, 0u), hi = lo;
    if (row < Co) {   // Kpad is a multiple of 64: whole vectors
        const float* src = w + (size_t)row * Kpad + k;
        lo = scaled(*(const float4*)src);
        hi = scaled(*(const float4*)(src + 16));
    }
    uint4 p[3];
    split8(lo, hi, p);
#pragma unroll
    for (int q = 0; q < 3; ++q) w3[((size_t)gc * 3 + q) * 64 + lane] = p[q];
}

// The wave's tile with the fp32 matrix instruction, operands straight from
// memory (the non-finite case only).
template <int FM>
__device__ __forceinline__ void f32_tile(const ConvGemmArgs& a, int m0, int co0, int lane,
                                         floatx4 (&acc)[FM][2])
{
    const auto wsrc = make_rsrc(a.w, (uint32_t)a.Co * a.Kpad * 4);
    const auto xsrc = make_rsrc(a.x, (uint32_t)a.N * a.H * a.W * a.C * 4);
    const int g = lane >> 4, r = lane & 15;
    PixelRow px[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) px[j] = pixel_row(a, m0 + j * 16 + r, 4);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    TapCursor cur;
    cur.start(a, 0);
    const int steps = (a.K + 15) / 16;
#pragma unroll 1
    for (int u = 0; u < steps; ++u) {
        uint4 av[FM], bv[2];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int co = co0 + i * 16 + r;
            av[i] = buf_load16(wsrc, co < a.Co ? (uint32_t)((co * a.Kpad + 16 * u + 4 * g) * 4) : OOB);
        }
        const int tap_off = ((cur.kh * a.W + cur.kw) * a.C + cur.ci + 4 * g) * 4;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const bool ok = 4 * g < a.C - cur.ci &&
                            ((px[j].hmask >> cur.kh) & (px[j].wmask >> cur.kw) & 1u);
            bv[j] = buf_load16(xsrc, ok ? (uint32_t)(px[j].off + tap_off) : OOB);
        }
        cur.advance(16, a.C, a.KW);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) Mfma<float>::step(av[i], bv[j], acc[i][j]);
    }
}

template <int FM, int WN, int KSP>
constexpr int split_lds_bytes()
{
    const int ring = 2 * KSP * FM * 3 * 1024;
    const int tile = WN * 32 * (FM * 16 + 4) * 4;
    return ring > tile ? ring : tile;
}

// Block tile: 16 FM channels x 32 WN pixels on WN x KSP waves.  Wave (wn, h)
// computes the 16 FM x 32 tile of pixel group wn over the 32-k chunks h,
// h + KSP, ...; the KSP partial tiles are summed in that order through LDS.
//
// Only the weight planes go through LDS (two stages of KSP chunks), where the
// WN waves of a K part share them; a pixel belongs to one wave of a K part, so
// its vectors go from memory to that wave's registers.  Step s multiplies
// chunk s while the activations of chunk s + 1 are split, the planes of chunk
// s + 1 move from registers to LDS and the loads of chunk s + 2 are in flight.
template <int FM, int WN, int KSP>
__global__ void __launch_bounds__(WN * KSP * 64, 2)
conv_gemm_split(SplitArgs p)
{
    const ConvGemmArgs& a = p.a;
    constexpr int NW = WN * KSP, NT = NW * 64;
    constexpr int BM = 16 * FM, BN = 32 * WN;
    constexpr int A_HALF = FM * 3 * 1024, STAGE = KSP * A_HALF;
    constexpr int LA = FM * 3 / WN;          // weight fragments loaded per wave and chunk
    static_assert(FM * 3 % WN == 0, "whole weight fragments per wave");

    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
    asm volatile("" ::"s"(p.w3), "s"(p.tiny), "s"(p.tiny_max));
    const int3 bg = load_args_now(a, (int)blockIdx.x, (int)gridDim.x);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, h = wave / WN;
    const int3 tt = tile_of_block(a, bg.x, bg.y);
    const int m0 = tt.x * BN, co0 = tt.y * BM;
    const int chunks = a.total_chunks;
    const int nst = (chunks + KSP - 1) / KSP;
    const int groups = (a.Co + 15) / 16;
    const auto wsrc = make_rsrc(p.w3, (uint32_t)groups * chunks * 3072u);
    const auto xsrc = make_rsrc(a.x, (uint32_t)a.N * a.H * a.W * a.C * 4);

    // weight fragments wn, wn + WN, ... of the wave's K part
    uint32_t a_off[LA];
#pragma unroll
    for (int q = 0; q < LA; ++q) {
        const int f = q * WN + wn;           // channel group f / 3, plane f % 3
        const int g = co0 / 16 + f / 3;
        a_off[q] = g < groups ? (uint32_t)((g * chunks * 3 + f % 3) * 1024 + lane * 16) : OOB;
    }
    // pixels 32 wn + 16 j + lane % 16; lane group g takes k = 4 g and 16 + 4 g
    // of every chunk.  A ragged 1x1 channel tail reads on into the next pixel
    // under zero weights (a non-finite value there only costs the fp32 pass).
    int b_off[2];
    uint32_t b_h[2], b_w[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const PixelRow px = pixel_row(a, m0 + wn * 32 + j * 16 + (lane & 15), 4);
        b_off[j] = px.off + 16 * (lane >> 4);
        b_h[j] = px.hmask;
        b_w[j] = px.wmask;
    }
    TapCursor cur;
    int lc = h;                              // next chunk to load
    cur.start(a, h * 32);
    uint4 ra[LA], rb[2][2];
    auto load = [&]() {
        const bool live = KSP == 1 || lc < chunks;   // past the end: weights read as zeros
        const int koff = (lc < chunks ? lc : chunks - 1) * 3072;
#pragma unroll
        for (int q = 0; q < LA; ++q)
            ra[q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  wsrc, live ? a_off[q] : OOB, koff, 0));
        const int tap_off = ((cur.kh * a.W + cur.kw) * a.C + cur.ci) * 4;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int in = (int)((b_h[j] << (31 - cur.kh)) & (b_w[j] << (31 - cur.kw)));
            const uint32_t off = in < 0 ? (uint32_t)(b_off[j] + tap_off) : OOB;
            rb[j][0] = buf_load16(xsrc, off);
            rb[j][1] = buf_load16(xsrc, off + 64);
        }
#pragma unroll
        for (int q = 0; q < KSP; ++q) {              // branch-free: one block per step
            const int ci = cur.ci + 32, wrap = ci >= a.C ? 1 : 0, kw = cur.kw + wrap;
            const int down = kw == a.KW ? 1 : 0;
            cur.ci = wrap ? 0 : ci;
            cur.kw = down ? 0 : kw;
            cur.kh += down;
        }
        lc += KSP;
    };
    auto put = [&](int slot) {
#pragma unroll
        for (int q = 0; q < LA; ++q)
            *(uint4*)(dyn_smem + slot * STAGE + h * A_HALF + (q * WN + wn) * 1024 + lane * 16) = ra[q];
    };

    // x0 w0 in one accumulator, the five small terms in another: the large
    // sum is rounded once per chunk
    floatx4 acc[FM][2], low[FM][2];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            acc[i][j] = low[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    uint4 b0[2][3], b1[2][3];
    load();
    put(0);
#pragma unroll
    for (int j = 0; j < 2; ++j) split8(rb[j][0], rb[j][1], b0[j]);
    load();
    // chunk s: activation planes bc, its weights in LDS slot s & 1; chunk s + 1:
    // in registers, split into bn; chunk s + 2: loaded once those are read
    auto step = [&](int s, const uint4 (&bc)[2][3], uint4 (&bn)[2][3]) {
        __syncthreads();   // planes of chunk s are in LDS, those of s - 1 consumed
        put((s + 1) & 1);
        const unsigned char* S = dyn_smem + (s & 1) * STAGE + h * A_HALF + lane * 16;
        uint4 af[3][FM];
        auto read = [&](int q) {
#pragma unroll
            for (int i = 0; i < FM; ++i) af[q][i] = *(const uint4*)(S + (i * 3 + q) * 1024);
        };
        uint32_t o[2][3][4];
        // Six rounds of 2 FM independent products (weight plane pa, activation
        // plane pb); four of them carry a quarter of the split, one or two
        // vector instructions per product.  The scheduling fences keep it so.
        auto round = [&](int pa, int pb, bool main, int part) {
            if (part < 4) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint4 v = rb[j][part >> 1];
                    const uint32_t e[4] = {v.x, v.y, v.z, v.w};
                    split2(__uint_as_float(e[2 * (part & 1)]), __uint_as_float(e[2 * (part & 1) + 1]),
                           o[j][0][part], o[j][1][part], o[j][2][part]);
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    Mfma<__bf16>::step(af[pa][i], bc[j][pb], main ? acc[i][j] : low[i][j]);
#pragma unroll
            for (int q = 0; q < 2 * FM; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        read(0);
        read(1);
        __builtin_amdgcn_sched_barrier(0);
        round(0, 0, true, 0);
        read(2);
        round(0, 2, false, 1);
        round(0, 1, false, 2);
        round(1, 1, false, 3);
        load();
        round(1, 0, false, 4);
        round(2, 0, false, 4);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                bn[j][q] = make_uint4(o[j][q][0], o[j][q][1], o[j][q][2], o[j][q][3]);
    };
    int s = 0;
    for (; s + 1 < nst; s += 2) {
        step(s, b0, b1);
        step(s + 1, b1, b0);
    }
    if (s < nst) step(s, b0, b1);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] += low[i][j];

    // ---- sum the K parts, check, then the one-pass epilogue ----
    constexpr int LROW = BM + 4;
    EpiPre<float, BM, BN, NT> epre;
    epre.load(a, m0, co0, tid);
    float* ept = (float*)dyn_smem;
    auto at = [&](int i, int j) {
        return (floatx4*)(ept + (wn * 32 + j * 16 + (lane & 15)) * LROW + i * 16 + 4 * (lane >> 4));
    };
#pragma unroll
    for (int q = KSP - 1; q > 0; --q) {   // part q + (the parts after it)
        __syncthreads();
        if (h == q) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) *at(i, j) = acc[i][j];
        }
        __syncthreads();
        if (h == q - 1) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] += *at(i, j);
        }
    }
    // largest and least magnitude (NaN propagates: v_maximum3, v_minimum3)
    float most = 0.0f;
    bool small = false;
    bool in_m[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) in_m[j] = m0 + wn * 32 + j * 16 + (lane & 15) < a.M;
    if (h == 0) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float least = INFINITY;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = fabsf(acc[i][j][q]);
                    most = __builtin_elementwise_maximum(most, v);
                    least = __builtin_elementwise_minimum(least, v);
                }
                // the tile's padding does not count
                small |= least < p.tiny_max && in_m[j] && co0 + i * 16 + 4 * (lane >> 4) < a.Co;
            }
    }
    const bool odd = !(most < INFINITY);
    bool f32 = false;     // the tile takes the fp32 instruction
    if (__syncthreads_or(odd || small)) {
        f32 = __syncthreads_or(odd);
        // again by each channel's own bound: filters of zeros have sums of zero
        small = false;
        if (h == 0) {
            const auto tsrc = make_rsrc(p.tiny, (uint32_t)a.Co * 4);
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const int co = co0 + i * 16 + 4 * (lane >> 4);
                const floatx4 t = __builtin_bit_cast(
                    floatx4, buf_load16(tsrc, co < a.Co ? (uint32_t)co * 4 : OOB));
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) small |= fabsf(acc[i][j][q]) < t[q] && in_m[j];
            }
        }
        if (__syncthreads_or(small) && !f32) {
            cur.start(a, h * 32);
            lc = h;
            bool lossy = false;
#pragma unroll 1
            for (int q = 0; q < nst; ++q) {
                load();
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const uint32_t e[4] = {rb[j][k].x, rb[j][k].y, rb[j][k].z, rb[j][k].w};
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            lossy |= (e[v] & 0x7fffffffu) - 1u < SPLIT_X_MIN - 1u;
                    }
            }
            f32 = __syncthreads_or(lossy);
        }
    }
    if (h == 0) {
        if (f32) f32_tile<FM>(a, m0 + wn * 32, co0, lane, acc);
        const float unscale = f32 ? 1.0f : SPLIT_UNSCALE;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) *at(i, j) = acc[i][j] * unscale;
    }
    __syncthreads();
    epre.template finish<LROW>(a, ept, m0, co0, tid);
}

template <int FM, int WN, int KSP>
hipError_t launch_one(const SplitArgs& p, hipStream_t s)
{
    constexpr int bytes = split_lds_bytes<FM, WN, KSP>();
    static const hipError_t attr =
        hipFuncSetAttribute((const void*)conv_gemm_split<FM, WN, KSP>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (attr != hipSuccess)
        return attr;
    PPIPE_LAUNCH((conv_gemm_split<FM, WN, KSP>), dim3((unsigned)(p.a.tiles_m * p.a.tiles_co)),
                 dim3(WN * KSP * 64), bytes, s, p);
    return hipGetLastError();
}

}  // namespace

size_t split_weight_bytes(int Co, int K)
{
    return (size_t)((Co + 15) / 16) * ((K + 31) / 32) * 3072;
}

hipError_t launch_split_weights(const void* w, void* w3, int Co, int K, int Kpad, hipStream_t s)
{
    const int chunks = (K + 31) / 32, groups = (Co + 15) / 16;
    const size_t n = (size_t)groups * chunks * 64;
    if (n > 0x7fffffffu)
        return hipErrorInvalidValue;
    PPIPE_LAUNCH(split_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                 (const float*)w, (uint4*)w3, Co, Kpad, chunks, groups);
    return hipGetLastError();
}

float split_tiny(const float* w, int K, float* tiny, int Co, int Kpad)
{
    float top = 0.0f;
    for (int co = 0; co < Co; ++co) {
        uint32_t m = 0;   // bit patterns order as the magnitudes do
        for (int k = 0; k < Kpad; ++k) {
            uint32_t u;
            std::memcpy(&u, w + (size_t)co * Kpad + k, 4);
            m = std::max(m, u & 0x7fffffffu);
        }
        float w_max;
        std::memcpy(&w_max, &m, 4);
        const double t = 0x1p-74 * K * (double)w_max;   // 2^-98 of at least the sum of |w|, scaled
        tiny[co] = std::isfinite(t) ? (float)t : INFINITY;
        top = std::max(top, tiny[co]);
    }
    return top;
}

hipError_t launch_conv_gemm_split(int cfg, const ConvGemmArgs& a, const void* w3,
                                  const float* tiny, float tiny_max, hipStream_t s)
{
    const SplitArgs p{a, w3, tiny, tiny_max};
    switch (cfg) {
    case GEMM_SPLIT_64x128: return launch_one<4, 4, 1>(p, s);
    case GEMM_SPLIT_64x64:  return launch_one<4, 2, 2>(p, s);
    case GEMM_SPLIT_32x64:  return launch_one<2, 2, 2>(p, s);
    case GEMM_SPLIT_32x32:  return launch_one<2, 1, 4>(p, s);
    default:                return hipErrorInvalidValue;
    }
}

}  // namespace ppipe
