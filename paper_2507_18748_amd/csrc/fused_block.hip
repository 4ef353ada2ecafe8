// Inverted-residual blocks in one launch: 1x1 expansion, 3x3 depthwise
// convolution and 1x1 projection (with its residual), 16-bit types.
//
// Run layer by layer, such a block writes and reads its expanded map (six
// times the channels) twice, and the three launches are bound by that traffic
// (MobileNetV2 at batch 32: 90 to 96 MB per launch at 5 TB/s on the 112x112
// maps) or, on small maps, by their latency.  Here a block of four waves owns
// a tile of at most 64 output pixels and walks the expanded channels 32 at a
// time, three chunks in flight:
//   * expansion of chunk i: the tile's input pixels with their halo are MFMA B
//     operands that stay in registers for all chunks (wave w: every fourth
//     group of 16 pixels); folded BN, activation and rounding give the chunk's
//     expanded map in LDS, zero outside the image;
//   * depthwise of chunk i - 1: wave w takes channels 8 w .. + 8 of the chunk,
//     lane l output pixel l, nine conflict-free 16-byte LDS reads; the weights
//     and the folded BN are wave-uniform and sit in scalar registers;
//   * projection of chunk i - 2: wave w's 16 pixels, the depthwise results
//     read back from LDS as MFMA B fragments, accumulated in registers.
// LDS maps are [8-channel vector][pixel][8 channels], two buffers each, and
// one barrier per chunk serves all three.  The expanded and the depthwise map
// are rounded to the storage type where the separate launches round them, and
// every sum runs in the same order, so the output has the same bits.
//
// What bounds it: instruction issue (a lone wave of a SIMD issues a vector
// instruction every 8 to 10 cycles, two waves fill it), about 1 us per chunk
// for a lone block.  Measured as a whole (MobileNetV2 [0, 39), bf16, one graph
// replay, layers -> blocks): batch 1 146 -> 139 us, 5 182 -> 144, 32 313 -> 237,
// 64 476 -> 342.
#include "gemm_device.h"

#include <algorithm>

namespace ppipe {

namespace {

constexpr int FB_THREADS = 256;
constexpr int FB_CH = 32;                 // expanded channels per chunk

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

// acc + x[half] * w[half] with the other half of w zero
template <typename T>
__device__ __forceinline__ float dot2(uint32_t x, uint32_t w, float acc)
{
    if constexpr (std::is_same<T, __bf16>::value)
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x),
                                               __builtin_bit_cast(bf16x2, w), acc, false);
    else
        return __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2, x), __builtin_bit_cast(halfx2, w),
                                      acc, false);
}
typedef float floatx2 __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ uint32_t pack2(float a, float b)   // nearest even
{
    typedef T T2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){a, b}, T2));
}
// Wave-uniform read-only data through the scalar cache.
template <typename V>
__device__ __forceinline__ V uniform_load(const void* p)
{
    return *(const __attribute__((address_space(4))) V*)(uintptr_t)p;
}
__device__ __forceinline__ float clamp_act(float v, float lo, float hi)
{
    return __builtin_amdgcn_fmed3f(v, lo, hi);
}

// Block index with the grid spread over the XCDs in contiguous ranges, so that
// tiles that share halo rows share an L2.
__device__ __forceinline__ uint32_t xcd_range(uint32_t b, uint32_t G)
{
    const uint32_t xcd = b % NUM_XCD, slot = b / NUM_XCD, per = G / NUM_XCD, rem = G % NUM_XCD;
    return xcd * per + (xcd < rem ? xcd : rem) + slot;
}

typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef float floatx8 __attribute__((ext_vector_type(8)));

// S: depthwise stride, NF: 16-pixel input groups per wave (halo of at most 64 NF
// pixels), CFO: 16-channel output fragments.
template <typename T, int S, int NF, int CFO>
__global__ void __launch_bounds__(FB_THREADS, 2)
fused_block_kernel(FusedBlockArgs a)
{
    constexpr int HALO = 64 * NF;
    constexpr int EB = 4 * HALO * 16, DB = 4 * 64 * 16;   // bytes of one chunk
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int Cpad = (a.Ce + FB_CH - 1) / FB_CH * FB_CH;
    unsigned char* s_e = smem;                            // expanded chunk, two buffers
    unsigned char* s_d = smem + 2 * EB;                   // depthwise chunk, two buffers
    float* s_bn = (float*)(smem + 2 * EB + 2 * DB);       // folded BN of the expansion

    int bid = (int)blockIdx.x, grid = (int)gridDim.x;
    asm volatile("" : "+s"(bid), "+s"(grid) : "s"(a.x), "s"(a.we), "s"(a.wd), "s"(a.wp), "s"(a.se),
                 "s"(a.be), "s"(a.sd), "s"(a.bd), "s"(a.sp), "s"(a.bp), "s"(a.res), "s"(a.y),
                 "s"(a.H), "s"(a.W), "s"(a.C), "s"(a.Ce), "s"(a.Co), "s"(a.Ho), "s"(a.Wo),
                 "s"(a.TH), "s"(a.TW), "s"(a.tiles_h), "s"(a.tiles_w));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, r = lane & 15;
    int t = (int)xcd_range((uint32_t)bid, (uint32_t)grid);
    const int tw = t % a.tiles_w;
    t /= a.tiles_w;
    const int th = t % a.tiles_h, n = t / a.tiles_h;
    const int oh0 = th * a.TH, ow0 = tw * a.TW;                // first output of the tile
    const int ih0 = oh0 * S - a.pad, iw0 = ow0 * S - a.pad;    // its halo's origin
    const int HW = (a.TW - 1) * S + 3, HH = (a.TH - 1) * S + 3, hpx = HH * HW;
    const int nch = Cpad / FB_CH;

    // ---- weights of the chunk to come: expansion rows, projection columns ----
    const auto wesrc = make_rsrc(a.we, (uint32_t)a.Ce * a.Kpe * 2);
    const auto wpsrc = make_rsrc(a.wp, (uint32_t)a.Co * a.Kpp * 2);
    uint4 ae[2], ap[CFO];
    // A row past the last lies past the buffer (c0 + 8 q < Kpp, 8 q < Kpe), where
    // the range check gives zeros.  Row tests and masks kept here as scalar pairs
    // made the loop spill scalar registers (64 output channels at stride 2: 123
    // moves to and from lanes per chunk).
    const uint32_t e_off = (uint32_t)(r * a.Kpe + 8 * q) * 2u, p_off = (uint32_t)(r * a.Kpp + 8 * q) * 2u;
    auto load_e = [&](int c0) {
#pragma unroll
        for (int f = 0; f < 2; ++f)
            ae[f] = buf_load16(wesrc, e_off + (uint32_t)((c0 + 16 * f) * a.Kpe * 2));
    };
    auto load_p = [&](int c0) {
#pragma unroll
        for (int f = 0; f < CFO; ++f)
            ap[f] = buf_load16(wpsrc, p_off + (uint32_t)((16 * f * a.Kpp + c0) * 2));
    };
    load_e(0);

    // ---- input pixels of the halo: groups wave, wave + 4, ... ----
    const auto xsrc = make_rsrc(a.x, (uint32_t)a.N * a.H * a.W * a.C * 2);
    uint4 xb[NF];
    uint32_t inside[NF];     // ones where the lane's pixel of group f is in the image
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int p = (f * 4 + wave) * 16 + r;
        const int hr = p / HW, hc = p - hr * HW;
        const int ih = ih0 + hr, iw = iw0 + hc;
        const bool ok = p < hpx && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
        inside[f] = ok ? 0xffffffffu : 0u;
        xb[f] = buf_load16(xsrc, ok && 8 * q < a.C
                                     ? (uint32_t)(((n * a.H + ih) * a.W + iw) * a.C + 8 * q) * 2u : OOB);
    }
    for (int i = tid; i < Cpad; i += FB_THREADS) {
        s_bn[i] = i < a.Ce ? a.se[i] : 0.0f;
        s_bn[Cpad + i] = i < a.Ce ? a.be[i] : 0.0f;
    }

    // depthwise: lane l is output pixel l of the tile (past the tile: pixel 0)
    const int orow = lane < a.TH * a.TW ? lane / a.TW : 0;
    const int ocol = lane < a.TH * a.TW ? lane - orow * a.TW : 0;
    const int e_rd = (wave * HALO + (orow * S) * HW + ocol * S) * 16;
    const int d_wr = (wave * 64 + lane) * 16;
    // projection: lane l is pixel 16 wave + l % 16, channels 8 (l / 16) .. + 8
    const int d_rd = (q * 64 + wave * 16 + r) * 16;

    const float elo = a.acte == ACT_NONE ? -INFINITY : 0.0f, ehi = a.acte == ACT_RELU6 ? 6.0f : INFINITY;
    const float dlo = a.actd == ACT_NONE ? -INFINITY : 0.0f, dhi = a.actd == ACT_RELU6 ? 6.0f : INFINITY;

    // epilogue: lane's pixel 16 wave + r, channels 16 f + 4 q .. + 4; the addresses
    // wait in vector registers (the loop needs the scalar ones)
    T* yp = nullptr;
    const T* rp = nullptr;
    const float *scp = a.sp + 4 * q, *bip = a.bp + 4 * q;
    {
        const int p = wave * 16 + r, prow = p / a.TW, oh = oh0 + prow, ow = ow0 + p - prow * a.TW;
        if (p < a.TH * a.TW && oh < a.Ho && ow < a.Wo) {
            const size_t base = ((size_t)(n * a.Ho + oh) * a.Wo + ow) * a.Co + 4 * q;
            yp = (T*)a.y + base;
            rp = a.res ? (const T*)a.res + base : nullptr;
        }
    }
    asm volatile("" : "+v"(yp), "+v"(rp));

    floatx4 acc[CFO];
#pragma unroll
    for (int f = 0; f < CFO; ++f) acc[f] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    uintx4 dw[9];            // depthwise weights, scale and shift of the wave's channels
    floatx8 dsc, dbi;
    auto load_d = [&](int c0) {
        const int c = min(c0 + 8 * wave, a.Ce - 8);
#pragma unroll
        for (int k = 0; k < 9; ++k)
            dw[k] = uniform_load<uintx4>((const char*)a.wd + (uint32_t)((k * a.Ce + c) * 2));
        dsc = uniform_load<floatx8>((const char*)a.sd + (uint32_t)(c * 4));
        dbi = uniform_load<floatx8>((const char*)a.bd + (uint32_t)(c * 4));
    };

    auto expand = [&](int i) {
        unsigned char* E = s_e + (i & 1) * EB;
        floatx4 v[NF][2];
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v[f][h] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
                Mfma<T>::step(ae[h], xb[f], v[f][h]);
            }
        if (i + 1 < nch) load_e((i + 1) * FB_CH);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float4 sc = *(const float4*)(s_bn + i * FB_CH + 16 * h + 4 * q);
            const float4 bi = *(const float4*)(s_bn + Cpad + i * FB_CH + 16 * h + 4 * q);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const floatx4 w = v[f][h];
                uint2 u;
                u.x = pack2<T>(clamp_act(w[0] * sc.x + bi.x, elo, ehi),
                               clamp_act(w[1] * sc.y + bi.y, elo, ehi));
                u.y = pack2<T>(clamp_act(w[2] * sc.z + bi.z, elo, ehi),
                               clamp_act(w[3] * sc.w + bi.w, elo, ehi));
                u.x &= inside[f];
                u.y &= inside[f];
                *(uint2*)(E + ((2 * h + (q >> 1)) * HALO + (f * 4 + wave) * 16 + r) * 16 + (q & 1) * 8) = u;
            }
        }
    };
    auto depthwise = [&](int i) {
        const unsigned char* E = s_e + (i & 1) * EB + e_rd;
        uint4 x[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) x[k] = *(const uint4*)(E + ((k / 3) * HW + k % 3) * 16);
        float d[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) d[c] = 0.0f;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const uint32_t xw[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                d[2 * c] = dot2<T>(xw[c], dw[k][c] & 0xffffu, d[2 * c]);
                d[2 * c + 1] = dot2<T>(xw[c], dw[k][c] & 0xffff0000u, d[2 * c + 1]);
            }
        }
        uint32_t o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            o[c] = pack2<T>(clamp_act(fmaf(d[2 * c], dsc[2 * c], dbi[2 * c]), dlo, dhi),
                            clamp_act(fmaf(d[2 * c + 1], dsc[2 * c + 1], dbi[2 * c + 1]), dlo, dhi));
        // channels past the last (a half chunk): zeros
        const bool in = i * FB_CH + 8 * wave < a.Ce;
        *(uint4*)(s_d + (i & 1) * DB + d_wr) = make_uint4(in ? o[0] : 0u, in ? o[1] : 0u,
                                                          in ? o[2] : 0u, in ? o[3] : 0u);
        if (i + 1 < nch) load_d((i + 1) * FB_CH);
    };
    auto project = [&](int i) {
        const uint4 b = *(const uint4*)(s_d + (i & 1) * DB + d_rd);
#pragma unroll
        for (int f = 0; f < CFO; ++f) Mfma<T>::step(ap[f], b, acc[f]);
        if (i + 1 < nch) load_p((i + 1) * FB_CH);
    };

    __syncthreads();         // the expansion's folded BN
    expand(0);
    load_d(0);
    __syncthreads();
    if (nch > 1) expand(1);
    load_p(0);
    depthwise(0);
    __syncthreads();
    for (int i = 2; i < nch; ++i) {
        project(i - 2);
        expand(i);
        depthwise(i - 1);
        __syncthreads();
    }
    if (nch > 1) {
        project(nch - 2);
        depthwise(nch - 1);
        __syncthreads();
    }
    project(nch - 1);

    // ---- epilogue: lane holds four output channels of its pixel ----
    if (!yp)
        return;
    const float plo = a.actp == ACT_NONE ? -INFINITY : 0.0f, phi = a.actp == ACT_RELU6 ? 6.0f : INFINITY;
#pragma unroll
    for (int f = 0; f < CFO; ++f) {
        const int co = 16 * f + 4 * q;
        if (co >= a.Co)
            continue;
        const float4 s4 = *(const float4*)(scp + 16 * f), b4 = *(const float4*)(bip + 16 * f);
        float4 v = make_float4(acc[f][0] * s4.x + b4.x, acc[f][1] * s4.y + b4.y,
                               acc[f][2] * s4.z + b4.z, acc[f][3] * s4.w + b4.w);
        if (rp) {
            const float4 z = Vec4<T>::load(rp + 16 * f);
            v.x += z.x; v.y += z.y; v.z += z.z; v.w += z.w;
        }
        v.x = clamp_act(v.x, plo, phi); v.y = clamp_act(v.y, plo, phi);
        v.z = clamp_act(v.z, plo, phi); v.w = clamp_act(v.w, plo, phi);
        Vec4<T>::store(yp + 16 * f, v);
    }
}

int halo_groups(int stride) { return stride == 2 ? 5 : 2; }   // NF
int fused_block_lds(int Ce, int stride)
{
    const int cpad = (Ce + FB_CH - 1) / FB_CH * FB_CH;
    return 2 * 4 * 64 * halo_groups(stride) * 16 + 2 * 4 * 64 * 16 + 2 * cpad * 4;
}

template <typename T, int S, int NF, int CFO>
hipError_t launch_one(const FusedBlockArgs& a, hipStream_t s)
{
    static const hipError_t attr =
        hipFuncSetAttribute((const void*)fused_block_kernel<T, S, NF, CFO>,
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            fused_block_lds(FUSED_MAX_CE, S));
    if (attr != hipSuccess)
        return attr;
    PPIPE_LAUNCH((fused_block_kernel<T, S, NF, CFO>),
                 dim3((unsigned)(a.N * a.tiles_h * a.tiles_w)), dim3(FB_THREADS),
                 fused_block_lds(a.Ce, a.stride), s, a);
    return hipGetLastError();
}
template <typename T, int S, int NF>
hipError_t launch_co(const FusedBlockArgs& a, hipStream_t s)
{
    if (a.Co <= 16) return launch_one<T, S, NF, 1>(a, s);
    if (a.Co <= 32) return launch_one<T, S, NF, 2>(a, s);
    return launch_one<T, S, NF, 4>(a, s);
}
template <typename T>
hipError_t launch_t(const FusedBlockArgs& a, hipStream_t s)
{
    const int px = ((a.TH - 1) * a.stride + 3) * ((a.TW - 1) * a.stride + 3);
    if (a.TH * a.TW > 64 || px > 64 * halo_groups(a.stride) || a.Co > FUSED_MAX_CO ||
        a.C > FUSED_MAX_C || a.Ce > FUSED_MAX_CE)
        return hipErrorInvalidValue;
    return a.stride == 1 ? launch_co<T, 1, 2>(a, s) : launch_co<T, 2, 5>(a, s);
}

}  // namespace

void fused_block_tile(int Ho, int Wo, int stride, int* TH, int* TW)
{
    double best = 0.0;
    for (int w = 1; w <= std::min(64, Wo); ++w)
        for (int h = 1; h * w <= 64 && h <= Ho; ++h) {
            const int px = ((h - 1) * stride + 3) * ((w - 1) * stride + 3);
            if (px > 64 * halo_groups(stride)) continue;
            const int nt = ((Ho + h - 1) / h) * ((Wo + w - 1) / w);
            // every tile costs the same whatever it holds; among equals the
            // smaller halo, then the wider tile
            const double cost = nt + px * 1e-4 - w * 1e-7;
            if (best == 0.0 || cost < best) {
                best = cost;
                *TH = h;
                *TW = w;
            }
        }
}

hipError_t launch_fused_block(int dt, const FusedBlockArgs& a, hipStream_t s)
{
    switch (dt) {
    case DT_F16:  return launch_t<_Float16>(a, s);
    case DT_BF16: return launch_t<__bf16>(a, s);
    default:      return hipErrorInvalidValue;
    }
}

const char* fused_block_name(int dt, int stride)
{
    static const char* n[2][2] = {{"fused_block<f16,s1>", "fused_block<f16,s2>"},
                                  {"fused_block<bf16,s1>", "fused_block<bf16,s2>"}};
    return n[dt == DT_BF16][stride == 2];
}

}  // namespace ppipe
