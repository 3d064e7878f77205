// Device-side helpers shared by the kernel files of libnpas (HIP only): storage conversions, the activations as
// one clamp, MFMA wrappers, fast division, streaming accesses.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "npas_internal.h"

namespace npas {

// Raises a kernel's dynamic LDS limit once per process (one std::once_flag per kernel instantiation).
template <typename K> static void allow_lds_once(std::once_flag &once, K kern, int bytes)
{
    std::call_once(once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    });
}

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

__device__ __forceinline__ uint32_t fastdiv(uint32_t n, uint32_t magic)
{
    return magic ? __umulhi(n, magic) : n; // magic = ceil(2^32 / d), 0 for d == 1; exact while n * d < 2^32
}
// The same exact for every n below 2^32 - d: the reciprocal is at most one too high (n * (d * magic - 2^32) < n * d), which the product shows.
__device__ __forceinline__ uint32_t fastdiv_any(uint32_t n, uint32_t magic, uint32_t d)
{
    const uint32_t q = fastdiv(n, magic);
    return q * d > n ? q - 1u : q;
}
// The same for every n below 2^31 from a reciprocal of 32 significant bits (magic_div_wide), without a second product: for vectors of pixels.
__device__ __forceinline__ uint32_t fastdiv_wide(uint32_t n, WideDiv d) { return d.magic ? __umulhi(n, d.magic) >> d.shift : n; }

// Streaming (non-temporal) 8-byte accesses for tensors that are written or read once per launch and
// are far larger than the L2: they leave the cache to the operands that are reused.
__device__ __forceinline__ void store_stream8(void *p, uint2 v)
{
    __builtin_nontemporal_store(__builtin_bit_cast(unsigned long long, v), reinterpret_cast<unsigned long long *>(p));
}
__device__ __forceinline__ uint2 load_stream8(const void *p)
{
    return __builtin_bit_cast(uint2, __builtin_nontemporal_load(reinterpret_cast<const unsigned long long *>(p)));
}
__device__ __forceinline__ void store_stream16(void *p, uint4 v)
{
    typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), reinterpret_cast<u32x4 *>(p));
}
__device__ __forceinline__ uint4 load_stream16(const void *p)
{
    typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p)));
}

__device__ __forceinline__ float act_apply(float v, int act)
{
    if (act == NPAS_ACT_RELU) return fmaxf(v, 0.0f);
    if (act == NPAS_ACT_RELU6) return fminf(fmaxf(v, 0.0f), 6.0f);
    if (act == NPAS_ACT_HARDSWISH) return v * fminf(fmaxf(v + 3.0f, 0.0f), 6.0f) * (1.0f / 6.0f);
    return v;
}

// The activations as one clamp to [lo, hi] (none: +-inf, ReLU: [0, inf), ReLU6: [0, 6]); hard-swish
// (v * clamp(v + 3, 0, 6) / 6) is that clamp of v + 3 times v / 6, behind a wave-uniform flag.
struct Clamp {
    float lo, hi;
    bool hs;
};
__device__ __forceinline__ Clamp clamp_of(int act)
{
    return Clamp{act == NPAS_ACT_NONE ? -INFINITY : 0.0f, (act == NPAS_ACT_RELU6 || act == NPAS_ACT_HARDSWISH) ? 6.0f : INFINITY,
                 act == NPAS_ACT_HARDSWISH};
}
// HSW: the launch has a hard-swish somewhere (a kernel body is instantiated with and without; without, an activation
// is the one clamp instruction and nothing else)
template <bool HSW = true> __device__ __forceinline__ float clampf(float v, Clamp c)
{
    if (HSW && c.hs) return v * __builtin_amdgcn_fmed3f(v + 3.0f, 0.0f, 6.0f) * (1.0f / 6.0f);
    return __builtin_amdgcn_fmed3f(v, c.lo, c.hi);
}

// fp32 -> 16-bit storage, round to nearest even.
template <int DT> __device__ __forceinline__ uint16_t to_storage(float v)
{
    if (DT == NPAS_BF16) {
        uint32_t u = __float_as_uint(v);
        if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40); // NaN stays NaN
        u += 0x7fffu + ((u >> 16) & 1u);
        return (uint16_t)(u >> 16);
    } else {
        _Float16 h = (_Float16)v;
        return __builtin_bit_cast(uint16_t, h);
    }
}

// two fp32 -> one dword of two 16-bit storage values (lo, hi), round to nearest even
template <int DT> __device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    if (DT == NPAS_BF16) {
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
    } else {
        typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, f16x2));
    }
}

template <int DT> __device__ __forceinline__ float from_storage(uint16_t b)
{
    if (DT == NPAS_BF16) return __uint_as_float((uint32_t)b << 16);
    return (float)__builtin_bit_cast(_Float16, b);
}

// element i of an activation tensor of storage type DT as fp32, and back
template <int DT> __device__ __forceinline__ float ld_act(const void *p, size_t i)
{
    if (DT == NPAS_F32) return reinterpret_cast<const float *>(p)[i];
    return from_storage<DT>(reinterpret_cast<const uint16_t *>(p)[i]);
}
template <int DT> __device__ __forceinline__ void st_act(void *p, size_t i, float v)
{
    if (DT == NPAS_F32) reinterpret_cast<float *>(p)[i] = v;
    else reinterpret_cast<uint16_t *>(p)[i] = to_storage<DT>(v);
}

template <int DT> __device__ __forceinline__ f32x4 mfma16(uint4 a, uint4 b, f32x4 c)
{
    if (DT == NPAS_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous run
// of logical ids so that workgroups sharing an activation patch share an L2.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t wg, uint32_t nwg)
{
    uint32_t xcd = wg & 7u, idx = wg >> 3, q = nwg >> 3, r = nwg & 7u;
    return xcd * q + (xcd < r ? xcd : r) + idx;
}

// Direct loads take their LDS address from M0, which the ISA wants written a wait state before a load to LDS reads it; inside an asm statement
// the compiler does not see to that.  (M0 is reserved: the compiler keeps nothing in it across statements.)
#define NPAS_M0_FROM_ARG0 "s_mov_b32 m0, %0\n\ts_nop 0\n\t"

// Direct global -> LDS load: 64 lanes x 16 bytes land lane-linearly in the 1 KB block at lds_addr; nothing is held in registers.
__device__ __forceinline__ void lds_dma16(const void *gptr, uint32_t lds_addr)
{
    asm volatile(NPAS_M0_FROM_ARG0 "global_load_lds_dwordx4 %1, off"
                 :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(gptr)
                 : "memory");
}

// The same with 4 bytes a lane (256 bytes of LDS).
__device__ __forceinline__ void lds_dma4(const void *gptr, uint32_t lds_addr)
{
    asm volatile(NPAS_M0_FROM_ARG0 "global_load_lds_dword %1, off"
                 :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(gptr)
                 : "memory");
}

// Raw buffer descriptor of `bytes` bytes at p: loads past them give zeros, stores past them vanish.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
__device__ __forceinline__ u32x4 buffer_of(const void *p, uint32_t bytes)
{
    const uint64_t u = (uint64_t)(uintptr_t)p;
    return u32x4{(uint32_t)u, (uint32_t)(u >> 32) & 0xffffu, bytes, 0x00020000u};
}
// Direct buffer -> LDS load: 64 lanes x 16 bytes land lane-linearly in the 1 KB block at lds_addr.
__device__ __forceinline__ void lds_buffer16(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds_addr)
{
    asm volatile(NPAS_M0_FROM_ARG0 "buffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory");
}

// Index of a 1 KB image of ring-format weights on nch 64-channel chunks: filters 64 f64 .. + 63, 32-channel step, image 0 .. 3 (row r is filter 4 r + image)
__device__ __forceinline__ uint32_t ring_image(uint32_t nch, uint32_t f64, uint32_t step, uint32_t image)
{
    return ((f64 >> 1) * nch + (step >> 1)) * 16u + (step & 1u) * 8u + (f64 & 1u) * 4u + image;
}

// Where the bias of filter f lies so that a lane reads its results' in their order: [64-filter chunk][quarter q][image j][i] for f = 16 q + 4 i + j
__device__ __forceinline__ uint32_t result_slot(uint32_t f) { return (f & ~15u) | (f & 3u) * 4u | (f >> 2 & 3u); }

// "At most n vector-memory operations of this wave outstanding" for a wave-uniform n < 64
// (the instruction takes an immediate).
__device__ __forceinline__ void wait_vmcnt(uint32_t n)
{
#define NPAS_W(k) case k: asm volatile("s_waitcnt vmcnt(" #k ")" ::: "memory"); break;
    switch (n) {
        NPAS_W(0) NPAS_W(1) NPAS_W(2) NPAS_W(3) NPAS_W(4) NPAS_W(5) NPAS_W(6) NPAS_W(7) NPAS_W(8) NPAS_W(9) NPAS_W(10)
        NPAS_W(11) NPAS_W(12) NPAS_W(13) NPAS_W(14) NPAS_W(15) NPAS_W(16) NPAS_W(17) NPAS_W(18) NPAS_W(19) NPAS_W(20)
        NPAS_W(21) NPAS_W(22) NPAS_W(23) NPAS_W(24) NPAS_W(25) NPAS_W(26) NPAS_W(27) NPAS_W(28) NPAS_W(29) NPAS_W(30)
        NPAS_W(31) NPAS_W(32) NPAS_W(33) NPAS_W(34) NPAS_W(35) NPAS_W(36) NPAS_W(37) NPAS_W(38) NPAS_W(39) NPAS_W(40)
        NPAS_W(41) NPAS_W(42) NPAS_W(43) NPAS_W(44) NPAS_W(45) NPAS_W(46) NPAS_W(47) NPAS_W(48) NPAS_W(49) NPAS_W(50)
        NPAS_W(51) NPAS_W(52) NPAS_W(53) NPAS_W(54) NPAS_W(55) NPAS_W(56) NPAS_W(57) NPAS_W(58) NPAS_W(59) NPAS_W(60)
        NPAS_W(61) NPAS_W(62)
    default: asm volatile("s_waitcnt vmcnt(63)" ::: "memory"); break;
    }
#undef NPAS_W
}

// The sums of NF consecutive outputs (pixel m, filters f .. f + NF - 1 of one quad) over their kept weights, in channel order, from
// ring-format images: for the kernels that multiply the zeros of pruned weights too and meet an infinite input.  16 bytes a load (in a plain
// loop: it needs few registers beside the next item's weights), and an end as soon as all sums are NaN, because a map that has overflowed comes here
// with all its outputs: 14 x 14 x 256 3x3 at batch 128, all inputs NaN 45 ms -> 0.11, one infinite channel 45 -> 4.4, one infinite value 8 -> 1.1.
// (The kernel's arguments, a struct with the geometry fields, are read again: kept for this they would take registers from the loop.)
// (AT: bytes of the arguments in front of the struct.)
template <int DT, typename Args, int NF, int AT = 0> __device__ __forceinline__ void kept_sums(uint32_t m, uint32_t f, float (&v)[NF])
{
    auto ka = (const __attribute__((address_space(4))) Args *)((const __attribute__((address_space(4))) uint8_t *)__builtin_amdgcn_kernarg_segment_ptr() + AT);
    asm volatile("" : "+s"(ka));
    const auto &a = *ka;
    const uint32_t n = m / (uint32_t)(a.Ho * a.Wo), p = m - n * (uint32_t)(a.Ho * a.Wo), oy = p / (uint32_t)a.Wo, ox = p - oy * (uint32_t)a.Wo;
    const int T = a.KH * a.KW, nch = a.C >> 6;
    const uint32_t img = (f >> 6 & 1u) * 4u + (f & 3u), r = f >> 2 & 15u; // first image of the 128-filter block, row of the images
    const uint16_t *w = reinterpret_cast<const uint16_t *>(a.wimg) + ((size_t)(f >> 7) * nch * T * 16 + img) * 512 + r * 8;
#pragma unroll
    for (int j = 0; j < NF; ++j) v[j] = 0.f;
    bool all = false;
#pragma unroll 1
    for (int t = 0; t < T && !all; ++t) {
        const int iy = (int)oy * a.stride - a.pad + t / a.KW, ix = (int)ox * a.stride - a.pad + t % a.KW;
        const bool in = (uint32_t)iy < (uint32_t)a.H && (uint32_t)ix < (uint32_t)a.W;
        const uint16_t *x = reinterpret_cast<const uint16_t *>(a.x) + (((size_t)n * a.H + iy) * a.W + ix) * a.C, *wt = w + (size_t)t * 8192;
#pragma unroll 1
        for (int s = in ? 0 : 8 * nch; s < 8 * nch && !all; ++s) { // 8 channels
            const uint4 xv = *reinterpret_cast<const uint4 *>(x + s * 8);
            const uint32_t xs[4] = {xv.x, xv.y, xv.z, xv.w};
            const uint16_t *ws = wt + (size_t)(s >> 3) * T * 8192 + (s >> 2 & 1) * 4096 + (s & 3) * 128;
            uint4 wv[NF];
#pragma unroll
            for (int j = 0; j < NF; ++j) wv[j] = *reinterpret_cast<const uint4 *>(ws + j * 512);
            all = true;
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                const uint32_t wc[4] = {wv[j].x, wv[j].y, wv[j].z, wv[j].w};
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint16_t c = (uint16_t)(wc[i >> 1] >> (i & 1) * 16);
                    const float sum = fmaf(from_storage<DT>(c), from_storage<DT>((uint16_t)(xs[i >> 1] >> (i & 1) * 16)), v[j]);
                    v[j] = c & 0x7fffu ? sum : v[j];
                }
                all = all && v[j] != v[j];
            }
        }
    }
}

} // namespace npas
