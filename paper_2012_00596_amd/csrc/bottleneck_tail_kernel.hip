// End of a bottleneck block and the first layer of the next one as one launch (gfx950, 16-bit storage):
//   y = act3(W3 a + residual + b3)          64 -> 256 channels       (or W3 a + Wsc x2 + b3 + bsc: a projection shortcut from 64 channels)
//   z = act1(W1 y + b1)                     256 -> 64 or 128 channels
// y is written once and is not read again for z; with the projection its own output never exists.
//
// Bound: HBM.  Per pixel 2 (64 + 256 + 256 + G) bytes (64 + 64 + 256 + G with the projection) against 2 (64 + 3 x 256 + G) in two launches
// (2 (2 x 64 + 4 x 256 + G) in three).  All weights (64 .. 128 KB) lie in LDS for the life of the workgroup, so there is no ring and no barrier: a
// wave is a stream of its own, 16 pixels at a time, and keeps the next 16 pixels' inputs (10 KB) on their way in registers.  Sixteen waves a
// CU are 160 KB in flight.  Every weight image is read from LDS for one MFMA only: a quarter of the LDS rate at the speed of HBM.
// 401408 pixels, bf16, inside the 50-layer stack: with the projection, G = 64, 165 us in three launches -> 62 (5.8 TB/s); with a residual, G = 64, 128 in
// two -> 91 (5.6 TB/s), G = 128 137 -> 105.
//
// The weights are the row operand, the pixels the column operand.  Row r of image j of 64 filters is filter 4 r + j, so that a lane's results of four
// images are sixteen consecutive channels of its pixel and, rounded, two column operands of the next layer's reduction (whose order of channels is
// free: its images are read from LDS in the same one).  So the images lie in LDS as they lie in memory, 1 KB a load; put together from 16-byte
// pieces in another order they took 7 us of every launch (25088 pixels with the projection, G = 64, 16.2 -> 12.8 us, with a residual 15.8 -> 14.0).
// A lane's two vectors are one 128-byte line of its pixel together with three other lanes; accesses of half a line each took 150 us where whole
// ones (swap_lines) take 105.
// Blocks are dealt to the workgroups one by one, so that a last round of few blocks is spread over all CUs: in runs of 16, 105 -> 93.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "npas_internal.h"
#include "device_util.h"

namespace npas {

constexpr int kTailWaves = 16;

template <int DT, int NG, bool JOIN>
__global__ __launch_bounds__(kTailWaves * 64) void bottleneck_tail_kernel(TailArgs a)
{
    constexpr int NU = 8, NS = JOIN ? 4 : 2;                 // 32-filter chunks of y; 32-deep steps of its reduction
    constexpr uint32_t kY = NU * 2 * NS, kZ = NU * 2 * NG;   // weight images of the two layers
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n16 = lane & 15, q = lane >> 4;
    const auto buf = [](const void *p, uint32_t bytes) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
    };
    // (loads of pixels past the last one give zeros, stores vanish: the descriptors' ranges end with the tensors)
    const __amdgpu_buffer_rsrc_t ar = buf(a.a, a.M * 128u), rr = buf(JOIN ? a.x2 : a.r, a.M * (JOIN ? 128u : 512u)), yr = buf(a.y, a.M * 512u),
                                 zr = buf(a.z, a.M * (uint32_t)(NG * 64));
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    constexpr int kStream = 2; // streaming access
    const auto load = [](__amdgpu_buffer_rsrc_t r, uint32_t off) __attribute__((always_inline)) {
        return __builtin_bit_cast(uint4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kStream));
    };
    const auto store = [](__amdgpu_buffer_rsrc_t r, uint32_t off, uint4 v) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)off, 0, kStream);
    };
    const Clamp c3 = clamp_of(a.act3), c1 = clamp_of(a.act1);
    // half h of the results of a 64-filter chunk, clamped and rounded: eight consecutive channels of a pixel
    const auto rounded = [](const f32x4 *d, int h, Clamp c) __attribute__((always_inline)) {
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = pack2<DT>(__builtin_amdgcn_fmed3f(d[2 * (i & 1)][2 * h + (i >> 1)], c.lo, c.hi), __builtin_amdgcn_fmed3f(d[2 * (i & 1) + 1][2 * h + (i >> 1)], c.lo, c.hi));
        return uint4{o[0], o[1], o[2], o[3]};
    };

    // A 128-byte line of a pixel is two such vectors of a lane.  Eight lanes hold half a line of their pixel; swapped with the lane eight pixels on,
    // one access of the wave covers eight whole lines (first: pixels 0 .. 7 of the block, second: 8 .. 15).
    const bool upper = n16 >= 8;
    const auto swap_lines = [&](uint4 &v0, uint4 &v1) __attribute__((always_inline)) {
        uint32_t x[4] = {v0.x, v0.y, v0.z, v0.w}, y[4] = {v1.x, v1.y, v1.z, v1.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(upper ? x[i] : y[i]), 0x128, 0xf, 0xf, false); // rotated by 8 lanes of 16
            x[i] = upper ? t : x[i];
            y[i] = upper ? y[i] : t;
        }
        v0 = uint4{x[0], x[1], x[2], x[3]};
        v1 = uint4{y[0], y[1], y[2], y[3]};
    };
    const uint32_t nblk = (a.M + 15u) >> 4, stride = gridDim.x * (uint32_t)kTailWaves;
    uint32_t blk = (uint32_t)wave * gridDim.x + blockIdx.x;
    // pixel and byte of a line access: of a lane's operand (8 channels of each half line), of its results (16 consecutive channels)
    const uint32_t lane_line = ((uint32_t)n16 & 7u), lane_vec = 16u * (uint32_t)q + (upper ? 64u : 0u), lane_res = 32u * (uint32_t)q + (upper ? 16u : 0u);
    uint4 av[NS], rv[JOIN ? 1 : 8];
    const auto fetch_a = [&](uint32_t b, uint4 (&v)[NS]) __attribute__((always_inline)) {
        const uint32_t o = (b * 16u + lane_line) * 128u + lane_vec;
#pragma unroll
        for (int s = 0; s < NS; ++s) v[s] = load(s < 2 ? ar : rr, o + 1024u * (s & 1));
    };
    fetch_a(blk, av);
    if (!JOIN) {
#pragma unroll
        for (int k = 0; k < 8; ++k) rv[k] = load(rr, (blk * 16u + lane_line + 8u * (k & 1)) * 512u + lane_res + 128u * (k >> 1));
    }
    {   // images in LDS as they lie in memory: [64-filter chunk][step][image] of the first layer, [step][64-filter chunk][image] of the second; then the biases
        const uint32_t lbase = (uint32_t)(uintptr_t)lds;
        for (uint32_t i = (uint32_t)wave; i < kY + kZ; i += kTailWaves) {
            const void *src = a.w1;
            uint32_t img;
            if (i < kY) {
                const uint32_t s = i / 4 % NS;
                if (s < 2) src = a.w3;
                else src = a.wsc;
                img = ring_image(1u, i / (4 * NS), s & 1u, i & 3u);
            } else img = ring_image(4u, (i - kY) / 4 % (NG / 2), (i - kY) / (2 * NG), i & 3u);
            lds_dma16(reinterpret_cast<const uint8_t *>(src) + (size_t)img * 1024u + (uint32_t)lane * 16u, lbase + i * 1024u);
        }
        float *lb = reinterpret_cast<float *>(lds + (kY + kZ) * 1024u);
        if (tid < 32 * NU + 32 * NG) {
            float b = 0.f;
            if (tid < 32 * NU) {
                if (a.b3) b += a.b3[tid];
                if (JOIN && a.bsc) b += a.bsc[tid];
            } else if (a.b1) b = a.b1[tid - 32 * NU];
            lb[result_slot((uint32_t)tid)] = b;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    while (blk < nblk) {
        const uint32_t next = blk + stride, yo = (blk * 16u + lane_line) * 512u + lane_res, ro = yo + stride * 16u * 512u;
        uint4 an[NS];
        fetch_a(next, an);
#pragma unroll
        for (int s = 0; s < NS; s += 2) swap_lines(av[s], av[s + 1]);
        // (of 64 channels of y a lane holds 16 q .. 16 q + 15 as two operands, so its weights for operand h are the vector 2 q + h of the chunk's eight)
        uint32_t wo = (uint32_t)lane * 16u, zo2 = (uint32_t)(n16 + 32 * (q & 1)) * 16u + (uint32_t)(q >> 1) * (2u * NG * 1024u), bo = (kY + kZ) * 1024u + 64u * (uint32_t)q;
        asm volatile("" : "+v"(wo), "+v"(zo2), "+v"(bo)); // keeps the weights from being read (and held) outside the loop
        const uint8_t *wl = lds + wo, *zl = lds + zo2, *bl = lds + bo;
        f32x4 z[2 * NG]; // [64-filter chunk, image j][i]: filter 16 q + 4 i + j of the chunk
        const auto biases = [&](int f, f32x4 *d) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = *reinterpret_cast<const f32x4 *>(bl + f * 4 + 16 * j);
        };
#pragma unroll
        for (int w = 0; w < NG / 2; ++w) biases(32 * NU + 64 * w, z + 4 * w);
#pragma unroll
        for (int c = 0; c < NU / 2; ++c) { // 64 channels of y
            if (!JOIN) swap_lines(rv[2 * c], rv[2 * c + 1]);
            f32x4 d[4];
            biases(64 * c, d);
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) d[j] = mfma16<DT>(*reinterpret_cast<const uint4 *>(wl + ((c * NS + s) * 4 + j) * 1024), av[s], d[j]);
            if (!JOIN) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t r[4] = {rv[2 * c + h].x, rv[2 * c + h].y, rv[2 * c + h].z, rv[2 * c + h].w};
#pragma unroll
                    for (int i = 0; i < 8; ++i) d[i & 3][2 * h + (i >> 2)] += from_storage<DT>((uint16_t)(r[i >> 1] >> 16 * (i & 1)));
                }
            }
            uint4 o[2] = {rounded(d, 0, c3), rounded(d, 1, c3)};
            if (!JOIN) {
#pragma unroll
                for (int h = 0; h < 2; ++h) rv[2 * c + h] = load(rr, ro + 4096u * h + 128u * c);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int v = 0; v < 2 * NG; ++v) z[v] = mfma16<DT>(*reinterpret_cast<const uint4 *>(zl + (kY + 4 * c * NG + v) * 1024 + 256 * h), o[h], z[v]);
            swap_lines(o[0], o[1]);
#pragma unroll
            for (int h = 0; h < 2; ++h) store(yr, yo + 4096u * h + 128u * c, o[h]);
            if (JOIN || NG == 2) __builtin_amdgcn_sched_barrier(0); // (the next chunk's images read here cost spills, 63 -> 80 us; with a rolled loop the waits count stores)
        }
        const uint32_t zo = (blk * 16u + lane_line) * (uint32_t)(NG * 64) + lane_res;
#pragma unroll
        for (int w = 0; w < NG; w += 2) {
            uint4 o[2] = {rounded(z + 2 * w, 0, c1), rounded(z + 2 * w, 1, c1)};
            swap_lines(o[0], o[1]);
#pragma unroll
            for (int h = 0; h < 2; ++h) store(zr, zo + (uint32_t)(NG * 64) * 8u * h + 64u * w, o[h]);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) av[s] = an[s];
        blk = next;
    }
}

template <int DT, int NG, bool JOIN> static void launch_tail_inst(const TailArgs &a, hipStream_t st)
{
    static std::once_flag once; // one per instantiation
    constexpr int lds_bytes = 8 * 2 * (JOIN ? 4 : 2) * 1024 + 8 * 2 * NG * 1024 + (256 + 32 * NG) * 4;
    auto kern = bottleneck_tail_kernel<DT, NG, JOIN>;
    allow_lds_once(once, kern, lds_bytes);
    const unsigned blocks = (a.M + 15u) / 16u, grid = std::min(256u, blocks);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kTailWaves * 64), lds_bytes, st, a);
}

int launch_bottleneck_tail(int dtype, const TailArgs &a, int G, bool join, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if ((dtype != NPAS_BF16 && dtype != NPAS_F16) || (G != 64 && G != 128) || a.M == 0 || a.M > kTailMaxPixels) {
        set_error("bottleneck_tail: unsupported shape or type");
        return NPAS_E_SHAPE;
    }
    auto pick = [&](auto dtc) {
        constexpr int DT = decltype(dtc)::value;
        if (join) G == 64 ? launch_tail_inst<DT, 2, true>(a, st) : launch_tail_inst<DT, 4, true>(a, st);
        else G == 64 ? launch_tail_inst<DT, 2, false>(a, st) : launch_tail_inst<DT, 4, false>(a, st);
    };
    if (dtype == NPAS_BF16) pick(std::integral_constant<int, NPAS_BF16>{});
    else pick(std::integral_constant<int, NPAS_F16>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("bottleneck_tail launch failed: %s", hipGetErrorString(e));
        return NPAS_E_HIP;
    }
    return NPAS_OK;
}

} // namespace npas
