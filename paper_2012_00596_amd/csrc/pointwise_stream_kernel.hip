// gfx950 kernel of libnpas for 16-bit 1x1 layers whose channel count is not a multiple of 64 (the expansions and projections
// of mobile networks): the flat form of the slab route.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "npas_internal.h"
#include "device_util.h"

namespace npas {

// ------------------------------------------------------------------------------
// pointwise_stream: y = act(W . x + b [+ residual]), one wave = 16 pixels at a time, all filters of its group.
// HBM-bound: 2 (C + F [+ F]) bytes per pixel.  A wave is a stream of its own, with no barrier after the weights are in place:
//   - the activations of its next 16 pixels are on their way (the column operand straight from global memory, 16 bytes
//     = 8 channels of a pixel per lane and 32-deep step, NS steps) while it works on the present ones;
//   - the weight images (row operand, every position present, pruned ones zero) and the bias lie in LDS, shared by the
//     workgroup, two 16-filter tiles multiplied side by side;
//   - a lane's result is 4 filters of one pixel; the tiles are put together in the wave's own LDS rows and written as
//     16-byte vectors, whole lines of y: one contiguous run (RUN: one filter group) or a segment of each pixel.
// The tiled slab kernel, which served these layers before, walks 64-channel chunks through LDS with one prefetch stage and a
// barrier each, and writes 8 bytes per lane in 16 different rows.
// bf16, 64 x 56 x 56: 24 -> 144 28.2 -> 13.7 us, 144 -> 24 21.3 -> 12.5 (a copy of the same bytes: 13.6); fp16,
// 64 x 57 x 57, 144 -> 40 with hard-swish 27.9 -> 16.7 (15.5); 2 x 28 x 27, 240 -> 20 7.0 -> 4.2.  Wide layers read the activations once
// per filter group; warm, 64 x 28 x 28: 240 -> 240 25.0 -> 15.9, 160 -> 960 63.1 -> 38.6, 24 -> 960 40.7 -> 25.6, 40 -> 1280
// 49.6 -> 35.3, 312 -> 1280 with hard-swish 112 -> 104.  Over 4600 layers (8 <= C <= 312, 12 <= F <= 1920, 49 .. 200704 pixels, 1x .. 20x
// pruned, also those below a quarter of the density, whose former kernel gathers single channels) none is slower than in the kernel it
// had before by more than 3 %, but for 8 x 28 x 28, 312 -> 1280 with hard-swish (19.0 -> 20.6).
// Layers with whole 64-channel chunks stay with the ring kernel, which multiplies 64 or 128 filters per activation read:
// 128 x 56 x 56, 64 -> 64 20.7 us here against 17.6 there, 64 -> 256 78 against 40, 256 -> 64 50 against 49.
template <int DT, int NS, bool HSW, bool RUN>
__global__ __launch_bounds__(256, NS <= 5 ? 4 : 3) void pointwise_stream_kernel(PwStreamArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n16 = lane & 15, q = lane >> 4;
    // groups of one pixel range are neighbours on one XCD: the range's activations come from its L2 after the first
    const uint32_t xcd = blockIdx.x & 7u, idx = blockIdx.x >> 3;
    const uint32_t groups = RUN ? 1u : (uint32_t)a.groups; // (RUN: one group)
    const int grp = (int)(idx % groups), t0 = grp * a.tpg, nt = RUN ? a.nt : min(a.tpg, a.nt - t0);
    const uint32_t wg = (idx / groups) * 8u + xcd, nwg = gridDim.x / groups;
    const uint32_t nblk = ((uint32_t)a.M + 15u) >> 4, step = nwg * 4u;
    const int f0 = 16 * t0, nf = RUN ? a.F : min(16 * nt, a.F - f0); // filters of this group
    uint4 *lw = reinterpret_cast<uint4 *>(lds);           // [nt][NS][64]
    float *lb = reinterpret_cast<float *>(lds + (size_t)a.tpg * NS * 1024);
    uint8_t *stage = lds + (size_t)a.tpg * NS * 1024 + (size_t)a.tpg * 64 + (size_t)wave * 16 * a.pitch; // 16 pixels x nf
    const uint8_t *xb = reinterpret_cast<const uint8_t *>(a.x);

    uint4 cur[NS], nxt[NS];
    auto load_x = [&](uint32_t blk, uint4 *v) __attribute__((always_inline)) {
        const uint32_t p = min(blk * 16u + n16, (uint32_t)a.M - 1u); // (past the last pixel: that pixel again, not stored)
        uint32_t ip = p;
        if (!a.flat) {
            const uint32_t n = p / (uint32_t)(a.Ho * a.Wo), r = p - n * (uint32_t)(a.Ho * a.Wo), oy = r / (uint32_t)a.Wo, ox = r - oy * (uint32_t)a.Wo;
            ip = (n * (uint32_t)a.H + oy * (uint32_t)a.stride) * (uint32_t)a.W + ox * (uint32_t)a.stride;
        }
        const uint8_t *row = xb + (size_t)ip * (uint32_t)(2 * a.C);
#pragma unroll
        for (int s = 0; s < NS; ++s) // (past the last channel the last ones again, replaced by zeros below)
            v[s] = *reinterpret_cast<const uint4 *>(row + 2u * (uint32_t)min(32 * s + 8 * q, a.C - 8));
    };
    uint32_t blk = wg * 4u + (uint32_t)wave;
    if (blk < nblk) load_x(blk, cur);
    const uint4 *wsrc = reinterpret_cast<const uint4 *>(a.wimg) + (size_t)t0 * NS * 64;
    for (int i = tid; i < nt * NS * 64; i += 256) lw[i] = wsrc[i];
    for (int i = tid; i < 16 * nt; i += 256) lb[i] = a.bias && f0 + i < a.F ? a.bias[f0 + i] : 0.f;
    __syncthreads();

    const Clamp cl = clamp_of(a.act);
    const int row_bytes = nf * 2;
    for (; blk < nblk; blk += step) {
        // past the last channel the weights are zero, but infinity times zero is not
        if (32 * (NS - 1) + 8 * q >= a.C) cur[NS - 1] = uint4{0u, 0u, 0u, 0u};
        if (blk + step < nblk) load_x(blk + step, nxt);
        const uint32_t p = min(blk * 16u + n16, (uint32_t)a.M - 1u);
        const uint8_t *rrow = reinterpret_cast<const uint8_t *>(a.residual) + ((size_t)p * (uint32_t)a.F + (uint32_t)f0) * 2u;
        uint2 rn[2] = {uint2{0u, 0u}, uint2{0u, 0u}};
        auto load_r = [&](int t) __attribute__((always_inline)) { // residual of tiles t, t + 1 (clamped to the last filters)
            rn[0] = *reinterpret_cast<const uint2 *>(rrow + 2 * min(16 * t + 4 * q, nf - 4));
            rn[1] = *reinterpret_cast<const uint2 *>(rrow + 2 * min(16 * t + 16 + 4 * q, nf - 4));
        };
        if (a.residual) load_r(0);
        for (int t = 0; t < nt; t += 2) {
            const uint2 rc[2] = {rn[0], rn[1]};
            if (a.residual && t + 2 < nt) load_r(t + 2);
            const int tb = min(t + 1, nt - 1);
            f32x4 acc[2] = {*reinterpret_cast<const f32x4 *>(lb + 16 * t + 4 * q), *reinterpret_cast<const f32x4 *>(lb + 16 * tb + 4 * q)};
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                acc[0] = mfma16<DT>(lw[(t * NS + s) * 64 + lane], cur[s], acc[0]);
                acc[1] = mfma16<DT>(lw[(tb * NS + s) * 64 + lane], cur[s], acc[1]);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int f = 16 * (t + h) + 4 * q;
                float v[4] = {acc[h][0], acc[h][1], acc[h][2], acc[h][3]};
                if (a.residual) {
                    v[0] += from_storage<DT>((uint16_t)(rc[h].x & 0xffffu));
                    v[1] += from_storage<DT>((uint16_t)(rc[h].x >> 16));
                    v[2] += from_storage<DT>((uint16_t)(rc[h].y & 0xffffu));
                    v[3] += from_storage<DT>((uint16_t)(rc[h].y >> 16));
                }
                uint2 o;
                o.x = pack2<DT>(clampf<HSW>(v[0], cl), clampf<HSW>(v[1], cl));
                o.y = pack2<DT>(clampf<HSW>(v[2], cl), clampf<HSW>(v[3], cl));
                if (f < nf) *reinterpret_cast<uint2 *>(stage + n16 * (RUN ? row_bytes : a.pitch) + 2 * f) = o;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t npx = min(16u, (uint32_t)a.M - blk * 16u); // pixels of this block
        uint8_t *yb = reinterpret_cast<uint8_t *>(a.y) + (size_t)blk * 32u * (uint32_t)a.F + 2u * (uint32_t)f0;
        if (RUN) { // one contiguous run
            const uint32_t total = npx * (uint32_t)row_bytes; // (a multiple of 8)
            for (uint32_t o = lane * 16u; o < total; o += 1024u) {
                if (o + 16u <= total) store_stream16(yb + o, *reinterpret_cast<const uint4 *>(stage + o));
                else store_stream8(yb + o, *reinterpret_cast<const uint2 *>(stage + o));
            }
        } else { // vectors of each pixel's segment
            const uint32_t segv = (uint32_t)row_bytes >> (a.store == PW_SEG16 ? 4 : 3), div_segv = a.div_segv[grp == (int)groups - 1];
            for (uint32_t v = lane; v < npx * segv; v += 64u) {
                const uint32_t px = fastdiv(v, div_segv), i = v - px * segv;
                uint8_t *d = yb + px * (uint32_t)a.F * 2u;
                const uint8_t *from = stage + px * (uint32_t)a.pitch;
                if (a.store == PW_SEG16) store_stream16(d + i * 16u, *reinterpret_cast<const uint4 *>(from + i * 16u));
                else store_stream8(d + i * 8u, *reinterpret_cast<const uint2 *>(from + i * 8u));
            }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < NS; ++s) cur[s] = nxt[s];
    }
}

// Pitch of a wave's LDS rows, an odd multiple of 16 bytes: half a wave writes 16 bytes in each of 16 rows, which meet all banks so
// (without the 16 bytes the rows of a group of 8 or 16 tiles met on the same ones: 40 -> 1280, 64 x 28 x 28 78 us instead of 57)
static int pw_stream_pitch(int tpg) { return tpg * 32 + 16; }
// LDS of a launch with tpg tiles per group
static size_t pw_stream_lds(int tpg, int ns) { return (size_t)tpg * ns * 1024 + (size_t)tpg * 64 + (size_t)64 * pw_stream_pitch(tpg); }

constexpr long kPwFill = 256; // workgroups up to which filter groups are added
static uint32_t magic32(uint32_t d) { return d <= 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d); }

bool pw_stream_supported(int C, int F) { return C % 8 == 0 && C >= 8 && C <= 320 && F % 4 == 0 && F >= 4; }

int launch_pointwise_stream(int dtype, PwStreamArgs a, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const int ns = (a.C + 31) / 32;
    if (!pw_stream_supported(a.C, a.F) || a.M <= 0) {
        set_error("pointwise stream: unsupported shape (C %d, F %d, %d pixels)", a.C, a.F, a.M);
        return NPAS_E_SHAPE;
    }
    a.nt = (a.F + 15) / 16;
    const long want = ((long)(a.M + 15) / 16 + 3) / 4; // workgroups that have pixels
    // filter groups: as few as keep the weights of one within half a CU's LDS; more while the launch has CUs to spare, since a wave
    // walks its tiles one pair after the other (16 -> 960 at 7 x 7 with three groups 7.7 us, with thirty 3.4; the tiled kernel 4.9)
    a.groups = 1;
    auto tpg = [&] { return (a.nt + a.groups - 1) / a.groups; };
    while (pw_stream_lds(tpg(), ns) > 80 * 1024 || (tpg() > 2 && want * a.groups < kPwFill)) ++a.groups;
    a.tpg = tpg();
    a.groups = (a.nt + a.tpg - 1) / a.tpg;
    const bool y16 = ((uintptr_t)a.y & 15u) == 0;
    // (one group: the run, unless its unpadded rows all meet the same quarter of the banks or less: 24 -> 128, 32 x 56 x 56 11.7 -> 7.8 us)
    a.store = y16 && a.groups == 1 && a.F % 32 != 0 ? PW_RUN : y16 && a.F % 8 == 0 ? PW_SEG16 : PW_SEG8;
    a.pitch = a.store == PW_RUN ? a.F * 2 : pw_stream_pitch(a.tpg);
    const uint32_t vec = a.store == PW_SEG16 ? 8 : 4; // filters a vector; vectors a segment of a full and of the last group
    a.div_segv[0] = magic32(16u * (uint32_t)a.tpg / vec);
    a.div_segv[1] = magic32((uint32_t)(a.F - 16 * a.tpg * (a.groups - 1)) / vec);
    const size_t lds = pw_stream_lds(a.tpg, ns);
    const int fit = std::min<int>(ns <= 5 ? 4 : 3, (int)(160 * 1024 / lds));
    // workgroups per group: a multiple of 8 (the groups of a range share an XCD), and all of them on the chip at once: a few more
    // than that run alone behind the others and double the time (520 workgroups of 40 -> 1280, five groups,
    // 64 x 28 x 28: 57 us, 480 of them 35)
    const long resident = std::max(8L, 256L * fit / a.groups / 8 * 8);
    const unsigned grid = (unsigned)(std::min((want + 7) / 8 * 8, resident) * a.groups);
    const bool hsw = a.act == NPAS_ACT_HARDSWISH;
    static std::once_flag once[2][10][4];
    auto go = [&](auto dtc, auto nsc) {
        constexpr int DT = decltype(dtc)::value, NS = decltype(nsc)::value;
        auto run = [&](auto kern, std::once_flag &flag) {
            allow_lds_once(flag, kern, 160 * 1024);
            hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, a);
        };
        std::once_flag *flags = once[DT == NPAS_F16][NS - 1];
        if (a.store == PW_RUN && hsw) run(pointwise_stream_kernel<DT, NS, true, true>, flags[0]);
        else if (a.store == PW_RUN) run(pointwise_stream_kernel<DT, NS, false, true>, flags[1]);
        else if (hsw) run(pointwise_stream_kernel<DT, NS, true, false>, flags[2]);
        else run(pointwise_stream_kernel<DT, NS, false, false>, flags[3]);
    };
    auto by_ns = [&](auto dtc) {
        switch (ns) {
#define NPAS_PW(k) case k: go(dtc, std::integral_constant<int, k>{}); break;
            NPAS_PW(1) NPAS_PW(2) NPAS_PW(3) NPAS_PW(4) NPAS_PW(5) NPAS_PW(6) NPAS_PW(7) NPAS_PW(8) NPAS_PW(9) NPAS_PW(10)
#undef NPAS_PW
        }
    };
    if (dtype == NPAS_BF16) by_ns(std::integral_constant<int, NPAS_BF16>{});
    else by_ns(std::integral_constant<int, NPAS_F16>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("pointwise_stream launch failed: %s", hipGetErrorString(e));
        return NPAS_E_HIP;
    }
    return NPAS_OK;
}

} // namespace npas
