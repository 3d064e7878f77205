// gfx950 kernel of libnpas for k x k layers with whole 64-channel chunks on many pixels: weights from the L2 straight into
// registers, activations through LDS.
//
// What bounds such a layer is feeding the matrix cores.  With weights and activations both in LDS, 64 x 64 outputs a wave and a barrier
// per 64-channel tap, a tap took 1.7-1.9 k cycles for 1024 of MFMAs: operand reads, their waits on both sides of every barrier, and
// an epilogue and a prologue that nothing hides.  Here
//   * a workgroup has four multiplying waves, one per SIMD, each up to 112 pixels x 64 filters: a step of 32 channels is 28 MFMAs
//     against 7 operand reads from LDS (a quarter of an LDS byte per multiply of the 64 x 64 tiling with weights in LDS) and 4 KB of
//     weight images, asked for three steps ahead in registers, from the L2;
//   * a barrier per 64-channel chunk (18 steps of a 3x3 layer), whose patch four more waves fetch while the chunk before is multiplied;
//   * every MFMA hides three other instructions, so all of a step's addresses, loads and bookkeeping are put between its MFMAs
//     (scheduling groups); behind them they cost a third of the step (815 -> 520-660 cycles for 448 of MFMAs);
//   * the four waves are 2 pixel groups x 2 filter halves, 4 x 1, or 1 x 2 and 2 x 1 with the reduction split over two waves that
//     meet in LDS once per tile: with the tile's height free this fits one round of 256 workgroups to a map (14 x 14 x 256 at
//     batch 128: one image x 128 filters each, 13 pixel blocks of 16 instead of 16).
// bf16, warm, against the streaming kernels before it: 14 x 14 x 256 at batch 128 30.3 -> 27.0 us, 28 x 28 x 128 32.8 -> 29.0, 7 x 7 x 512 34.7 -> 29.6,
// 56 x 56 x 64 35.1 -> 33.7; at stride 2 256 -> 256 onto 14 x 14 42.0 -> 33.9; 192 -> 192 at 33 x 33, batch 48 41.9 -> 33.4; against the tiled and split ones
// 256 -> 256 at 14 x 14, batch 16 17.2 -> 10.2.  A chip at work all over is slower: 256 items of 14 x 14 x 256 take 26.9 us, 64 of the same items 22.9.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "npas_internal.h"
#include "device_util.h"

namespace npas {

struct DirectItem {
    int n0, ty0, tx0, fb;
};

__device__ __forceinline__ DirectItem direct_item(const SpatialDirectArgs &a, uint32_t item)
{
    DirectItem it;
    const uint32_t tile = fastdiv(item, a.div_nfb), row = fastdiv(tile, a.div_tx), img = fastdiv(row, a.div_ty);
    it.fb = (int)(item - tile * (uint32_t)a.nfb);
    it.tx0 = (int)(tile - row * (uint32_t)a.tilesX) * a.TW;
    it.ty0 = (int)(row - img * (uint32_t)a.tilesY) * a.TH;
    it.n0 = (int)img * a.NI;
    return it;
}

constexpr uint32_t kOutside = 0xffffffffu; // byte offset of what lies outside a tensor: past the buffer descriptor's range, so loads give zeros and stores vanish
__device__ __forceinline__ uint32_t add_sat(uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); }

// Byte offset in the input of patch pixel pp of an item (channel 0; a multiple of 128), kOutside for padding; bits 4-6 hold the
// pixel's key: its 16-byte vector cv lies in LDS at cv ^ key.  Keys count as if the patch had the tile's width, so the
// operand reads of any tap meet eight keys in eight consecutive tile pixels, also across the ends of rows and images.
__device__ __forceinline__ uint32_t direct_patch_entry(const SpatialDirectArgs &a, const DirectItem &it, uint32_t pp)
{
    const uint32_t img = fastdiv(pp, a.div_phpw), r = pp - img * (uint32_t)(a.PH * a.PW);
    const uint32_t py = fastdiv(r, a.div_pw), px = r - py * (uint32_t)a.PW;
    const int n = it.n0 + (int)img, iy = it.ty0 * a.stride - a.pad + (int)py, ix = it.tx0 * a.stride - a.pad + (int)px;
    const bool in = (int)img < a.NI && n < a.N && (uint32_t)iy < (uint32_t)a.H && (uint32_t)ix < (uint32_t)a.W;
    const uint32_t key = img * (uint32_t)(a.TH * a.TW) + (py >> (a.stride - 1)) * (uint32_t)a.TW + (px >> (a.stride - 1));
    return in ? (uint32_t)((n * a.H + iy) * a.W + ix) * (uint32_t)a.C * 2u | (key & 7u) << 4 : kOutside;
}
// Byte offset in the output of tile pixel m of an item (filter 0), kOutside where there is none.
__device__ __forceinline__ uint32_t direct_out_entry(const SpatialDirectArgs &a, const DirectItem &it, uint32_t m)
{
    const uint32_t thtw = (uint32_t)(a.TH * a.TW), img = fastdiv(m, a.div_thtw), r = m - img * thtw;
    const uint32_t ty = fastdiv(r, a.div_tw), tx = r - ty * (uint32_t)a.TW;
    const int n = it.n0 + (int)img, oy = it.ty0 + (int)ty, ox = it.tx0 + (int)tx;
    return (int)img < a.NI && n < a.N && oy < a.Ho && ox < a.Wo ? (uint32_t)((n * a.Ho + oy) * a.Wo + ox) * (uint32_t)a.F * 2u : kOutside;
}

// Epilogue of a multiplying wave for its pixel blocks S0 .. S1-1: bias, residual, activation, round, store.  Result
// register i of acc[j][s] is tile pixel m0 + 16 s + i (m0 = the wave's first pixel + 4 q), filter fcol + j: a lane
// writes 4 consecutive filters of a pixel, the 16 lanes of a quarter wave one whole 128-byte run of its row.  `ot`
// points at the lane's entry m0 of the item's output offsets.  The activation kind and the residual are wave-uniform and compiled in.
// HELD (wave-uniform): pixels with a sum that is NaN are not stored; their shortcut, which lies in y, is still to be read.
template <int DT, int S0, int S1, int NB, bool HS, bool RES>
__device__ __forceinline__ void direct_store_tile(const SpatialDirectArgs &a, const uint8_t *ot, const f32x4 (&acc)[4][NB], float4 b4, uint32_t fbyte, Clamp cl, bool held = false)
{
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(a.y, 0, (int)a.ybytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.residual), 0, (int)a.ybytes, 0x00020000);
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
    asm volatile("" : "+v"(b4.x), "+v"(b4.y), "+v"(b4.z), "+v"(b4.w)); // (keeps the variants' common sums from being formed ahead of the branch: 112 registers)
#pragma unroll
    for (int s = S0; s < S1; ++s) {
        __builtin_amdgcn_sched_barrier(0); // (a block's values and addresses one after the other: interleaved they spill beside the next item's weights)
        const uint4 p4 = *reinterpret_cast<const uint4 *>(ot + s * 64);
        uint32_t o[4] = {add_sat(p4.x, fbyte), add_sat(p4.y, fbyte), add_sat(p4.z, fbyte), add_sat(p4.w, fbyte)};
        u32x2 r2[4];
        if (RES)
#pragma unroll
            for (int i = 0; i < 4; ++i) r2[i] = (u32x2)__builtin_amdgcn_raw_buffer_load_b64(rr, (int)o[i], 0, 0);
        if (RES && __builtin_expect(held, 0))
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = __builtin_isunordered(acc[0][s][i], acc[1][s][i]) || __builtin_isunordered(acc[2][s][i], acc[3][s][i]) ? kOutside : o[i];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v[4] = {acc[0][s][i] + b4.x, acc[1][s][i] + b4.y, acc[2][s][i] + b4.z, acc[3][s][i] + b4.w};
            if (RES) {
                v[0] += from_storage<DT>((uint16_t)(r2[i].x & 0xffffu));
                v[1] += from_storage<DT>((uint16_t)(r2[i].x >> 16));
                v[2] += from_storage<DT>((uint16_t)(r2[i].y & 0xffffu));
                v[3] += from_storage<DT>((uint16_t)(r2[i].y >> 16));
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[j] = HS ? v[j] * __builtin_amdgcn_fmed3f(v[j] + 3.0f, 0.0f, 6.0f) * (1.0f / 6.0f) : __builtin_amdgcn_fmed3f(v[j], cl.lo, cl.hi);
            const u32x2 out = {pack2<DT>(v[0], v[1]), pack2<DT>(v[2], v[3])};
            __builtin_amdgcn_raw_buffer_store_b64(out, yr, (int)o[i], 0, 0);
        }
    }
}
// Whether a sum of the wave is NaN: one running maximum that lets NaN pass.
template <int S0, int S1, int NB> __device__ __forceinline__ bool direct_any_nan(const f32x4 (&acc)[4][NB])
{
    float any = 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = S0; s < S1; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            any = __builtin_elementwise_maximum(__builtin_elementwise_maximum(any, acc[0][s][i]), acc[1][s][i]);
            any = __builtin_elementwise_maximum(__builtin_elementwise_maximum(any, acc[2][s][i]), acc[3][s][i]);
        }
    return __any(any != any);
}
// The lane's pixels (bit 4 s + i) one of whose four sums is NaN.
template <int S0, int S1, int NB> __device__ __forceinline__ uint32_t direct_nan_pixels(const f32x4 (&acc)[4][NB])
{
    uint32_t todo = 0;
    if (__builtin_expect(!direct_any_nan<S0, S1, NB>(acc), 1)) return todo;
#pragma unroll
    for (int s = S0; s < S1; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            todo |= __builtin_isunordered(acc[0][s][i], acc[1][s][i]) || __builtin_isunordered(acc[2][s][i], acc[3][s][i]) ? 1u << (4 * s + i) : 0u;
    return todo;
}
// A sum that is NaN (an infinite input against the zero of a pruned weight) is formed again over the kept weights, behind the
// stores, and with it the other three of its pixel.  (In one place for all variants of the epilogue, by the bits alone: within one of
// them the sums stayed in registers for the others.)
template <int DT> __device__ __forceinline__ void direct_mend_nan(const uint8_t *ot, uint32_t todo, int fcol)
{
    if (__builtin_expect(!__any(todo), 1)) return;
    auto ka = (const __attribute__((address_space(4))) SpatialDirectArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ka)); // (the arguments are read again: kept for this they would take registers from the loop)
    const auto &a = *ka;
    if (fcol >= a.F) return;
    const Clamp cl = clamp_of(a.act);
    const uint16_t *rp = reinterpret_cast<const uint16_t *>(a.residual);
    uint16_t *yp = reinterpret_cast<uint16_t *>(a.y);
#pragma unroll 1
    for (; todo; todo &= todo - 1u) {
        const uint32_t k = (uint32_t)__builtin_ctz(todo), o = *reinterpret_cast<const uint32_t *>(ot + (k >> 2) * 64u + (k & 3u) * 4u);
        if (o == kOutside) continue;
        const size_t e = (size_t)(o >> 1) + (size_t)(uint32_t)fcol;
        float sum[4];
        kept_sums<DT, SpatialDirectArgs>((o >> 1) / (uint32_t)a.F, (uint32_t)fcol, sum);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float v = sum[j] + (a.bias ? a.bias[fcol + j] : 0.f);
            if (rp) v += from_storage<DT>(rp[e + j]);
            yp[e + j] = to_storage<DT>(clampf(v, cl));
        }
    }
}
template <int DT, int S0, int S1, int NB>
__device__ __forceinline__ uint32_t direct_epilogue(const SpatialDirectArgs &a, const uint8_t *ot, const f32x4 (&acc)[4][NB], float4 b4, int fcol, Clamp cl)
{
    const uint32_t fbyte = fcol < a.F ? (uint32_t)fcol * 2u : kOutside;
    if (__builtin_expect(!a.residual, 1)) {
        if (__builtin_expect(!cl.hs, 1)) direct_store_tile<DT, S0, S1, NB, false, false>(a, ot, acc, b4, fbyte, cl);
        else direct_store_tile<DT, S0, S1, NB, true, false>(a, ot, acc, b4, fbyte, cl);
    } else {
        const bool held = a.residual == a.y && direct_any_nan<S0, S1, NB>(acc); // (the shortcut added in place)
        if (cl.hs) direct_store_tile<DT, S0, S1, NB, true, true>(a, ot, acc, b4, fbyte, cl, held);
        else direct_store_tile<DT, S0, S1, NB, false, true>(a, ot, acc, b4, fbyte, cl, held);
    }
    return direct_nan_pixels<S0, S1, NB>(acc);
}

constexpr int kDirectFetchWaves = 4, kDirectThreads = (4 + kDirectFetchWaves) * 64;
constexpr uint32_t kDirectExchange = 2u * 16384u; // LDS of the partial sums' exchange (KS == 2): 16 KB per filter half

template <int DT, int G, int H, int KS, int NB>
__global__ __launch_bounds__(kDirectThreads) void spatial_direct_kernel(SpatialDirectArgs a)
{
    static_assert(G * H * KS == 4 && (KS == 1 || (NB <= 8 && G * H == 2)), "four multiplying waves, one per SIMD");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const uint32_t lbase = (uint32_t)(uintptr_t)lds;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n16 = lane & 15, q = lane >> 4;
    const uint32_t nwg = gridDim.x, nitems = (uint32_t)a.nitems;
    const int T = a.KH * a.KW, nch = a.C >> 6, sh = a.stride - 1; // (stride 1 or 2)
    const uint32_t npx = (uint32_t)a.npb * 8u, ppb = (uint32_t)a.npb * 1024u; // pixels, bytes of one patch buffer (npb is even)
    constexpr uint32_t kPix = G * NB * 16;                        // pixels of a tile
    const uint32_t lex = 2u * ppb;                                // partial sums' exchange
    const uint32_t lbias = lex + (KS == 2 ? kDirectExchange : 0u); // two 1 KB bias buffers (item parity)
    const uint32_t lotab = lbias + 2048u;                         // output offsets of the tile's pixels (item parity)
    const uint32_t lbtab = lotab + 2u * kPix * 4u;                // byte of a tile pixel's tap (0, 0) in a patch buffer
    const uint32_t lptab = lbtab + kPix * 4u;                     // input offsets of the patch's pixels (item parity)
    uint32_t c_item = xcd_remap(blockIdx.x, nwg);
    if (c_item >= nitems) return;
    DirectItem it = direct_item(a, c_item);

    // An item's tables.  The entries of a patch block are written by the wave that will fetch it (nw waves, this one w).
    auto tables = [&](const DirectItem &ti, uint32_t par, int w, int nw) __attribute__((always_inline)) {
        for (int blk = w + (lane >> 3) * nw; blk < a.npb; blk += 8 * nw) {
            const uint32_t pp = (uint32_t)(blk * 8 + (lane & 7));
            reinterpret_cast<uint32_t *>(lds + lptab)[par * npx + pp] = direct_patch_entry(a, ti, pp);
        }
        for (uint32_t m = (uint32_t)(w * 64 + lane); m < kPix; m += (uint32_t)(nw * 64)) reinterpret_cast<uint32_t *>(lds + lotab)[par * kPix + m] = direct_out_entry(a, ti, m);
    };
    // Blocks w, w + nw, ... (8 pixels each) of a patch chunk.
    const u32x4 xr = buffer_of(a.x, (uint32_t)a.xbytes);
    auto patch = [&](int cc, uint32_t buf, uint32_t par, int w, int nw) __attribute__((always_inline)) {
        const uint32_t lv = (uint32_t)(lane & 7) * 16u; // (kOutside with its key bits flipped is still past the end: tensors of whole 128-byte pixels)
        const uint32_t *tab = reinterpret_cast<const uint32_t *>(lds + lptab) + par * npx + (uint32_t)(lane >> 3);
        for (int b0 = w; b0 < a.npb; b0 += 4 * nw) {
            uint32_t e[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) e[j] = tab[min(b0 + j * nw, a.npb - 1) * 8] ^ lv;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (b0 + j * nw < a.npb) lds_buffer16(xr, e[j], (uint32_t)cc * 128u, lbase + buf * ppb + (uint32_t)(b0 + j * nw) * 1024u);
        }
    };
    tables(it, 0, wave, kDirectThreads / 64);
    for (uint32_t m = (uint32_t)tid; m < kPix; m += kDirectThreads) {
        const uint32_t thtw = (uint32_t)(a.TH * a.TW), img = fastdiv(m, a.div_thtw), r = m - img * thtw;
        const uint32_t ty = fastdiv(r, a.div_tw), tx = r - ty * (uint32_t)a.TW;
        reinterpret_cast<uint32_t *>(lds + lbtab)[m] = (int)img < a.NI ? (img * (uint32_t)(a.PH * a.PW) + (ty * (uint32_t)a.PW + tx) * (uint32_t)a.stride) * 128u : 0u;
    }
    __syncthreads();
    patch(0, 0, 0, wave, kDirectThreads / 64); // the first chunk: all eight waves

    if (wave >= 4) {
        // ---- patch fetch, and the tables of the next item --------------------------------------------------
        const int wl = wave - 4;
        // bias of an item's 64 H filters (lanes past them fetch a copy that nobody reads)
        auto bias_block = [&](const DirectItem &pi, uint32_t buf) __attribute__((always_inline)) {
            if (!a.bias || wl != 0) return;
            const int f = pi.fb * (64 * H) + (lane & (16 * H - 1)) * 4;
            lds_dma16(a.bias + (f < a.F ? f : 0), lbase + lbias + buf * 1024u);
        };
        // The next chunk's weights into the XCD's L2 ahead of their use (its workgroups share the lines; the loaded words land in
        // 256 bytes that nobody reads): in a network the weights come from memory, and three steps of lookahead do not cover that
        // (14 x 14 x 256 inside the 50-layer stack 31.1 -> 28.5 us, 7 x 7 x 512 32.3 -> 30.3; with the weights in a cache no difference).  Not with
        // two chunks (28 x 28 x 128 in the stack and alone: no difference), nor at stride 2, where four times the patch is on its way (56 x
        // 56 x 128 46.4 -> 47.5).  Returns the loads issued.
        auto touch = [&](int cc) __attribute__((always_inline)) -> uint32_t {
            uint32_t count = 0;
            const uint32_t lines = (uint32_t)T * 128u, all = (uint32_t)((a.F + 127) >> 7) * lines; // of a 128-filter block, of all
            const uint32_t per = all / ((nwg + 7u) >> 3) + 1u, l0 = (blockIdx.x >> 3) * per, l1 = min(l0 + per, all);
            for (uint32_t k = l0 + (uint32_t)wl * 64u; k < l1; k += kDirectFetchWaves * 64u, ++count) {
                const uint32_t l = min(k + (uint32_t)lane, l1 - 1u), fb = l / lines;
                lds_dma4(reinterpret_cast<const uint8_t *>(a.wimg) + ((size_t)(fb * (uint32_t)nch + (uint32_t)cc) * lines + (l - fb * lines)) * 128u, lbase + lptab + 2u * npx * 4u);
            }
            return count;
        };
        bias_block(it, 0);
        uint32_t pbuf = 0, par = 0;
        // One item (false: it was the last).  TOUCH: the workgroup's first item of a long reduction.
        auto fetch_item = [&](auto touching) __attribute__((always_inline)) -> bool {
            constexpr bool TOUCH = decltype(touching)::value;
            uint32_t pending = 0; // loads behind the patch's: a wave's loads return in order, so these need not be awaited
            const bool more_items = c_item + nwg < nitems;
            if (more_items) it = direct_item(a, c_item + nwg);
            for (int cc = 0; cc < nch; ++cc) {
                if (TOUCH) wait_vmcnt(pending); // this chunk's patch (and the tables) have landed
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier(); // ... and the other buffer has been multiplied
                asm volatile("" ::: "memory");
                if (cc == 0 && more_items) { // (the other parity was last read in the epilogue before this item)
                    tables(it, par ^ 1u, wl, kDirectFetchWaves);
                    bias_block(it, par ^ 1u);
                }
                if (cc + 1 < nch) {
                    patch(cc + 1, pbuf ^ 1u, par, wl, kDirectFetchWaves);
                    if (TOUCH) pending = touch(cc + 1);
                } else {
                    if (more_items) patch(0, pbuf ^ 1u, par ^ 1u, wl, kDirectFetchWaves);
                    pending = 0;
                }
                pbuf ^= 1u;
            }
            if (KS == 2) { // the multiplying waves' exchange
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_s_barrier();
            }
            c_item += nwg;
            par ^= 1u;
            return more_items;
        };
        // (later items find the weights in the L2)
        bool more = nch >= 4 && !sh ? fetch_item(std::true_type{}) : fetch_item(std::false_type{});
        while (more) more = fetch_item(std::false_type{});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }

    // ---- multiply ------------------------------------------------------------------------
    const int wg = wave / (H * KS), wh = (wave / KS) % H, wk = wave % KS; // pixel group, filter half, share of the reduction
    const Clamp cl = clamp_of(a.act);
    constexpr int R = 4;                                 // steps of weights in registers, the present one included
    constexpr uint32_t kStep = KS == 2 ? 16384u : 8192u; // bytes from one of this wave's steps to the next
    const uint32_t nst = (uint32_t)(nch * T) * (KS == 2 ? 1u : 2u), wlast = (nst - 1u) * kStep;
    const uint32_t lane16 = (uint32_t)lane * 16u;
    const uint32_t qv = (uint32_t)(q + (KS == 2 ? 4 * wk : 0)) * 16u;
    uint4 Wt[R][4], B[NB];
    const uint8_t *wbase;
    uint32_t woff;
    auto weight_base = [&](int fb) __attribute__((always_inline)) {
        const uint32_t half = (uint32_t)(fb * H + wh); // 64-filter half of the layer
        wbase = reinterpret_cast<const uint8_t *>(a.wimg) + (size_t)(half >> 1) * (size_t)(nch * T) * 16384u + (half & 1u) * 4096u + (KS == 2 ? (uint32_t)wk * 8192u : 0u);
        woff = 0;
    };
    auto load_w = [&](uint4 (&w)[4]) __attribute__((always_inline)) { // the next step's four images (past the end: the last step's again)
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = *reinterpret_cast<const uint4 *>(wbase + (size_t)woff + (lane16 + (uint32_t)j * 1024u));
        woff = min(woff + kStep, wlast);
    };
    weight_base(it.fb);
#pragma unroll
    for (int r = 0; r + 1 < R; ++r) load_w(Wt[r]);
    uint32_t pb0[NB]; // byte of this lane's operand rows (tile pixels 16 (NB wg + s) + n16) at tap (0, 0) in a patch buffer
#pragma unroll
    for (int s = 0; s < NB; ++s) pb0[s] = reinterpret_cast<const uint32_t *>(lds + lbtab)[(wg * NB + s) * 16 + n16];
    uint32_t pbuf = 0, par = 0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this wave's blocks of the first chunk

    for (;;) { // one item per iteration
        f32x4 acc[4][NB];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < NB; ++s) acc[j][s] = f32x4{0.f, 0.f, 0.f, 0.f};
        const bool more_items = c_item + nwg < nitems;
        uint32_t kh = 0, kw = 0, tap = 0, key = 0, left = 0; // tap of the step; its byte offset, buffer included, and its key; taps left in the chunk
        uint32_t bbase = 0;                                  // the chunk's buffer
        const uint32_t krow = (uint32_t)(a.PW - a.KW) * 128u;
        // this lane's part of an operand address: the tap and the vector qv / 16 behind the pixel's key (tile pixel 16 k + n16)
        auto lane_part = [&](uint32_t half) __attribute__((always_inline)) -> uint32_t {
            return tap + ((((uint32_t)n16 + key) << 4 & 0x70u) ^ (qv ^ half * 64u));
        };
        auto fragment = [&](int s, uint32_t lp) __attribute__((always_inline)) -> uint4 { return *reinterpret_cast<const uint4 *>(lds + (pb0[s] + lp)); };
        // One 32-deep step.  The next step's fragment of block s - 1 is asked for between the MFMAs of block s, and the weights of
        // the step R - 1 ahead into the registers that the step before has left: every MFMA hides three other instructions, so
        // all of a step's addresses, loads and bookkeeping lie between its MFMAs.
        auto step = [&](uint4 (&w)[4], uint4 (&wn)[4], int half) __attribute__((always_inline)) {
            const bool new_tap = KS == 2 || half == 1;
            if ((KS == 2 || half == 0) && left == 0) { // a chunk begins
                __builtin_amdgcn_s_barrier(); // its patch is in LDS
                asm volatile("" ::: "memory");
                bbase = tap = pbuf * ppb;
                pbuf ^= 1u;
                left = (uint32_t)T;
                kh = kw = key = 0;
                const uint32_t lp = lane_part(0);
#pragma unroll
                for (int s = 0; s < NB; ++s) B[s] = fragment(s, lp);
            }
            // the next step's tap (behind the chunk's last step: the first tap again, its fragments are read anew after the barrier)
            if (new_tap) {
                --left;
                ++kw;
                tap += 128u + (kw == (uint32_t)a.KW ? krow : 0u);
                kh += kw == (uint32_t)a.KW ? 1u : 0u;
                kw = kw == (uint32_t)a.KW ? 0u : kw;
                tap = left == 0 ? bbase : tap;
                key = (kh >> sh) * (uint32_t)a.TW + (kw >> sh);
            }
            const uint32_t lp = lane_part(new_tap ? 0u : 1u);
            load_w(wn);
#pragma unroll
            for (int s = 0; s < NB; ++s) {
                acc[0][s] = mfma16<DT>(B[s], w[0], acc[0][s]);
                acc[1][s] = mfma16<DT>(B[s], w[1], acc[1][s]);
                acc[2][s] = mfma16<DT>(B[s], w[2], acc[2][s]);
                if (s > 0) B[s - 1] = fragment(s - 1, lp);
                acc[3][s] = mfma16<DT>(B[s], w[3], acc[3][s]);
            }
            B[NB - 1] = fragment(NB - 1, lp);
#pragma unroll
            for (int s = 0; s < NB; ++s) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0); // MFMA
                __builtin_amdgcn_sched_group_barrier(0x6, 3, 0); // VALU, SALU
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x6, 3, 0);
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                if (s > 0) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); // LDS read
                if (s > 0 && s < 3) __builtin_amdgcn_sched_group_barrier(0x20, 2, 0); // global loads
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                if (s == NB - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x6, 2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        for (uint32_t t = 0;;) {
            step(Wt[0], Wt[3], 0);
            if (KS == 2 && ++t == nst) break;
            step(Wt[1], Wt[0], 1);
            if ((t += 3 - KS) == nst) break;
            step(Wt[2], Wt[1], 0);
            if (KS == 2 && ++t == nst) break;
            step(Wt[3], Wt[2], 1);
            if ((t += 3 - KS) == nst) break;
        }
        const int fcol = it.fb * (64 * H) + wh * 64 + 4 * n16;
        if (more_items) { // the next item's first weights travel during the epilogue
            it = direct_item(a, c_item + nwg);
            weight_base(it.fb);
            load_w(Wt[0]);
            load_w(Wt[1]);
        }
        float4 b4 = float4{0.f, 0.f, 0.f, 0.f};
        if (a.bias) b4 = *reinterpret_cast<const float4 *>(lds + lbias + par * 1024u + (uint32_t)(wh * 64 + 4 * n16) * 4u);
        const uint8_t *ot = lds + lotab + (par * kPix + (uint32_t)(wg * NB * 16 + 4 * q)) * 4u;
        uint32_t nan_pixels;
        if (KS == 2) {
            // the two shares of the reduction meet: wave 0 of a pair finishes pixel blocks 0 .. K0-1, wave 1 the others
            constexpr int K0 = (NB + 1) / 2;
            f32x4 *ex = reinterpret_cast<f32x4 *>(lds + lex + (uint32_t)(wg * H + wh) * 16384u) + lane;
            if (wk == 1) {
#pragma unroll
                for (int s = 0; s < K0; ++s)
#pragma unroll
                    for (int j = 0; j < 4; ++j) ex[(s * 4 + j) * 64] = acc[j][s];
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (wk == 0) {
#pragma unroll
                for (int s = 0; s < K0; ++s)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const f32x4 o = ex[(s * 4 + j) * 64];
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[j][s][i] += o[i];
                        if (K0 + s < NB) ex[(s * 4 + j) * 64] = acc[j][K0 + s < NB ? K0 + s : 0];
                    }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (wk == 0) nan_pixels = direct_epilogue<DT, 0, K0, NB>(a, ot, acc, b4, fcol, cl);
            else {
#pragma unroll
                for (int s = K0; s < NB; ++s)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const f32x4 o = ex[((s - K0) * 4 + j) * 64];
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[j][s][i] += o[i];
                    }
                nan_pixels = direct_epilogue<DT, K0, NB, NB>(a, ot, acc, b4, fcol, cl);
            }
        } else
            nan_pixels = direct_epilogue<DT, 0, NB, NB>(a, ot, acc, b4, fcol, cl);
        direct_mend_nan<DT>(ot, nan_pixels, fcol);
        if (!more_items) break;
        load_w(Wt[2]);
        c_item += nwg;
        par ^= 1u;
    }
}

size_t spatial_direct_lds_bytes(int npb, int G, int KS, int NB)
{
    return (size_t)2 * npb * 1024 + (KS == 2 ? kDirectExchange : 0) + 2048 + (size_t)npb * 64 + 256 + (size_t)G * NB * 192;
}

template <int DT, int G, int H, int KS, int NB> static void launch_direct_inst(const SpatialDirectArgs &a, unsigned grid, size_t lds_bytes, hipStream_t st)
{
    auto kern = spatial_direct_kernel<DT, G, H, KS, NB>;
    static std::once_flag once; // one per instantiation
    allow_lds_once(once, kern, 160 * 1024);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kDirectThreads), lds_bytes, st, a);
}

template <int DT> static bool launch_direct_dt(const SpatialDirectArgs &a, unsigned grid, size_t lds_bytes, hipStream_t st)
{
#define NPAS_D(g, h, k, b) if (a.G == g && a.Hf == h && a.KS == k && a.NB == b) { launch_direct_inst<DT, g, h, k, b>(a, grid, lds_bytes, st); return true; }
#define NPAS_DN(g, h, k) NPAS_D(g, h, k, 3) NPAS_D(g, h, k, 4) NPAS_D(g, h, k, 5) NPAS_D(g, h, k, 6) NPAS_D(g, h, k, 7)
    NPAS_DN(2, 2, 1)
    NPAS_DN(1, 2, 2)
    NPAS_DN(4, 1, 1)
    NPAS_DN(2, 1, 2)
#undef NPAS_DN
#undef NPAS_D
    return false;
}

int launch_spatial_direct(int dtype, const SpatialDirectArgs &a, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const size_t lds_bytes = spatial_direct_lds_bytes(a.npb, a.G, a.KS, a.NB);
    const long items = (long)a.tilesN * a.tilesY * a.tilesX * a.nfb;
    const unsigned grid = (unsigned)std::min<long>(items, 256);
    if (lds_bytes > 160 * 1024 || a.C % 64 != 0 || a.npb % 2 != 0 || a.npb * 8 < a.NI * a.PH * a.PW || a.NI * a.TH * a.TW > 16 * a.NB * a.G ||
        (a.stride != 1 && a.stride != 2) || a.PH != (a.TH - 1) * a.stride + a.KH || a.PW != (a.TW - 1) * a.stride + a.KW || items != a.nitems ||
        items * std::max(a.nfb, std::max(a.tilesX, a.tilesY)) > 0xffffffffL /* divided by reciprocals */ ||
        (size_t)a.N * a.H * a.W * a.C * 2 != a.xbytes || (size_t)a.N * a.Ho * a.Wo * a.F * 2 != a.ybytes) {
        set_error("spatial_direct: tile plan does not fit the kernel");
        return NPAS_E_SHAPE;
    }
    bool ok;
    if (dtype == NPAS_BF16) ok = launch_direct_dt<NPAS_BF16>(a, grid, lds_bytes, st);
    else if (dtype == NPAS_F16) ok = launch_direct_dt<NPAS_F16>(a, grid, lds_bytes, st);
    else {
        set_error("spatial_direct needs a 16-bit storage type");
        return NPAS_E_DTYPE;
    }
    if (!ok) {
        set_error("spatial_direct: no such tile shape");
        return NPAS_E_SHAPE;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("spatial_direct launch failed: %s", hipGetErrorString(e));
        return NPAS_E_HIP;
    }
    return NPAS_OK;
}

} // namespace npas
