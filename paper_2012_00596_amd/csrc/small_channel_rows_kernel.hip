// gfx950 kernel of libnpas for the stem of an image network: k x k layers (k = 3, 5, 7) at stride 2 on 1 to 3 input channels and at
// most 64 filters, with the 3 x 3 / stride 2 / pad 1 max pool that may follow.
//
// By its bytes such a layer is bound by HBM; the whole-reduction kernel (conv_smallc_mfma) spent its time on vector instructions instead
// (about 1700 a wave and 256 conv pixels, against 80 MFMAs): operands gathered 2 bytes at a time, staging addresses by division, every conv pixel's
// place, activation and rounding, then the pool's reads, conversions and maxima.  Here
//   * the reduction is laid out kernel row by kernel row, 32 slots each (weights past the row's KW C values are zero): a lane's 8
//     values of a step are 16 contiguous bytes of an input row in LDS, and one such fragment serves both conv rows of a pair (row r of the one,
//     row r - 2 of the other): 9 fragments for 56 MFMAs at k = 7;
//   * a wave owns 16 conv columns and walks down the image with its weights in registers and a ring of 32 input rows in LDS of its own, filled
//     by direct loads (a 256-byte row each, padding by the buffer descriptor's range) five steps ahead: no barrier, no staging arithmetic;
//   * the pool is three maxima per conv value in registers: rows as they come, columns within a lane's four plus one from the next quarter
//     wave; activation and rounding, which are monotone (hard-swish is not and comes first), are left to the pooled value.
//   * operand words are read four kernel rows ahead, and the step's loads, the columns' maxima of the step before and its stores lie between MFMAs (in front
//     of them and behind them: 47 us instead of 41, of which four rows ahead were worth 2.7).
// 56 MFMAs of 16 cycles stand against about 110 vector instructions a step, on two waves a SIMD (235 registers).  7 x 7 x 3 -> 64 with the pool at
// 224 x 224, batch 128, inside the 50-layer stack 103 -> 45 us (41 where clocks are up; matrix floor 22, HBM 18); the stack 1888 -> 1827 us, at batch 1 247 -> 244.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "npas_internal.h"
#include "device_util.h"

namespace npas {

constexpr int kRowsRing = 32;  // input rows of a wave's ring, 256 bytes each
constexpr int kRowsAhead = 5;  // steps (of 4 input rows) whose rows are asked for ahead: k + 2 rows in use, 4 per step in flight, k + 2 + 20 <= 32
constexpr uint32_t kRowsOutside = 0xffffffffu; // past any buffer descriptor's range: loads give zeros, stores vanish

typedef __attribute__((ext_vector_type(2))) uint32_t rows_u32x2;

// Direct buffer -> LDS load of 64 lanes x 4 bytes to lds_addr.
__device__ __forceinline__ void lds_buffer4(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds_addr)
{
    asm volatile(NPAS_M0_FROM_ARG0 "buffer_load_dword %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory");
}

// The maximum of three, a NaN counting as nothing (fmaxf quiets every operand first, an instruction each: MFMA results need that as little as activated ones).
// The compiler does not keep an asm statement's distance from the MFMAs whose results it reads: results_ready() stands between.
__device__ __forceinline__ float max3(float a, float b, float c)
{
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ void results_ready(f32x4 (&A)[4], f32x4 (&B)[4])
{
    asm volatile("s_nop 15\n\ts_nop 7" : "+v"(A[0]), "+v"(A[1]), "+v"(A[2]), "+v"(A[3]), "+v"(B[0]), "+v"(B[1]), "+v"(B[2]), "+v"(B[3]));
}

template <int DT, int KH, bool POOL, bool HSW>
__device__ __forceinline__ void conv_smallc_rows_kernel_body(const SmallCRowsArgs &a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int lane = threadIdx.x & 63, n16 = lane & 15, q = lane >> 4;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t item = xcd_remap(blockIdx.x, gridDim.x) * 4u + wave;
    if (item >= a.nitems) return; // (no barrier below)
    const uint32_t n = fastdiv(item, a.div_img), r0 = item - n * (uint32_t)(a.nblk * a.nband);
    const uint32_t bandi = fastdiv(r0, a.div_blk), blk = r0 - bandi * (uint32_t)a.nblk;
    const int t0 = (int)bandi * a.band, t1 = min(t0 + a.band, a.nsteps); // steps: a pair of conv rows each, 2 t and 2 t + 1
    const int ox0 = POOL ? 14 * (int)blk - 1 : 16 * (int)blk;            // the wave's first conv column
    const Clamp cl = clamp_of(a.act);

    // ---- input rows: row i of the wave is image row iy0 + i and lies at ring slot i % 32 ----
    const uint32_t ring = wave * (uint32_t)(kRowsRing * 256);
    const uint32_t rowbytes = (uint32_t)(a.W * a.C) * 2u;
    const u32x4 xr = buffer_of(reinterpret_cast<const uint8_t *>(a.x) + (uint64_t)n * (uint64_t)a.H * rowbytes, (uint32_t)a.H * rowbytes);
    const int iy0 = (2 * t0 - 1) * 2 - a.pad, nrows = KH + 4 * (t1 - t0);
    const int v0 = (((ox0 * 2 - a.pad) * a.C) & ~1) + 2 * lane; // the lane's first value of a row (an even one: both or neither in the row)
    const uint32_t xv = v0 >= 0 && v0 < a.W * a.C && lane < 60 ? (uint32_t)v0 * 2u : kRowsOutside; // (a row's last 16 bytes are zeros: see lrow)
    auto ask = [&](int i) __attribute__((always_inline)) {
        const bool in = (uint32_t)(iy0 + i) < (uint32_t)a.H && i < nrows;
        lds_buffer4(xr, in ? xv : kRowsOutside, in ? (uint32_t)(iy0 + i) * rowbytes : 0u, ring + (uint32_t)(i & (kRowsRing - 1)) * 256u);
    };
    for (int i = 0; i < KH + 4 * kRowsAhead; ++i) ask(i);

    uint4 w[KH][4];
    const uint4 *wimg = reinterpret_cast<const uint4 *>(a.wimg) + lane;
#pragma unroll
    for (int r = 0; r < KH; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) w[r][j] = wimg[(r * 4 + j) * 64];
    const int fcol = 4 * n16;
    f32x4 bias[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float b = a.bias && fcol < a.F ? a.bias[fcol + j] : 0.0f;
        bias[j] = f32x4{b, b, b, b};
    }
    // slots of the lane that belong to the kernel row: the others hold neighbouring pixels, which must not meet a zero weight (they may be infinite)
    const int ph = (a.pad * a.C) & 1; // a pixel's first value is an odd one of its row: the row starts one slot later
    uint32_t mask[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 8 * q + 2 * i - ph;
        mask[i] = ((uint32_t)k < (uint32_t)a.kwc ? 0xffffu : 0u) | ((uint32_t)(k + 1) < (uint32_t)a.kwc ? 0xffff0000u : 0u);
    }
    // (lanes without any such slot read zeros: pixels and their slots end 228 bytes into a row)
    const uint8_t *lrow = lds + ring + (8 * q < a.kwc + ph ? (uint32_t)(n16 * 2 * a.C) * 2u + (uint32_t)q * 16u : 240u);
    auto words = [&](int i) __attribute__((always_inline)) {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(lrow + (uint32_t)(i & (kRowsRing - 1)) * 256u); // (4-byte aligned)
        return uint4{p[0], p[1], p[2], p[3]};
    };
    auto own = [&](uint4 v) __attribute__((always_inline)) {
        return uint4{v.x & mask[0], KH == 7 ? v.y : v.y & mask[1], v.z & mask[2], v.w & mask[3]}; // (7, 8, 14, 21 or 22 slots leave no pair 1 incomplete)
    };
    auto fragment = [&](int i) __attribute__((always_inline)) { return own(words(i)); };

    // ---- output ----
    const int oH = POOL ? a.PHo : a.Ho, oW = POOL ? a.PWo : a.Wo;
    const uint32_t orow = (uint32_t)(oW * a.F) * 2u, obytes = (uint32_t)oH * orow;
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc((uint8_t *)a.y + (uint64_t)n * obytes, 0, (int)obytes, 0x00020000);
    uint32_t ov[4]; // POOL: the lane's two pooled pixels; otherwise its four conv pixels
    bool colok[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int cx = ox0 + 4 * q + i, px = 7 * (int)blk + 2 * q + i;
        colok[i] = (uint32_t)cx < (uint32_t)a.Wo;
        const bool ok = fcol < a.F && (POOL ? i < 2 && 2 * q + i < 7 && px < a.PWo : colok[i]);
        ov[i] = ok ? (uint32_t)((POOL ? px : cx) * a.F + fcol) * 2u : kRowsOutside;
    }
    const bool edge = ox0 < 0 || ox0 + 16 > a.Wo;
    auto activate = [&](f32x4 v) __attribute__((always_inline)) {
        return f32x4{clampf<HSW>(v[0], cl), clampf<HSW>(v[1], cl), clampf<HSW>(v[2], cl), clampf<HSW>(v[3], cl)};
    };

    const f32x4 none = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    f32x4 prev[4] = {none, none, none, none}; // POOL: conv row 2 t - 1
    if (POOL && t0 > 0) {
        asm volatile("s_waitcnt vmcnt(20)" ::: "memory"); // rows 0 .. KH-1 have landed
#pragma unroll
        for (int r = 0; r < KH; ++r) {
            const uint4 f = fragment(r);
#pragma unroll
            for (int j = 0; j < 4; ++j) prev[j] = mfma16<DT>(f, w[r][j], r == 0 ? bias[j] : prev[j]);
        }
        if (HSW)
#pragma unroll
            for (int j = 0; j < 4; ++j) prev[j] = activate(prev[j]);
    }
    // POOL: the vertical maxima of the step before, whose columns are taken among this step's MFMAs, and where they go
    f32x4 v[4] = {none, none, none, none};
    uint32_t pv0 = kRowsOutside, pv1 = kRowsOutside;
    float right[4], p0[4], p1[4];
    auto columns_right = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) right[j] = __int_as_float(__builtin_amdgcn_ds_bpermute((lane + 16) * 4, __float_as_int(v[j][0]))); // column 4 (q + 1)
    };
    auto columns_finish = [&](float (&p)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) p[j] = HSW ? fmaxf(p[j], -INFINITY) /* a window of nothing but NaN */ : clampf<false>(p[j], cl);
    };
    auto columns0 = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) p0[j] = max3(v[j][0], v[j][1], v[j][2]);
        columns_finish(p0);
    };
    auto columns1 = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) p1[j] = max3(v[j][2], v[j][3], right[j]);
        columns_finish(p1);
    };
    auto columns_store = [&](int t) __attribute__((always_inline)) {
        const rows_u32x2 o0 = {pack2<DT>(p0[0], p0[1]), pack2<DT>(p0[2], p0[3])}, o1 = {pack2<DT>(p1[0], p1[1]), pack2<DT>(p1[2], p1[3])};
        __builtin_amdgcn_raw_buffer_store_b64(o0, yr, (int)pv0, (int)((uint32_t)t * orow), 0);
        __builtin_amdgcn_raw_buffer_store_b64(o1, yr, (int)pv1, (int)((uint32_t)t * orow), 0);
    };
    for (int t = t0, i0 = 2; t < t1; ++t, i0 += 4) { // i0: the input row of conv row 2 t's first kernel row
        asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); // all but the rows of kRowsAhead - 1 steps to come (4 each) have landed
        f32x4 A[4], B[4];
        uint4 raw[KH + 2];
#pragma unroll
        for (int r = 0; r < 4; ++r) raw[r] = words(i0 + r);
#pragma unroll
        for (int r = 0; r < KH + 2; ++r) {
            __builtin_amdgcn_sched_barrier(0);
            if (r + 4 < KH + 2) raw[r + 4 < KH + 2 ? r + 4 : 0] = words(i0 + r + 4);
            const uint4 f = own(raw[r]);
            // The step's other work lies between its MFMAs.  The slots filled here were last read in the step before at the latest, whose
            // maxima or stores needed what was read.
            if (r >= 1 && r <= 4) ask(i0 - 2 + KH + 4 * kRowsAhead + r - 1);
            if (POOL && r == 1) columns_right();
            if (POOL && r == 2) columns0();
            if (POOL && r == 3) columns1();
            if (POOL && r == 4) columns_store(t - 1);
            if (r < KH)
#pragma unroll
                for (int j = 0; j < 4; ++j) A[j] = mfma16<DT>(f, w[r < KH ? r : 0][j], r == 0 ? bias[j] : A[j]);
            if (r >= 2)
#pragma unroll
                for (int j = 0; j < 4; ++j) B[j] = mfma16<DT>(f, w[r >= 2 ? r - 2 : 0][j], r == 2 ? bias[j] : B[j]);
        }
        const bool rowB = 2 * t + 1 < a.Ho;
        if (POOL) {
            if (HSW)
#pragma unroll
                for (int j = 0; j < 4; ++j) { A[j] = activate(A[j]); B[j] = activate(B[j]); }
            if (!rowB)
#pragma unroll
                for (int j = 0; j < 4; ++j) B[j] = none;
            results_ready(A, B);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[j][i] = max3(A[j][i], B[j][i], prev[j][i]);
                prev[j] = B[j];
            }
            if (edge)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[j][i] = colok[i] ? v[j][i] : -INFINITY;
            pv0 = ov[0];
            pv1 = ov[1];
        } else {
            const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((uint8_t *)const_cast<void *>(a.residual) + (uint64_t)n * obytes, 0, (int)obytes, 0x00020000);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && !rowB) break;
                const int so = (int)((uint32_t)(2 * t + h) * orow);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    f32x4 v = {(h ? B : A)[0][i], (h ? B : A)[1][i], (h ? B : A)[2][i], (h ? B : A)[3][i]};
                    if (a.residual) {
                        const rows_u32x2 r2 = (rows_u32x2)__builtin_amdgcn_raw_buffer_load_b64(rr, (int)ov[i], so, 0);
                        v += f32x4{from_storage<DT>((uint16_t)(r2.x & 0xffffu)), from_storage<DT>((uint16_t)(r2.x >> 16)),
                                   from_storage<DT>((uint16_t)(r2.y & 0xffffu)), from_storage<DT>((uint16_t)(r2.y >> 16))};
                    }
                    v = activate(v);
                    const rows_u32x2 o = {pack2<DT>(v[0], v[1]), pack2<DT>(v[2], v[3])};
                    __builtin_amdgcn_raw_buffer_store_b64(o, yr, (int)ov[i], so, 0);
                }
            }
        }
    }
    if (POOL) {
        columns_right();
        columns0();
        columns1();
        columns_store(t1 - 1);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // nothing lands in LDS that is no longer this workgroup's
}

template <int DT, int KH, bool POOL>
__global__ __launch_bounds__(256, 2) void conv_smallc_rows_kernel(SmallCRowsArgs a)
{
    if (a.act == NPAS_ACT_HARDSWISH) conv_smallc_rows_kernel_body<DT, KH, POOL, true>(a);
    else conv_smallc_rows_kernel_body<DT, KH, POOL, false>(a);
}

template <int DT, int KH> static void launch_rows_inst(const SmallCRowsArgs &a, hipStream_t st)
{
    const unsigned grid = (a.nitems + 3) / 4;
    if (a.pool) hipLaunchKernelGGL((conv_smallc_rows_kernel<DT, KH, true>), dim3(grid), dim3(256), 4 * kRowsRing * 256, st, a);
    else hipLaunchKernelGGL((conv_smallc_rows_kernel<DT, KH, false>), dim3(grid), dim3(256), 4 * kRowsRing * 256, st, a);
}

template <int DT> static int launch_rows_dt(const SmallCRowsArgs &a, hipStream_t st)
{
    switch (a.KH) {
    case 3: launch_rows_inst<DT, 3>(a, st); return NPAS_OK;
    case 5: launch_rows_inst<DT, 5>(a, st); return NPAS_OK;
    case 7: launch_rows_inst<DT, 7>(a, st); return NPAS_OK;
    }
    set_error("conv_smallc_rows: kernel height %d", a.KH);
    return NPAS_E_SHAPE;
}

int launch_conv_smallc_rows(int dtype, const SmallCRowsArgs &a, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const bool wide_ok = a.C >= 1 && a.C <= 3 && (a.W * a.C) % 2 == 0 && a.kwc <= 31; // 15 pixels x 2 C values and 32 slots within a 128-value row
    if (!wide_ok || a.F < 4 || a.F > 64 || a.F % 4 || (a.pool && a.residual) || a.band < 1) {
        set_error("conv_smallc_rows: plan does not fit the kernel");
        return NPAS_E_SHAPE;
    }
    int rc = NPAS_E_DTYPE;
    if (dtype == NPAS_BF16) rc = launch_rows_dt<NPAS_BF16>(a, st);
    else if (dtype == NPAS_F16) rc = launch_rows_dt<NPAS_F16>(a, st);
    else set_error("conv_smallc_rows needs a 16-bit storage type");
    if (rc) return rc;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("conv_smallc_rows launch failed: %s", hipGetErrorString(e));
        return NPAS_E_HIP;
    }
    return NPAS_OK;
}

} // namespace npas
