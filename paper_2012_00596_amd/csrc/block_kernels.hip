// gfx950 kernels of libnpas: the fused 1x1 pair and the depthwise 3x3 layer on its own (the fused block of the two is in
// inverted_residual_kernel.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "npas_internal.h"
#include "device_util.h"

namespace npas {

// ------------------------------------------------------------------------------
// Fused pointwise pair: y = act2(W2 * act1(W1 * x + b1) + b2) for two 1x1 layers
// whose intermediate tensor has no other reader (the expand -> project pair of an
// inverted-residual bottleneck).  HBM-bound: x is read once and y written once,
// the F1-channel intermediate never leaves registers.
//
// One wave owns 16 pixels at a time.  Layer 1: the B operand is the pixel's C1
// (<= 32) channels straight from global memory, one MFMA per 16 intermediate
// channels.  The 16x16 result tile of MFMA t holds, in lane (pixel n, quarter q),
// channels 16t + 4q .. 4q+3 of that pixel; two such tiles, activated and rounded
// to the storage type, are exactly the B operand of a 32-deep MFMA of layer 2
// whose K slots are ordered  slot 8q+i <-> channel 16(2j) + 4q + i      (i < 4)
//                            slot 8q+4+i <-> channel 16(2j+1) + 4q + i
// and layer 2's weights are stored pre-permuted to that order.  All weights live
// in registers for the life of the wave.
//
// Pruning shows up twice.  An intermediate channel that no filter of layer 2 keeps
// is dead and layer 1 never computes it; the live channels are renumbered ("slots")
// so that the ones each 16-filter tile of layer 2 needs are contiguous and dead
// channels cost nothing (use[u] records which 32-slot chunks tile u really needs).
struct FppArgs {
    const void *x;
    void *y;
    const void *wblob;   // [NT1 + NT2*NCH][64 lanes][8] 16-bit weight images
    int M, C1, F2;       // pixels, input channels, output channels
    int act1, act2;
    uint32_t use[2];     // per layer-2 tile: which 32-slot chunks it needs
};

constexpr int kFppBlocksPerWave = 8; // 16-pixel blocks a wave owns; all their loads are issued up front

// Straight-line body for a wave that owns exactly CNT blocks starting at block b0.
// No branch between the loads and their uses, so the compiler can wait for block k's
// activations alone (s_waitcnt vmcnt(n)) while later blocks are still in flight.
template <int DT, int NT1, int NT2, int CNT, bool HSW>
__device__ __forceinline__ void fpp_body(const FppArgs &a, int b0, int n16, int q, int lane)
{
    constexpr int NCH = NT1 / 2;
    const uint16_t *x16 = reinterpret_cast<const uint16_t *>(a.x);
    uint16_t *y16 = reinterpret_cast<uint16_t *>(a.y);
    const bool ld_on = 8 * q < a.C1;
    const Clamp c1 = clamp_of(a.act1), c2 = clamp_of(a.act2);
    const uint4 *wb = reinterpret_cast<const uint4 *>(a.wblob) + lane;
    uint4 A1[NT1], A2[NT2][NCH];
#pragma unroll
    for (int t = 0; t < NT1; ++t) A1[t] = wb[t * 64];
#pragma unroll
    for (int u = 0; u < NT2; ++u)
#pragma unroll
        for (int j = 0; j < NCH; ++j) A2[u][j] = wb[(NT1 + u * NCH + j) * 64];
    // Rows of a partial last output tile repeat its valid rows (the weight image is built
    // that way), so every lane holds real outputs and stores them, some twice, unpredicated.
    int fst[NT2];
#pragma unroll
    for (int u = 0; u < NT2; ++u) {
        const int nvq = min(4, (a.F2 - 16 * u) >> 2); // valid groups of 4 rows in tile u
        const int q1 = q - nvq, q2 = q1 - nvq;         // q mod nvq without a division
        fst[u] = 16 * u + 4 * (q < nvq ? q : (q1 < nvq ? q1 : (nvq == 1 ? 0 : q2)));
    }
    // Pixels past M are clamped to pixel M-1 for the load AND the store: such a lane
    // recomputes pixel M-1 and writes the same bytes again, which needs no branch.
    uint4 xin[CNT];
    const int cq = ld_on ? 8 * q : 0;
    const uint32_t lmask = ld_on ? 0xffffffffu : 0u;
#pragma unroll
    for (int k = 0; k < CNT; ++k) {
        const int pix = min((b0 + k) * 16 + n16, a.M - 1);
        xin[k] = load_stream16(x16 + (size_t)pix * a.C1 + cq);
    }
    __builtin_amdgcn_sched_barrier(0); // keep every load above the first use (memory-level parallelism)
    // A layer-2 tile that keeps nothing in a chunk has an all-zero image there; it is multiplied
    // anyway rather than branched around (the MFMA pipe has slack, and a branch here would
    // make every load wait).
#pragma unroll
    for (int k = 0; k < CNT; ++k) {
        uint4 xb = xin[k];
        xb.x &= lmask; xb.y &= lmask; xb.z &= lmask; xb.w &= lmask; // K slots past C1 are zero
        f32x4 d1[NT1];
#pragma unroll
        for (int t = 0; t < NT1; ++t) d1[t] = mfma16<DT>(A1[t], xb, f32x4{0.f, 0.f, 0.f, 0.f});
        f32x4 d2[NT2];
#pragma unroll
        for (int u = 0; u < NT2; ++u) d2[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            uint4 b;
            b.x = pack2<DT>(clampf<HSW>(d1[2 * j][0], c1), clampf<HSW>(d1[2 * j][1], c1));
            b.y = pack2<DT>(clampf<HSW>(d1[2 * j][2], c1), clampf<HSW>(d1[2 * j][3], c1));
            b.z = pack2<DT>(clampf<HSW>(d1[2 * j + 1][0], c1), clampf<HSW>(d1[2 * j + 1][1], c1));
            b.w = pack2<DT>(clampf<HSW>(d1[2 * j + 1][2], c1), clampf<HSW>(d1[2 * j + 1][3], c1));
#pragma unroll
            for (int u = 0; u < NT2; ++u) d2[u] = mfma16<DT>(A2[u][j], b, d2[u]);
        }
        const int pix = min((b0 + k) * 16 + n16, a.M - 1);
#pragma unroll
        for (int u = 0; u < NT2; ++u) {
            uint2 o;
            o.x = pack2<DT>(clampf<HSW>(d2[u][0], c2), clampf<HSW>(d2[u][1], c2));
            o.y = pack2<DT>(clampf<HSW>(d2[u][2], c2), clampf<HSW>(d2[u][3], c2));
            store_stream8(y16 + (size_t)pix * a.F2 + fst[u], o); // written once, read by nobody in this launch
        }
    }
}

template <int DT, int NT1, int NT2>
__global__ __launch_bounds__(256, 2) void fused_pointwise_pair_kernel(FppArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n16 = lane & 15, q = lane >> 4;
    const int nblk = (a.M + 15) >> 4;
    const int nw = gridDim.x * 4, gw = blockIdx.x * 4 + wave;
    // contiguous run of blocks per wave, remainder spread over the first waves
    const int base = nblk / nw, extra = nblk % nw;
    const int b0 = gw * base + min(gw, extra), cnt = base + (gw < extra ? 1 : 0);
    // (the activation kinds compiled in: see clampf)
    auto run = [&](auto hsw) __attribute__((always_inline)) {
        constexpr bool H = decltype(hsw)::value;
        switch (cnt) { // wave-uniform
        case 1: fpp_body<DT, NT1, NT2, 1, H>(a, b0, n16, q, lane); break;
        case 2: fpp_body<DT, NT1, NT2, 2, H>(a, b0, n16, q, lane); break;
        case 3: fpp_body<DT, NT1, NT2, 3, H>(a, b0, n16, q, lane); break;
        case 4: fpp_body<DT, NT1, NT2, 4, H>(a, b0, n16, q, lane); break;
        case 5: fpp_body<DT, NT1, NT2, 5, H>(a, b0, n16, q, lane); break;
        case 6: fpp_body<DT, NT1, NT2, 6, H>(a, b0, n16, q, lane); break;
        case 7: fpp_body<DT, NT1, NT2, 7, H>(a, b0, n16, q, lane); break;
        case 8: fpp_body<DT, NT1, NT2, 8, H>(a, b0, n16, q, lane); break;
        default: break;
        }
    };
    if (a.act1 == NPAS_ACT_HARDSWISH || a.act2 == NPAS_ACT_HARDSWISH) run(std::true_type{});
    else run(std::false_type{});
}

template <int DT, int NT1, int NT2> static void fpp_launch(const FppArgs &a, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL((fused_pointwise_pair_kernel<DT, NT1, NT2>), dim3(grid), dim3(256), 0, st, a);
}

// nt1 = live intermediate tiles rounded up to an even count, nt2 = output tiles
bool fpp_supported(int nt1, int nt2) { return nt1 >= 2 && nt1 <= 12 && nt1 % 2 == 0 && (nt2 == 1 || nt2 == 2); }

int launch_fused_pointwise_pair(int dtype, const void *x, void *y, const void *wblob, int M, int C1, int nt1, int F2,
                                int act1, int act2, uint32_t use0, uint32_t use1, void *stream)
{
    FppArgs a{x, y, wblob, M, C1, F2, act1, act2, {use0, use1}};
    hipStream_t st = (hipStream_t)stream;
    const int nt2 = (F2 + 15) / 16;
    const int nblk = (M + 15) / 16;
    // two workgroups per CU when the batch allows it, more when a wave would otherwise own
    // more than kFppBlocksPerWave blocks
    const int min_grid = (nblk + 4 * kFppBlocksPerWave - 1) / (4 * kFppBlocksPerWave);
    unsigned grid = (unsigned)std::max(min_grid, std::min((nblk + 3) / 4, 512));
#define NPAS_FPP_CASE(N1, N2)                                                              \
    if (nt1 == N1 && nt2 == N2) {                                                          \
        if (dtype == NPAS_BF16) fpp_launch<NPAS_BF16, N1, N2>(a, grid, st);                \
        else fpp_launch<NPAS_F16, N1, N2>(a, grid, st);                                    \
    } else
    NPAS_FPP_CASE(2, 1) NPAS_FPP_CASE(2, 2) NPAS_FPP_CASE(4, 1) NPAS_FPP_CASE(4, 2) NPAS_FPP_CASE(6, 1)
    NPAS_FPP_CASE(6, 2) NPAS_FPP_CASE(8, 1) NPAS_FPP_CASE(8, 2) NPAS_FPP_CASE(10, 1) NPAS_FPP_CASE(10, 2)
    NPAS_FPP_CASE(12, 1) NPAS_FPP_CASE(12, 2)
    {
        set_error("fused pointwise pair: unsupported tile counts %d, %d", nt1, nt2);
        return NPAS_E_SHAPE;
    }
#undef NPAS_FPP_CASE
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("fused_pointwise_pair launch failed: %s", hipGetErrorString(e));
        return NPAS_E_HIP;
    }
    return NPAS_OK;
}

// ------------------------------------------------------------------------------
// Depthwise 3x3, padding 1: one thread per (output pixel, vector of V channels); V * element
// size = 16 bytes when the channel count allows it, so every load and store is one 16-byte
// access, coalesced along the channels.  HBM-bound: the nine taps of a pixel come from L1 / L2.
// fp32 storage accumulates in fp64, like the fp32 convolution kernel (products of two fp32
// values are exact in fp64, so the stored result is the correctly rounded one).
template <int DT, int V>
__global__ __launch_bounds__(256) void depthwise3x3_kernel(const void *x, void *y, const void *w, const float *bias,
                                                           const void *residual, int N, int H, int W, int C, int Ho,
                                                           int Wo, int stride, int act)
{
    const int CV = C / V;
    const size_t total = (size_t)N * Ho * Wo * CV;
    const Clamp cl = clamp_of(act);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const int cv = (int)(i % CV);
        size_t r = i / CV;
        const int ox = (int)(r % Wo);
        r /= Wo;
        const int oy = (int)(r % Ho), n = (int)(r / Ho);
        using Acc = typename std::conditional<DT == NPAS_F32, double, float>::type;
        Acc acc[V];
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] = bias ? (Acc)bias[cv * V + k] : (Acc)0;
#pragma unroll
        for (int kh = 0; kh < 3; ++kh) {
            const int iy = oy * stride + kh - 1;
            if (iy < 0 || iy >= H) continue;
#pragma unroll
            for (int kw = 0; kw < 3; ++kw) {
                const int ix = ox * stride + kw - 1;
                if (ix < 0 || ix >= W) continue;
                const size_t xo = ((size_t)(n * H + iy) * W + ix) * C + (size_t)cv * V;
                const size_t wo = (size_t)(kh * 3 + kw) * C + (size_t)cv * V;
                if (V == 8) { // 16-bit storage, 8 channels
                    const uint4 xv = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(x) + xo);
                    const uint4 wv = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(w) + wo);
                    const uint32_t xs[4] = {xv.x, xv.y, xv.z, xv.w}, ws[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        acc[2 * k] += from_storage<DT>((uint16_t)(xs[k] & 0xffffu)) * from_storage<DT>((uint16_t)(ws[k] & 0xffffu));
                        acc[2 * k + 1] += from_storage<DT>((uint16_t)(xs[k] >> 16)) * from_storage<DT>((uint16_t)(ws[k] >> 16));
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < V; ++k) acc[k] += (Acc)ld_act<DT>(x, xo + k) * (Acc)ld_act<DT>(w, wo + k);
                }
            }
        }
        const size_t yo = ((size_t)(n * Ho + oy) * Wo + ox) * C + (size_t)cv * V;
        if (residual) {
#pragma unroll
            for (int k = 0; k < V; ++k) acc[k] += (Acc)ld_act<DT>(residual, yo + k);
        }
        if (V == 8) {
            uint4 out;
            out.x = pack2<DT>(clampf((float)acc[0], cl), clampf((float)acc[1], cl));
            out.y = pack2<DT>(clampf((float)acc[2], cl), clampf((float)acc[3], cl));
            out.z = pack2<DT>(clampf((float)acc[4], cl), clampf((float)acc[5], cl));
            out.w = pack2<DT>(clampf((float)acc[6], cl), clampf((float)acc[7], cl));
            *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(y) + yo) = out;
        } else {
#pragma unroll
            for (int k = 0; k < V; ++k) st_act<DT>(y, yo + k, clampf((float)acc[k], cl));
        }
    }
}

// 16-bit storage, C a multiple of 8, stride 1 or 2: one thread owns 8 channels of R consecutive output rows of CX
// output columns.  What bounded the layer was a chain of memory latencies (an input row asked for, multiplied, the next
// one asked for), so every input vector a thread needs is asked for before the first multiply; the zero padding comes
// from the buffer descriptor's range check (an offset past the end reads zeros), which leaves no branch between the
// loads.  The multiplies go input column by input column: a tap's weights and an input vector are unpacked to fp32 once each
// and feed up to three output rows (an input vector those of two columns); fp32 multiply-adds issue in half the time of a dot2 with one half zeroed.
// Consecutive lanes are consecutive 16-byte channel vectors of a pixel, then consecutive pixels of a row; an XCD gets runs of
// 16 workgroups (a few row blocks) so that most rows two row blocks share come from its own L2, while the chip as a whole
// works on one stretch of the tensors: with inputs beyond the Infinity Cache 64 x 56 x 56 x 144 36.4 us against 38.1 with one run per
// XCD and 36.3 with none, 60 x 60 x 60 x 480 119.5 / 125.3 / 122.1, inside it 32 x 57 x 57 x 144 17.8 / 17.8 / 19.2.
// 64 x 56 x 56 x 144, bf16, launches over three sets of tensors in turn: stride 1 31 -> 28 us (a copy of the same bytes: 23), stride 2
// 57 -> 13 us (the thread of four rows had spilled); 32 x 57 x 57 x 144 with a bias 23 -> 17.2 us (22.6 -> 16.8 on one set, warm),
// with two columns a thread 16.0: vector instructions are half of it, two waves per SIMD whose loads and multiplies overlap only in part the rest;
// 1 x 46 x 28 x 272 at stride 2 16.5 -> 2.9 us.
struct DwArgs {
    const void *x;
    void *y;
    const void *w;        // [9][C] storage type, tap-major
    const float *bias;
    const void *residual;
    const void *zeros;                  // >= 16 bytes of zeros on the device
    int N, H, W, C, Ho, Wo, act;
    uint32_t xbytes;                    // size of x (read where it is below 2 GiB: see launch_depthwise3x3)
    uint32_t CV, nxb, nyb, total;       // channel vectors, column and row blocks per image, threads
    uint32_t div_cv, div_nxb, div_nyb;  // fastdiv magics
};

template <int DT> __device__ __forceinline__ void unpack8(uint4 v, float *f)
{
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f[2 * k] = from_storage<DT>((uint16_t)(u[k] & 0xffffu));
        f[2 * k + 1] = DT == NPAS_BF16 ? __uint_as_float(u[k] & 0xffff0000u) : from_storage<DT>((uint16_t)(u[k] >> 16));
    }
}

// BIG: the input does not fit a buffer descriptor's range check, or the reciprocals do not divide the thread index: 64-bit
// addresses, a block of zeros for the padding, plain divisions.  Such launches took the one-output kernel: 65 x 256 x 256 x 256
// 3380 -> 1216 us (3.6 TB/s), stride 2 924 -> 527; 32 x 512 x 512 x 64 at stride 2 (1 GiB, 2^32 as index times divisor) 404 -> 250.
template <int DT, int STRIDE, int R, int CX, bool HSW, bool BIG>
__global__ __launch_bounds__(256, R == 4 ? 2 : 3) void depthwise3x3_rows_kernel(DwArgs a)
{
    // runs of 16 workgroups per XCD (see above); the last, partial window of eight runs stays as it is
    const uint32_t win = blockIdx.x >> 7, in = blockIdx.x & 127u;
    const uint32_t blk = (win + 1u) << 7 <= gridDim.x ? (win << 7) + (in & 7u) * 16u + (in >> 3) : blockIdx.x;
    const uint32_t idx = blk * 256u + threadIdx.x;
    if (idx >= a.total) return;
    const uint32_t t = BIG ? idx / a.CV : fastdiv(idx, a.div_cv);
    const uint32_t cv = idx - t * a.CV;
    const uint32_t t2 = BIG ? t / a.nxb : fastdiv(t, a.div_nxb);
    const int ox = (int)(t - t2 * a.nxb) * CX;
    const uint32_t n = BIG ? t2 / a.nyb : fastdiv(t2, a.div_nyb);
    const int oy0 = (int)(t2 - n * a.nyb) * R;
    constexpr int NR = (R - 1) * STRIDE + 3, NC = (CX - 1) * STRIDE + 3; // input rows and columns this thread reads
    const int ix0 = ox * STRIDE - 1, iy0 = oy0 * STRIDE - 1;

    typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)a.xbytes, 0x00020000);
    const uint32_t pixb = (uint32_t)a.C * 2u, rowb = (uint32_t)a.W * pixb;
    // byte offset of input pixel (iy0, ix0); may lie before the image, in which case it is not used
    const uint32_t org = (n * (uint32_t)a.H + (uint32_t)iy0) * rowb + (uint32_t)ix0 * pixb + cv * 16u;
    uint32_t rowo[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) rowo[r] = (uint32_t)(iy0 + r) < (uint32_t)a.H ? org + (uint32_t)r * rowb : 0x80000000u;
    uint4 xv[NC][NR], wv[3][3];
#pragma unroll
    for (int kw = 0; kw < NC; ++kw) {
        const bool ok = (uint32_t)(ix0 + kw) < (uint32_t)a.W;
#pragma unroll
        for (int kh = 0; kh < 3 && kw < 3; ++kh)
            wv[kw][kh] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(a.w) + (size_t)(kh * 3 + kw) * a.C + cv * 8u);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (BIG) {
                const uint8_t *px = reinterpret_cast<const uint8_t *>(a.x) + (((size_t)n * a.H + (size_t)(iy0 + r)) * a.W + (size_t)(ix0 + kw)) * pixb + cv * 16u;
                xv[kw][r] = *reinterpret_cast<const uint4 *>(ok && (uint32_t)(iy0 + r) < (uint32_t)a.H ? px : reinterpret_cast<const uint8_t *>(a.zeros));
                continue;
            }
            const uint32_t off = ok && rowo[r] != 0x80000000u ? rowo[r] + (uint32_t)kw * pixb : 0x80000000u;
            xv[kw][r] = __builtin_bit_cast(uint4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(xr, (int)off, 0, 0));
        }
    }
    f32x4 b0 = f32x4{0.f, 0.f, 0.f, 0.f}, b1 = b0;
    if (a.bias) { // two 16-byte loads (any 4-byte alignment): as eight 4-byte ones, 32 bytes apart from lane to lane, they cost as much as the taps
        typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4u;
        b0 = *reinterpret_cast<const f32x4u *>(a.bias + cv * 8u);
        b1 = *reinterpret_cast<const f32x4u *>(a.bias + cv * 8u + 4u);
    }
    __builtin_amdgcn_sched_barrier(0); // every load above the first use
    float acc[CX][R][8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int o = 0; o < CX; ++o) acc[o][j][k] = k < 4 ? b0[k] : b1[k - 4];
#pragma unroll
    for (int ic = 0; ic < NC; ++ic) {
        float wf[CX][3][8]; // of the tap column that input column ic is for output column o
#pragma unroll
        for (int o = 0; o < CX; ++o) {
            const int kw = ic - o * STRIDE; // compile-time after unrolling, as kh
            if (kw < 0 || kw > 2) continue;
#pragma unroll
            for (int kh = 0; kh < 3; ++kh) unpack8<DT>(wv[kw][kh], wf[o][kh]);
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            float xf[8];
            unpack8<DT>(xv[ic][r], xf);
#pragma unroll
            for (int o = 0; o < CX; ++o) {
                if (ic - o * STRIDE < 0 || ic - o * STRIDE > 2) continue;
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const int kh = r - j * STRIDE;
                    if (kh < 0 || kh > 2) continue;
#pragma unroll
                    for (int k = 0; k < 8; ++k) acc[o][j][k] = fmaf(xf[k], wf[o][kh][k], acc[o][j][k]);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0); // one column's unpacked weights live at a time
    }
    const Clamp cl = clamp_of(a.act);
#pragma unroll
    for (int jo = 0; jo < R * CX; ++jo) {
        const int j = jo / CX, o = jo % CX, oy = oy0 + j;
        if (oy >= a.Ho || (CX > 1 && ox + o >= a.Wo)) continue;
        const size_t yo = (((size_t)n * a.Ho + (size_t)oy) * a.Wo + (size_t)(ox + o)) * a.C + (size_t)cv * 8;
        if (a.residual) {
            float rf[8];
            unpack8<DT>(*reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(a.residual) + yo), rf);
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[o][j][k] += rf[k];
        }
        uint4 out;
        out.x = pack2<DT>(clampf<HSW>(acc[o][j][0], cl), clampf<HSW>(acc[o][j][1], cl));
        out.y = pack2<DT>(clampf<HSW>(acc[o][j][2], cl), clampf<HSW>(acc[o][j][3], cl));
        out.z = pack2<DT>(clampf<HSW>(acc[o][j][4], cl), clampf<HSW>(acc[o][j][5], cl));
        out.w = pack2<DT>(clampf<HSW>(acc[o][j][6], cl), clampf<HSW>(acc[o][j][7], cl));
        store_stream16(reinterpret_cast<uint16_t *>(a.y) + yo, out);
    }
}

static uint32_t magic32(uint32_t d) { return d <= 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d); }

int launch_depthwise3x3(int dt, const void *x, void *y, const void *w, const float *bias, const void *residual, int N, int H,
                        int W, int C, int stride, int act, const void *zeros, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
    const bool vec = dt != NPAS_F32 && C % 8 == 0;
    const size_t xbytes = (size_t)N * H * W * C * 2;
    if (vec && (stride == 1 || stride == 2)) {
        const uint32_t CV = (uint32_t)C / 8;
        // Output rows per thread.  Four share input vectors (4.5 loads an output instead of 9) and are the faster form of a
        // launch that fills the chip anyway: 64 x 56 x 56 x 144 at stride 1 28.2 us (4.1 TB/s) against 36.1 with one row.
        // With one row a thread is a shorter chain, which wins while all waves of the launch (three per SIMD) are resident at
        // once: 3 x 28 x 28 x 144 3.1 us against 4.1, 16 x 28 x 28 x 240 (twice that many) 6.3 against 5.5.  At stride 2 the rows
        // share one input row in five: one row is never slower by more than a tenth and mostly faster (12.9 us against 15.3 with two).
        const int R = stride == 1 && (double)N * Ho * Wo * CV > 256.0 * 12 * 64 ? 4 : 1;
        const uint32_t nyb = (uint32_t)((Ho + R - 1) / R);
        // Two columns a thread share two of their four input columns (3 loads an output, a tenth fewer vector instructions) and halve the number of
        // threads, which wants launches of several rounds (2 x 256 workgroups are resident): from 2.75 rounds of one-column threads on, 32 x 57 x 57 x 144
        // 17.4 -> 16.1 us, 64 x 56 x 56 x 144 28.8 -> 27.0, 64 x 60 x 60 x 240 65.0 -> 58.3; with 2.3 rounds 64 x 28 x 28 x 192 11.9 against 12.2, with
        // 0.7 16 x 28 x 28 x 240 5.6 against 6.5 (some launches between one and two rounds would gain, 8 x 60 x 60 x 240 10.0 -> 9.2, others not).
        // The last pair of an odd row computes a column for nothing: up to a ninth more columns.  64 images of 64 channels, 400 000 / 700 000 one-column
        // threads, us with one column / with two: 9 columns 14.7 / 13.9 and 22.0 / 20.9, 7 14.7 / 13.8 and 21.7 / 22.7, 5 14.6 / 13.9 and 21.7 / 22.7,
        // 3 14.6 / 16.4 and 21.9 / 24.5, one 14.4 / 15.4 and 21.5 / 22.8; 2 columns 14.4 / 13.8 and 21.6 / 20.6.
        const int CX = R == 4 && (double)N * nyb * Wo * CV >= 2.75 * 512 * 256 && (Wo % 2 == 0 || Wo >= 9) ? 2 : 1;
        const uint32_t nxb = (uint32_t)((Wo + CX - 1) / CX);
        const double threads = (double)N * nyb * nxb * CV;
        // Offset 2 GiB is past the end for the descriptor's range check; the index decode divides by CV, nxb and nyb with 32-bit
        // reciprocals, exact while index * divisor < 2^32.
        const bool big = xbytes >= 0x80000000u || threads * std::max({CV, nxb, nyb}) >= 4294967296.0;
        DwArgs a{x, y, w, bias, residual, zeros, N, H, W, C, Ho, Wo, act, (uint32_t)xbytes, CV, nxb, nyb, (uint32_t)threads,
                 magic32(CV), magic32(nxb), magic32(nyb)};
        const unsigned grid = (a.total + 255u) / 256u;
        auto go = [&](auto dtc, auto sc, auto rc, auto cc) {
            constexpr int DT = decltype(dtc)::value, S = decltype(sc)::value, RR = decltype(rc)::value, CC = decltype(cc)::value;
            auto run = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, a); };
            const bool hsw = act == NPAS_ACT_HARDSWISH;
            if (big) run(hsw ? depthwise3x3_rows_kernel<DT, S, RR, CC, true, true> : depthwise3x3_rows_kernel<DT, S, RR, CC, false, true>);
            else run(hsw ? depthwise3x3_rows_kernel<DT, S, RR, CC, true, false> : depthwise3x3_rows_kernel<DT, S, RR, CC, false, false>);
        };
        auto rows = [&](auto dtc) {
            using std::integral_constant;
            integral_constant<int, 1> one;
            if (stride == 2) go(dtc, integral_constant<int, 2>{}, one, one);
            else if (R == 4 && CX == 2) go(dtc, one, integral_constant<int, 4>{}, integral_constant<int, 2>{});
            else if (R == 4) go(dtc, one, integral_constant<int, 4>{}, one);
            else go(dtc, one, one, one);
        };
        if (dt == NPAS_BF16) rows(std::integral_constant<int, NPAS_BF16>{});
        else rows(std::integral_constant<int, NPAS_F16>{});
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            set_error("depthwise3x3_rows launch failed: %s", hipGetErrorString(e));
            return NPAS_E_HIP;
        }
        return NPAS_OK;
    }
    const size_t total = (size_t)N * Ho * Wo * (vec ? C / 8 : C);
    const unsigned grid = (unsigned)std::min<size_t>((total + 255) / 256, 256 * 32);
#define NPAS_DW(DT, V) hipLaunchKernelGGL((depthwise3x3_kernel<DT, V>), dim3(grid), dim3(256), 0, st, x, y, w, bias, residual, N, H, W, C, Ho, Wo, stride, act)
    if (dt == NPAS_BF16) {
        if (vec) NPAS_DW(NPAS_BF16, 8);
        else NPAS_DW(NPAS_BF16, 1);
    } else if (dt == NPAS_F16) {
        if (vec) NPAS_DW(NPAS_F16, 8);
        else NPAS_DW(NPAS_F16, 1);
    } else NPAS_DW(NPAS_F32, 1);
#undef NPAS_DW
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("depthwise3x3 launch failed: %s", hipGetErrorString(e));
        return NPAS_E_HIP;
    }
    return NPAS_OK;
}

} // namespace npas
