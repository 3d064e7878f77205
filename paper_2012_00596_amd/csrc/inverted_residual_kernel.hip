// gfx950 kernel of libnpas that runs the cascade 1x1 -> depthwise 3x3 -> 1x1 as one launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "npas_internal.h"
#include "device_util.h"

namespace npas {

// ------------------------------------------------------------------------------
// fused_inverted_residual: y = act3(W3 . act2(DW3x3(act1(W1 . x + b1)) + b2) + b3 [+ x]) for the cascade
// 1x1 -> 3x3 depthwise (stride 1 or 2) -> 1x1 of the search space (section 5.1.1) when the two wide
// tensors between the layers have no other reader.  They never leave the CU: HBM sees x once and y once.
// The block input is added at stride 1 only (at stride 2 the shapes differ); the biases are optional.
//
// A workgroup (4 waves) owns an output tile of TH x TW pixels.
//   1. Expansion: for the input pixels under the tile plus a one-pixel halo ((TH-1) stride + 3 rows),
//      16 pixels at a time, layer 1's MFMAs (K = C1 <= 32 in one step) produce 16 x 16 output tiles that
//      start from their bias, are clamped, rounded and written to LDS as [halo pixel][slot] in the storage
//      type.  Halo pixels outside the image are written as zero, as the padding of the depthwise layer must
//      be.  A slot is an intermediate channel some filter of layer 3 keeps; channels nobody keeps are dead
//      and are never computed (the pruning of layer 3 pays in layers 1 and 2).
//   2. Depthwise, 16 output pixels x 16 slots at a time, on the matrix cores: the row operand is diagonal,
//      row r = slot 16 s + r, and a 32-deep step holds two taps of 16 slots, so nine taps are five steps
//      (the tenth half is zero).  A lane of the row operand then has at most one nonzero weight: the weights
//      are kept as one word per lane and step, in place for its half of a 16-bit pair, and four constant lane
//      masks spread it over the operand's four words.  A lane of the column operand reads 8 consecutive
//      slots of one halo pixel, 16 bytes of LDS.
//   3. Projection: two neighbouring result tiles of step 2, clamped and rounded, are exactly the column
//      operand of a 32-deep step of layer 3 whose K order is
//          position 8 q + i <-> slot 32 k + 4 q + i,   position 8 q + 4 + i <-> slot 32 k + 16 + 4 q + i   (i < 4).
//      After all steps: residual (x again, 8 bytes per lane), clamp, round, store.
// All weights of steps 2 and 3 stay in registers (NK = slots / 32 is compiled in for that).
// Biases, layer 3's images and (at 96 slots) the depthwise weights lie in LDS, the other weights in registers; a workgroup
// walks tiles and asks for the next tile's activations before it works on this one's steps 2 and 3, and its barriers wait for
// LDS alone, so that those loads and the stores stay in flight.
// The depthwise layer on the vector ALUs, as this kernel had it before (dot2 on packed pairs with one half of the weight
// zero, tap weights read from LDS beside the activations), was bound by both: 27 16-byte LDS reads and 109 vector
// instructions per 16 pixels x 32 slots, where there are now 10 reads and about 50 (the masks shared by two pixel blocks).  It is
// now a mix: of 18 us the vector ALUs are busy 7.5, the LDS 6 and the matrix cores 3.6, on three waves per SIMD that
// work in step.  64 x 56 x 56, 24 -> 144 (83 live) -> 24, bf16, launches over three sets of tensors in turn: 28.7 -> 18.0 us with biases
// (26.9 -> 16.3 on one set, warm), 25.2 -> 17.5 without, 41 -> 20.8 with hard-swish, stride 2 19.6 -> 12.8; 32 -> 192 -> 32 (all live)
// 70.6 -> 33.1; one image 10.7 -> 4.8.

// Pitches in LDS.  A 16-byte access is served eight lanes at a time, four neighbouring lanes of one quarter wave with four of
// the next, whose 16 bytes lie one unit further: neighbouring output pixels have to be 2 or 6 units of 16 bytes apart
// (mod 8) to meet all banks.  At stride 1 that is one halo pixel (4 NK + 2 units), at stride 2 two (4 NK + 1 units each).  A halo row
// is padded so that the step from the last output pixel of a tile row to the first of the next is the same (mod 8).
__host__ __device__ constexpr uint32_t ir_pitch(int nslots, int stride) { return (uint32_t)nslots * 2u + (stride == 1 ? 32u : 16u); }
__host__ __device__ constexpr uint32_t ir_row_pitch(int nslots, int stride, int PW)
{
    const uint32_t p = ir_pitch(nslots, stride);
    return (uint32_t)PW * p + 16u * ((stride == 1 ? 6u : 7u) * (p / 16u) % 8u); // -2 p or -p units, mod 8
}
struct IrArgs {
    const void *x;
    void *y;
    const void *w1;      // [nt1][64 lanes][8] layer-1 row-operand images, rows in slot order
    const void *w3;      // [nt3][nk][64 lanes][8] layer-3 row-operand images, K in the order above
    const uint32_t *wdw; // [nt1][5][64 lanes]: the lane's one weight of a depthwise step (see build_ir)
    const int *perm;     // [nslots] intermediate channel of each slot, -1: padding slot
    const float *b1, *b2, *b3; // biases of the three layers in channel order, or null
    int N, H, W, C1, F3;
    int stride, Ho, Wo;  // of the depthwise layer; output map
    int nt3;             // ceil(F3 / 16)
    int TH, TW, tilesY, tilesX;
    int act1, act2, act3;
    int residual;        // 1: add the block input (needs F3 == C1 and stride 1)
    uint32_t ntiles;     // N * tilesY * tilesX
    int fast;            // the reciprocals are exact for every tile index
    uint32_t div_tw, div_pw, div_tx, div_ty;
};

// The activations compiled in; a branch per value, as the last kind has it, keeps the compiler from interleaving loads, MFMAs and
// epilogue arithmetic across values (hard-swish blocks with it, fp16, stride 2: 1 x 28 x 28, 32 -> 192 -> 32 13.0 us, now 8.9; the
// kernel with the depthwise layer on the vector ALUs 11.6).
// Where the first activation has no upper bound, an expanded value may be infinite in the storage type; the diagonal operand's
// zeros then make NaN in all sixteen slots of a step, while the slot itself may be finite again after ReLU or ReLU6.  In such
// kernels the second activation lets NaN pass (maximum, minimum instead of the median), so that layer 3's sums show it: a pixel with
// a NaN among them is worked out again one product at a time.  With ReLU6 first there is nothing to look for, and without a
// lower bound second (none, hard-swish) the pixel's results are not finite whatever its other slots are.
enum { IR_PLAIN,              // clamps (none, ReLU, ReLU6), first ReLU6 or second none
       IR_RELU,               // clamps, second ReLU
       IR_HS_CLAMP, IR_CLAMP_HS, IR_HS_HS, // the first two; third a clamp
       IR_MIXED };            // the rest
__host__ __device__ constexpr bool ir_looks_for_nan(int act) { return act == IR_RELU || act == IR_HS_CLAMP || act == IR_MIXED; }
static int ir_kind(int act1, int act2, int act3)
{
    const bool h1 = act1 == NPAS_ACT_HARDSWISH, h2 = act2 == NPAS_ACT_HARDSWISH;
    if (act3 == NPAS_ACT_HARDSWISH) return IR_MIXED;
    if (h1 || h2) return h1 && h2 ? IR_HS_HS : h1 ? IR_HS_CLAMP : IR_CLAMP_HS;
    if (act1 == NPAS_ACT_RELU6 || act2 == NPAS_ACT_NONE) return IR_PLAIN;
    return act2 == NPAS_ACT_RELU ? IR_RELU : IR_MIXED;
}

// bytes in front of the halo tile: biases of the three layers, layer 3's images
// (and the depthwise weights where the registers of three workgroups per CU do not hold them: at 96 slots, and at 64 in a kernel that
// looks for NaN, which spilled 16-24 of them otherwise: 64 x 56 x 56, 16 -> 64 -> 16 at stride 2 with ReLU 12.4 us, 9.3 so)
__host__ __device__ constexpr bool ir_wd_in_lds(int nslots, int act) { return nslots == 96 || (nslots == 64 && ir_looks_for_nan(act)); }
__host__ __device__ constexpr uint32_t ir_lds_front(int nslots, int act)
{
    return (uint32_t)nslots * 8u + 128u + (uint32_t)nslots / 32u * 2048u + (ir_wd_in_lds(nslots, act) ? (uint32_t)nslots / 16u * 1280u : 0u);
}

template <bool HS> __device__ __forceinline__ float ir_act(float v, Clamp c)
{
    if (HS) return v * __builtin_amdgcn_fmed3f(v + 3.0f, 0.0f, 6.0f) * (1.0f / 6.0f);
    return __builtin_amdgcn_fmed3f(v, c.lo, c.hi);
}
template <int ACT> __device__ __forceinline__ float ir_act1(float v, Clamp c)
{
    return ACT == IR_MIXED ? clampf(v, c) : ir_act<ACT == IR_HS_CLAMP || ACT == IR_HS_HS>(v, c);
}
template <int ACT> __device__ __forceinline__ float ir_act2(float v, Clamp c)
{
    if (ACT == IR_RELU) return __builtin_elementwise_maximum(v, 0.0f);
    if (ACT == IR_MIXED && c.hs) return ir_act<true>(v, c);
    if (ACT == IR_HS_CLAMP || ACT == IR_MIXED) return __builtin_elementwise_minimum(__builtin_elementwise_maximum(v, c.lo), c.hi);
    return ir_act<ACT == IR_CLAMP_HS || ACT == IR_HS_HS>(v, c);
}
template <int ACT> __device__ __forceinline__ float ir_act3(float v, Clamp c) { return clampf<ACT == IR_MIXED>(v, c); }

template <int DT, int NK, int ACT> __global__ __launch_bounds__(256, fused_ir_wgs_per_cu(32 * NK)) void fused_inverted_residual_kernel(IrArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    constexpr int NT1 = 2 * NK, NSLOTS = 32 * NK;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n16 = lane & 15, q = lane >> 4;
    const int PH = (a.TH - 1) * a.stride + 3, PW = (a.TW - 1) * a.stride + 3;
    const int nhb = (PH * PW + 15) >> 4, nob = (a.TH * a.TW + 15) >> 4; // 16-pixel blocks of the halo tile / the tile
    const uint32_t pitch = ir_pitch(NSLOTS, a.stride), rpitch = ir_row_pitch(NSLOTS, a.stride, PW);
    float *lb1 = reinterpret_cast<float *>(lds), *lb2 = lb1 + NSLOTS, *lb3 = lb2 + NSLOTS; // biases in slot / filter order
    uint4 *lw3 = reinterpret_cast<uint4 *>(lb3 + 32);                                      // [2][NK][64] layer 3's images
    constexpr bool WDL = ir_wd_in_lds(NSLOTS, ACT);
    uint32_t *lwd = reinterpret_cast<uint32_t *>(lw3 + 2 * NK * 64); // [NT1][5][64] depthwise weights
    uint8_t *y1 = lds + ir_lds_front(NSLOTS, ACT);

    // What the launch keeps for all its tiles: the weight images in registers (layer 3's in LDS), the biases in LDS.  Everything
    // is asked for here together with the first tile's activations: one memory latency instead of one per step.
    const bool biased = a.b1 || a.b2;
    const int bch = biased && tid < NSLOTS ? a.perm[tid] : -1; // (NSLOTS <= 192 threads)
    uint4 w1r[NT1], w3v[(NK + 1) / 2], xv[4];
    uint32_t wd[NT1][5], wdv[WDL ? (NT1 * 5 + 3) / 4 : 1];
    uint32_t hpos[4]; // the lane's halo pixel of round r: row << 16 | column (rows past the halo tile stay past it)
    uint32_t inside;  // bit r: it lies in the image
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t hp = (uint32_t)((wave + 4 * r) * 16 + n16), py = fastdiv(hp, a.div_pw);
        hpos[r] = py << 16 | (hp - py * (uint32_t)PW);
    }
    const uint32_t cq = (uint32_t)min(8 * q, a.C1 - 8);
    int n, ty0, tx0; // image and first output pixel of the tile at hand
    auto load_x = [&](uint32_t item) __attribute__((always_inline)) {
        const uint32_t t = xcd_remap(item, a.ntiles), t1 = a.fast ? fastdiv(t, a.div_tx) : t / (uint32_t)a.tilesX;
        tx0 = (int)(t - t1 * (uint32_t)a.tilesX) * a.TW;
        n = (int)(a.fast ? fastdiv(t1, a.div_ty) : t1 / (uint32_t)a.tilesY);
        ty0 = (int)(t1 - (uint32_t)n * (uint32_t)a.tilesY) * a.TH;
        const uint8_t *ximg = reinterpret_cast<const uint8_t *>(a.x) + (size_t)n * a.H * a.W * a.C1 * 2; // (an image is below 4 GiB)
        inside = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int iy = ty0 * a.stride - 1 + (int)(hpos[r] >> 16), ix = tx0 * a.stride - 1 + (int)(hpos[r] & 0xffffu);
            const bool in = (int)(hpos[r] >> 16) < PH && (uint32_t)iy < (uint32_t)a.H && (uint32_t)ix < (uint32_t)a.W;
            inside |= in ? 1u << r : 0u;
            // no branch: outside the image some pixel of it (the result is replaced by zero), past the last channel the last ones
            // again (replaced by zeros below: their weights are zero, but infinity times zero is not)
            xv[r] = *reinterpret_cast<const uint4 *>(ximg + ((in ? (uint32_t)(iy * a.W + ix) * (uint32_t)a.C1 : 0u) + cq) * 2u);
        }
    };
    // An LDS-only barrier: loads of the next tile and stores of the last one stay in flight across it.
    auto lds_barrier = [] __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    load_x(blockIdx.x);
    const uint4 *w1 = reinterpret_cast<const uint4 *>(a.w1), *w3 = reinterpret_cast<const uint4 *>(a.w3);
#pragma unroll
    for (int t = 0; t < NT1; ++t) w1r[t] = w1[t * 64 + lane];
    float bv1 = 0.f, bv2 = 0.f, bv3 = 0.f;
    if (bch >= 0) {
        if (a.b1) bv1 = a.b1[bch];
        if (a.b2) bv2 = a.b2[bch];
    }
    if (a.b3 && tid < a.F3) bv3 = a.b3[tid];
#pragma unroll
    for (int i = 0; i < (NK + 1) / 2; ++i) w3v[i] = tid + 256 * i < 64 * NK * a.nt3 ? w3[tid + 256 * i] : uint4{0u, 0u, 0u, 0u};
    if (WDL) {
#pragma unroll
        for (int i = 0; i < (NT1 * 5 + 3) / 4; ++i) wdv[i] = a.wdw[min(tid + 256 * i, NT1 * 320 - 1)];
    } else {
#pragma unroll
        for (int t = 0; t < NT1; ++t)
#pragma unroll
            for (int m = 0; m < 5; ++m) wd[t][m] = a.wdw[(t * 5 + m) * 64 + lane];
    }
    if (tid < NSLOTS) {
        lb1[tid] = bv1;
        lb2[tid] = bv2;
    }
    if (tid < 32) lb3[tid] = bv3;
#pragma unroll
    for (int i = 0; i < (NK + 1) / 2; ++i)
        if (tid + 256 * i < 128 * NK) lw3[tid + 256 * i] = w3v[i];
    if (WDL) {
#pragma unroll
        for (int i = 0; i < (NT1 * 5 + 3) / 4; ++i)
            if (tid + 256 * i < NT1 * 320) lwd[tid + 256 * i] = wdv[i];
    }
    lds_barrier();

    const Clamp cl1 = clamp_of(a.act1), cl2 = clamp_of(a.act2), cl3 = clamp_of(a.act3);
    uint32_t mask[4], toff[5];
#pragma unroll
    for (int j = 0; j < 4; ++j) mask[j] = (n16 & 7) >> 1 == j ? 0xffffffffu : 0u;
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        const int tap = min(2 * m + (q >> 1), 8); // (the second half of the last step has no weights)
        toff[m] = (uint32_t)(tap / 3) * rpitch + (uint32_t)(tap % 3) * pitch + (uint32_t)(q & 1) * 16u;
    }
    for (uint32_t item = blockIdx.x;;) {
    // what derives from these is formed again for every tile: kept from tile to tile it costs more registers than there are
    asm("" : "+v"(hpos[0]), "+v"(hpos[1]), "+v"(hpos[2]), "+v"(hpos[3]));
    // ---- 1. expansion into LDS ------------------------------------------------------------
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (wave + 4 * r >= nhb) break; // wave-uniform
        const bool in_tile = (int)(hpos[r] >> 16) < PH; // otherwise written to the spare pixel behind the halo tile
        uint8_t *dst = y1 + (in_tile ? (hpos[r] >> 16) * rpitch + (hpos[r] & 0xffffu) * pitch : (uint32_t)PH * rpitch) + (uint32_t)q * 16u;
        const uint32_t keep = 0u - (inside >> r & 1u); // padding of the depthwise layer is zero, whatever the bias
        const uint4 xr = 8 * q < a.C1 ? xv[r] : uint4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            uint32_t o[4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // result register i: slot 32 k + 8 q + 4 h + i (the two tiles of a step interleaved: one 16-byte write)
                const int t = 2 * k + h;
                const f32x4 d = mfma16<DT>(w1r[t], xr, *reinterpret_cast<const f32x4 *>(lb1 + 32 * k + 8 * q + 4 * h));
                o[2 * h] = pack2<DT>(ir_act1<ACT>(d[0], cl1), ir_act1<ACT>(d[1], cl1));
                o[2 * h + 1] = pack2<DT>(ir_act1<ACT>(d[2], cl1), ir_act1<ACT>(d[3], cl1));
            }
            *reinterpret_cast<uint4 *>(dst + k * 64) = uint4{o[0] & keep, o[1] & keep, o[2] & keep, o[3] & keep};
        }
    }
    const int oy0 = ty0, ox0 = tx0;
    const uint8_t *ximg = reinterpret_cast<const uint8_t *>(a.x) + (size_t)n * a.H * a.W * a.C1 * 2;
    uint8_t *yimg = reinterpret_cast<uint8_t *>(a.y) + (size_t)n * a.Ho * a.Wo * a.F3 * 2;
    item += gridDim.x;
    if (item < a.ntiles) load_x(item); // the next tile's activations travel during steps 2 and 3
    lds_barrier();

    // ---- 2. depthwise and 3. projection ---------------------------------------------------
    uint64_t nan = 0; // lanes with a NaN among the tile's sums
    // NB 16-pixel blocks at a time (ob0 and ob0 + 4), so that a step's operand words are formed once for both
    auto blocks = [&](auto nbc, int ob0) __attribute__((always_inline)) {
        constexpr int NB = decltype(nbc)::value;
        bool valid[NB];
        uint32_t pix[NB];
        const uint8_t *base[NB];
        uint2 rx[NB][2]; // the block input of a lane's pixel, asked for ahead of its use
        f32x4 acc[NB][2];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            uint32_t p = (uint32_t)((ob0 + 4 * j) * 16 + n16);
            asm("" : "+v"(p));
            const uint32_t ty = fastdiv(p, a.div_tw), tx = p - ty * (uint32_t)a.TW;
            const int oy = oy0 + (int)ty, ox = ox0 + (int)tx;
            valid[j] = (int)ty < a.TH && oy < a.Ho && ox < a.Wo;
            base[j] = y1 + (valid[j] ? (ty * rpitch + tx * pitch) * (uint32_t)a.stride : 0u);
            pix[j] = (uint32_t)(oy * a.Wo + ox);
            rx[j][0] = rx[j][1] = uint2{0u, 0u};
            if (a.residual) { // (C1 == F3; lanes without an output load some other value and store nothing)
                const uint32_t o = valid[j] ? pix[j] * (uint32_t)a.C1 : 0u;
                rx[j][0] = *reinterpret_cast<const uint2 *>(ximg + (o + (uint32_t)min(4 * q, a.F3 - 4)) * 2u);
                rx[j][1] = *reinterpret_cast<const uint2 *>(ximg + (o + (uint32_t)min(16 + 4 * q, a.F3 - 4)) * 2u);
            }
            acc[j][0] = *reinterpret_cast<const f32x4 *>(lb3 + 4 * q);
            acc[j][1] = *reinterpret_cast<const f32x4 *>(lb3 + 16 + 4 * q);
        }
        // the operand words are formed at their use: hoisted out of this loop they take four times the weights' registers
        asm("" : "+v"(mask[0]), "+v"(mask[1]), "+v"(mask[2]), "+v"(mask[3]));
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            uint32_t b[NB][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = 2 * k + h;
                const f32x4 bias = *reinterpret_cast<const f32x4 *>(lb2 + 16 * t + 4 * q);
                f32x4 d[NB];
#pragma unroll
                for (int m = 0; m < 5; ++m) {
                    const uint32_t w = WDL ? lwd[(t * 5 + m) * 64 + lane] : wd[t][m];
                    const uint4 wv = uint4{w & mask[0], w & mask[1], w & mask[2], w & mask[3]};
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        d[j] = mfma16<DT>(wv, *reinterpret_cast<const uint4 *>(base[j] + toff[m] + t * 32), m ? d[j] : bias);
                }
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    b[j][2 * h] = pack2<DT>(ir_act2<ACT>(d[j][0], cl2), ir_act2<ACT>(d[j][1], cl2));
                    b[j][2 * h + 1] = pack2<DT>(ir_act2<ACT>(d[j][2], cl2), ir_act2<ACT>(d[j][3], cl2));
                }
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const uint4 w3a = lw3[k * 64 + lane], w3b = lw3[(NK + k) * 64 + lane];
                const uint4 bv = uint4{b[j][0], b[j][1], b[j][2], b[j][3]};
                acc[j][0] = mfma16<DT>(w3a, bv, acc[j][0]);
                acc[j][1] = mfma16<DT>(w3b, bv, acc[j][1]);
            }
        }
        // (a NaN slot makes NaN of all the pixel's sums)
        if (ir_looks_for_nan(ACT)) nan |= __builtin_amdgcn_ballot_w64(__builtin_isunordered(acc[0][0][0], acc[NB - 1][0][0]));
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (!valid[j]) continue;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int f = 16 * u + 4 * q;
                if (f >= a.F3) continue;
                float v[4] = {acc[j][u][0], acc[j][u][1], acc[j][u][2], acc[j][u][3]};
                if (a.residual) {
                    const uint2 r = rx[j][u];
                    v[0] += from_storage<DT>((uint16_t)(r.x & 0xffffu));
                    v[1] += from_storage<DT>((uint16_t)(r.x >> 16));
                    v[2] += from_storage<DT>((uint16_t)(r.y & 0xffffu));
                    v[3] += from_storage<DT>((uint16_t)(r.y >> 16));
                }
                uint2 o;
                o.x = pack2<DT>(ir_act3<ACT>(v[0], cl3), ir_act3<ACT>(v[1], cl3));
                o.y = pack2<DT>(ir_act3<ACT>(v[2], cl3), ir_act3<ACT>(v[3], cl3));
                store_stream8(yimg + (pix[j] * (uint32_t)a.F3 + (uint32_t)f) * 2u, o);
            }
        }
    };
    for (int ob = wave; ob < nob; ob += 8) { // wave-uniform
        if (ob + 4 < nob) blocks(std::integral_constant<int, 2>{}, ob);
        else blocks(std::integral_constant<int, 1>{}, ob);
    }
    if (ir_looks_for_nan(ACT) && nan) { // the wave's blocks again, four filters at a time, without products of zeros that are no weights
        // (the arguments are read again here: kept for this they would take scalar registers from the loops above)
        auto ka = (const __attribute__((address_space(4))) IrArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(ka));
#pragma unroll 1
        for (int i = 2 * wave; i < 2 * nob; i += i & 1 ? 7 : 1) {
            const int u = i & 1, f = 16 * u + 4 * q;
            const uint32_t p = (uint32_t)(i >> 1) * 16u + n16, ty = fastdiv(p, ka->div_tw), tx = p - ty * (uint32_t)ka->TW;
            const int oy = oy0 + (int)ty, ox = ox0 + (int)tx;
            if (f >= ka->F3 || (int)ty >= ka->TH || oy >= ka->Ho || ox >= ka->Wo) continue;
            const uint8_t *px = y1 + (ty * rpitch + tx * pitch) * (uint32_t)ka->stride;
            f32x4 v = *reinterpret_cast<const f32x4 *>(lb3 + f);
#pragma unroll 1
            for (int s = 0; s < NSLOTS; ++s) {
                const int r = s & 15;
                float d = lb2[s];
#pragma unroll 1
                for (int tap = 0; tap < 9; ++tap) {
                    const uint32_t w = ka->wdw[((s >> 4) * 5 + (tap >> 1)) * 64 + (2 * (tap & 1) + (r >> 3)) * 16 + r] >> (16 * (r & 1));
                    const uint16_t e = *reinterpret_cast<const uint16_t *>(px + (uint32_t)(tap / 3) * rpitch + (uint32_t)(tap % 3) * pitch + 2 * s);
                    d = fmaf(from_storage<DT>((uint16_t)(w & 0xffffu)), from_storage<DT>(e), d);
                }
                d = from_storage<DT>(to_storage<DT>(clampf(d, clamp_of(ka->act2))));
                // slot s is element 4 (s / 16 % 2) + s % 4 of lanes 16 (s / 4 % 4) + filter in layer 3's image of step s / 32
                const uint16_t *w3 = reinterpret_cast<const uint16_t *>(lw3 + (u * NK + (s >> 5)) * 64 + (r >> 2) * 16 + 4 * q) + 4 * (s >> 4 & 1) + (s & 3);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (w3[8 * k] & 0x7fffu) v[k] = fmaf(from_storage<DT>(w3[8 * k]), d, v[k]);
            }
            const uint32_t pix = (uint32_t)(oy * ka->Wo + ox);
            uint16_t *yp = reinterpret_cast<uint16_t *>(yimg) + pix * (uint32_t)ka->F3 + (uint32_t)f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (ka->residual) v[k] += from_storage<DT>(reinterpret_cast<const uint16_t *>(ximg)[pix * (uint32_t)ka->C1 + f + k]);
                yp[k] = to_storage<DT>(ir_act3<ACT>(v[k], clamp_of(ka->act3)));
            }
        }
    }
    if (item >= a.ntiles) break; // (the same for the whole workgroup)
    lds_barrier(); // the halo tile is free again
    }
}

size_t fused_ir_lds_bytes(int TH, int TW, int nslots, int stride, int act1, int act2, int act3)
{
    return ir_lds_front(nslots, ir_kind(act1, act2, act3)) + (size_t)((TH - 1) * stride + 3) * ir_row_pitch(nslots, stride, (TW - 1) * stride + 3) + ir_pitch(nslots, stride);
}

template <int DT, int NK> static void ir_launch(const IrArgs &a, unsigned grid, size_t lds_bytes, hipStream_t st)
{
    static std::once_flag once[6];
    auto go = [&](auto kern, std::once_flag &flag) {
        allow_lds_once(flag, kern, 160 * 1024);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds_bytes, st, a);
    };
    switch (ir_kind(a.act1, a.act2, a.act3)) {
    case IR_PLAIN: go(fused_inverted_residual_kernel<DT, NK, IR_PLAIN>, once[0]); break;
    case IR_RELU: go(fused_inverted_residual_kernel<DT, NK, IR_RELU>, once[1]); break;
    case IR_HS_CLAMP: go(fused_inverted_residual_kernel<DT, NK, IR_HS_CLAMP>, once[2]); break;
    case IR_CLAMP_HS: go(fused_inverted_residual_kernel<DT, NK, IR_CLAMP_HS>, once[3]); break;
    case IR_HS_HS: go(fused_inverted_residual_kernel<DT, NK, IR_HS_HS>, once[4]); break;
    default: go(fused_inverted_residual_kernel<DT, NK, IR_MIXED>, once[5]); break;
    }
}

int launch_fused_inverted_residual(int dtype, const IrLaunch &l, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const int N = l.N, H = l.H, W = l.W, C1 = l.C1, F3 = l.F3, nslots = l.nslots, TH = l.TH, TW = l.TW, stride = l.stride;
    IrArgs a;
    a.x = l.x; a.y = l.y; a.w1 = l.w1; a.w3 = l.w3; a.wdw = l.wdw; a.perm = l.perm;
    a.b1 = l.b1; a.b2 = l.b2; a.b3 = l.b3;
    a.N = N; a.H = H; a.W = W; a.C1 = C1; a.F3 = F3;
    a.stride = stride; a.Ho = (H - 1) / stride + 1; a.Wo = (W - 1) / stride + 1; // 3 x 3, padding 1
    a.nt3 = (F3 + 15) / 16;
    a.TH = TH; a.TW = TW; a.tilesY = (a.Ho + TH - 1) / TH; a.tilesX = (a.Wo + TW - 1) / TW;
    a.act1 = l.act1; a.act2 = l.act2; a.act3 = l.act3; a.residual = l.residual;
    const int PH = (TH - 1) * stride + 3, PW = (TW - 1) * stride + 3;
    a.div_tw = TW <= 1 ? 0u : (uint32_t)(((1ull << 32) + TW - 1) / TW);
    a.div_pw = (uint32_t)(((1ull << 32) + PW - 1) / PW);
    const size_t lds_bytes = fused_ir_lds_bytes(TH, TW, nslots, stride, l.act1, l.act2, l.act3);
    if (nslots <= 0 || nslots % 32 || nslots > 192 || TH < 1 || TW < 1 || PH * PW > 256 || a.nt3 < 1 || a.nt3 > 2 || C1 > 32 || C1 % 8 || F3 % 4 ||
        lds_bytes > 160 * 1024 || (stride != 1 && stride != 2) || (l.residual && (F3 != C1 || stride != 1)) || !l.perm) {
        set_error("fused inverted residual: unsupported shape (slots %d, C1 %d, F3 %d, stride %d, LDS %zu)", nslots, C1, F3, stride, lds_bytes);
        return NPAS_E_SHAPE;
    }
    if (dtype != NPAS_BF16 && dtype != NPAS_F16) {
        set_error("fused inverted residual needs a 16-bit storage type");
        return NPAS_E_DTYPE;
    }
    auto magic = [](int d) { return d <= 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d); };
    a.div_tx = magic(a.tilesX);
    a.div_ty = magic(a.tilesY);
    // a workgroup per CU for every copy of the kernel that fits there (LDS, and the registers its launch bounds allow)
    const int fit = std::min<int>((int)(160 * 1024 / lds_bytes), fused_ir_wgs_per_cu(nslots));
    a.ntiles = (uint32_t)((long)N * a.tilesY * a.tilesX);
    a.fast = (uint64_t)a.ntiles * (uint64_t)std::max(a.tilesX, a.tilesY) < (1ull << 32);
    const unsigned grid = std::min<uint32_t>(a.ntiles, 256u * fit);
    auto go = [&](auto dtc) {
        constexpr int DT = decltype(dtc)::value;
        switch (nslots / 32) {
        case 1: ir_launch<DT, 1>(a, grid, lds_bytes, st); break;
        case 2: ir_launch<DT, 2>(a, grid, lds_bytes, st); break;
        case 3: ir_launch<DT, 3>(a, grid, lds_bytes, st); break;
        case 4: ir_launch<DT, 4>(a, grid, lds_bytes, st); break;
        case 5: ir_launch<DT, 5>(a, grid, lds_bytes, st); break;
        default: ir_launch<DT, 6>(a, grid, lds_bytes, st); break;
        }
    };
    if (dtype == NPAS_BF16) go(std::integral_constant<int, NPAS_BF16>{});
    else go(std::integral_constant<int, NPAS_F16>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("fused_inverted_residual launch failed: %s", hipGetErrorString(e));
        return NPAS_E_HIP;
    }
    return NPAS_OK;
}

} // namespace npas
