// The pointwise -> depthwise -> pointwise block with the expanded tensor in registers (the block of ago_fused_invres.hip,
// whose workgroups pass E and D from stage to stage through LDS).
//
// A wave owns a unit of R output rows x 16 lane slots of output columns and runs, 16 expanded channels at a time,
//   E = relu6(W1^T X + b1)      matrix instruction, rows = channels, columns = input pixels: a lane holds 4 consecutive
//                               channels of one input column, the registers run over the unit's input rows
//   D = relu6(dw(E) + bd)       vector ALUs: vertical taps are other registers, horizontal taps other lanes of the same
//                               16-lane row, which the multiply-add reads through its data-parallel shift at no cost
//   Y += W2^T D                 D's layout is the matrix instruction's operand layout for a reduction over 16 channels
// so E and D never leave the registers, nothing is exchanged between waves and no barrier separates the stages.
// Lane slots: stride 1: slot j = output column ox0 + j - pad, the pad slots on either side are halo (recomputed by the
// neighbouring strip); stride 2: two E tiles per input row, even and odd input columns, slot j = output column
// ox0 + j - 1.  Maps at most 7 columns wide put two row blocks side by side, 8 slots each, with the columns beyond the
// map (E = 0) as the separator.  E outside the image is 0: relu6's upper bound is 0 there instead of 6.
//
// The workgroup's waves share the weights, which sit in LDS in their own layouts (bf16: read with the transposing LDS
// read).  nwu units x nwc channel parts: with nwc > 1 the waves of a unit divide its expanded channels and add their
// partial projections through LDS in part order.  The weights are staged once per workgroup, which walks its units; where
// they do not fit LDS, csplit channels at a time: staged again for every unit (CHUNKED; the chip is full anyway), or one
// piece per workgroup (nsplit > 1: few units), which leaves fp32 partial projections to invres_reduce_kernel.
//
// What bounds it: the vector ALUs, 9 (25) multiply-adds per expanded output element plus about 3 for the two relu6, the
// conversion and the halo; small maps by the launch and the chain of loads.
// Measured (us, LDS-staged kernel -> this one): 32 x 56 x 56, 24 -> 144 -> 24 bf16: 75.8 -> 12.9; 9 x 93 x 112, 24 -> 96 -> 24:
// 57.9 -> 10.3; 26 x 34 x 34, 128 -> 512 -> 128: 134 -> 59; 8 x 29 x 27 5 x 5 stride 2, 40 -> 240 -> 80: 15.8 -> 9.3;
// 512 x 7 x 7, 160 -> 960 -> 160: 142 -> 60.  Staging and the fragments cost about 2 us of launch, so at batch 1 the shapes
// with a specialised LDS-staged instantiation stay there (1 x 28 x 28, 32 -> 192 -> 64: 3.9 against 5.7).
#pragma once
#include "ago_dev.hpp"
#include "ago_launch.hpp"
#include <type_traits>

namespace ago {

struct InvresRegParams {
    const void* x; const void* w1; const float* b1; const void* wd; const float* bd;
    const void* w2; const float* b2; void* y;
    float* part;                            // nsplit > 1: [nsplit][N][OH][OW][Cout] fp32
    int N, H, W, Cin, Cexp, Cout, OH, OW, residual;
    unsigned x_bytes, out_elems;            // bytes of x, elements of y
    int rows;                               // output rows of a unit (R)
    int strips, segs, yblocks, rowblocks, units;   // column strips, row blocks side by side in a unit, row blocks per image, in all, units
    unsigned inv_strips, inv_yblocks;       // ceil(2^32 / d): divisions as multiplications
    int nwu, nwc_log;                       // units and log2 of the channel parts of a workgroup; nwu << nwc_log waves
    int csplit, cspan, nsplit;              // channels staged at a time, per workgroup (multiples of 16); workgroups per unit (grid.y)
    int n1, n2;                             // 1 KB loads of W1 and W2
    int q1_log, q2;                         // log2 of the 16-byte pieces per row of csplit channels (csplit < Cexp), pieces per row of W2
    unsigned inv2;                          // of q2
    int nk;                                 // reduction steps of the expansion: ceil(Cin / 32), fp32: ceil(Cin / 16)
    int p1, p2;                             // LDS bytes per row of W1, W2
    int off_w2, off_wd, off_x, off_red;     // LDS byte offsets (W1 at 0)
};

struct InvresRegPlan {
    InvresRegParams p;
    int ropt, xr, nco, threads, groups, cogroups;     // groups: workgroups along the units
    size_t smem;
    double us;
};
int invres_reg_num_cfgs();
bool invres_reg_plan_cfg(InvresRegPlan& q, int cfg, int N, int H, int W, int Cin, int Cexp, int Cout, int stride, int ksize, bool bf16);
size_t invres_reg_split_bytes(const InvresRegPlan& q);
hipError_t invres_reg_launch(const InvresRegPlan& q, int stride, int ksize, bool bf16, hipStream_t s);   // pointers in q.p

template <bool BF16, int STRIDE, int KS, int R, int XR, int NCO>
struct InvresRegCfg {
    static constexpr int PAD = (KS - 1) / 2, ROWS = (R - 1) * STRIDE + KS, TILES = STRIDE;
    static constexpr int LH = STRIDE == 1 ? PAD : 1;                       // halo slots on the left
    static constexpr int VX = 16 - LH - (STRIDE == 1 ? PAD : KS == 5 ? 1 : 0);   // output columns of a strip
    static constexpr int KG = BF16 ? 32 : 16;                              // input channels per step
};

typedef __attribute__((address_space(3))) unsigned char lds_u8_t;

// d[r][q] += w[q] * e[r * STEP][q] of lane + SH in the same row of 16 lanes (0 beyond it), for the rows of a unit, 4 channels
// each.  The shift rides on the multiply-add (a data-parallel operand; the compiler does not fold it into a fused
// multiply-add, which cost 3 moves per output element); the s_nop covers the two wait states such an operand needs after
// a vector write.
#define AGO_FMAC(D, E, W, SHIFT) "v_fmac_f32_dpp %" #D ", %" #E ", %" #W " " SHIFT " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define AGO_DW2(SHIFT)                                                                                                             \
    asm("s_nop 1\n\t" AGO_FMAC(0, 8, 16, SHIFT) AGO_FMAC(1, 9, 17, SHIFT) AGO_FMAC(2, 10, 18, SHIFT) AGO_FMAC(3, 11, 19, SHIFT)     \
            AGO_FMAC(4, 12, 16, SHIFT) AGO_FMAC(5, 13, 17, SHIFT) AGO_FMAC(6, 14, 18, SHIFT) AGO_FMAC(7, 15, 19, SHIFT)               \
        : "+v"(d0[0]), "+v"(d0[1]), "+v"(d0[2]), "+v"(d0[3]), "+v"(d1[0]), "+v"(d1[1]), "+v"(d1[2]), "+v"(d1[3])                    \
        : "v"(e0[0]), "v"(e0[1]), "v"(e0[2]), "v"(e0[3]), "v"(e1[0]), "v"(e1[1]), "v"(e1[2]), "v"(e1[3]), "v"(w[0]), "v"(w[1]),       \
          "v"(w[2]), "v"(w[3]))
#define AGO_DW1(SHIFT)                                                                                                             \
    asm("s_nop 1\n\t" AGO_FMAC(0, 4, 8, SHIFT) AGO_FMAC(1, 5, 9, SHIFT) AGO_FMAC(2, 6, 10, SHIFT) AGO_FMAC(3, 7, 11, SHIFT)         \
        : "+v"(d0[0]), "+v"(d0[1]), "+v"(d0[2]), "+v"(d0[3])                                                                        \
        : "v"(e0[0]), "v"(e0[1]), "v"(e0[2]), "v"(e0[3]), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]))
template <int SH>
__device__ __forceinline__ void dw_rows2(f32x4& d0, f32x4& d1, const f32x4& e0, const f32x4& e1, const f32x4& w) {
    if constexpr (SH == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) { d0[q] = fmaf(e0[q], w[q], d0[q]); d1[q] = fmaf(e1[q], w[q], d1[q]); }
    } else if constexpr (SH == 1) AGO_DW2("row_shl:1");
    else if constexpr (SH == 2) AGO_DW2("row_shl:2");
    else if constexpr (SH == -1) AGO_DW2("row_shr:1");
    else AGO_DW2("row_shr:2");
}
template <int SH>
__device__ __forceinline__ void dw_row(f32x4& d0, const f32x4& e0, const f32x4& w) {
    if constexpr (SH == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) d0[q] = fmaf(e0[q], w[q], d0[q]);
    } else if constexpr (SH == 1) AGO_DW1("row_shl:1");
    else if constexpr (SH == 2) AGO_DW1("row_shl:2");
    else if constexpr (SH == -1) AGO_DW1("row_shr:1");
    else AGO_DW1("row_shr:2");
}
#undef AGO_FMAC
#undef AGO_DW1
#undef AGO_DW2

// 16 rows (channels or output channels) x 32 reduction indices of a row-major weight tile in LDS: `p` is this lane's
// address in the first of the 32 k-rows + its group's offset, lo half k-rows 4 g .. + 3, hi half 16 further on
__device__ __forceinline__ bf16x8 invres_wfrag(const lds_u8_t* p, int pitch) {
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 16 * pitch));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// rows = output channels, columns = pixels, 16 reduction indices of which group g holds 4 g .. + 3
__device__ __forceinline__ f32x4 invres_mfma16(bf16x4 a, bf16x4 b, f32x4 c) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}

// Raw buffer accesses: a lane whose offset is kNowhere reads 0 and stores nothing, so that image borders, reduction tails and
// ragged tiles need neither branches nor clamped addresses (the straight-line code ahead of and behind the channel loop
// is what small maps spend their time on).  Tensors reached this way are below 2 GiB.
constexpr unsigned kNowhere = 0x80000000u;
typedef unsigned u32x4_b __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_b __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4_b buf_ld16(__amdgpu_buffer_rsrc_t r, unsigned off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }
// 16 bytes per lane to LDS at `dst` + 16 * lane (an instruction of its own: the compiler would wait for it before every
// LDS read); m0, the LDS base, is a reserved register that nothing else here uses
__device__ __forceinline__ void buf_to_lds(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(off), "s"(r) : "memory");
}

template <bool BF16, int STRIDE, int KS, int R, int XR, int NCO, int WPE, bool CHUNKED>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(WPE))) void invres_reg_kernel(const InvresRegParams p) {
    typedef InvresRegCfg<BF16, STRIDE, KS, R, XR, NCO> G;
    constexpr int PAD = G::PAD, ROWS = G::ROWS, TILES = G::TILES, ES = BF16 ? 2 : 4, KG = G::KG;
    extern __shared__ __align__(16) unsigned char smem[];
    lds_u8_t* lds = (lds_u8_t*)smem;
    const int tid = threadIdx.x, lane = tid & 63, nthreads = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    // per 16 channels: b1, bd, then the KS x KS taps, 16 fp32 each (constant offsets from one address)
    constexpr int kTileFloats = (2 + KS * KS) * 16;
    const int cb = blockIdx.y * p.cspan, ce = min(p.cspan + cb, p.Cexp);          // this workgroup's expanded channels
    const int co0 = blockIdx.z * NCO * 16;

    // Weights -> LDS.  W1 [k][channel] and W2 [channel][output channel] go as they are, 1 KB per wave and direct-to-LDS load:
    // all of their rows in one piece, or (channel split: a power of two) rows of csplit channels.  k-rows beyond Cin read
    // as 0.  Taps and biases are widened on the way, 4 channels per thread.
    auto stage = [&](int cs0, int cw) {
        const auto w1b = buffer_of(p.w1, p.Cin * p.Cexp * ES), w2b = buffer_of(p.w2, p.Cexp * p.Cout * ES);
        const unsigned lds0 = (unsigned)(uintptr_t)lds;
        for (int i = wave; i < p.n1; i += nthreads >> 6) {        // piece index 64 i + lane
            const int it = i * 64 + lane;
            const unsigned off = p.csplit == p.Cexp ? it * 16u : (unsigned)(((it >> p.q1_log) * p.Cexp + cs0) * ES + (it & ((1 << p.q1_log) - 1)) * 16);
            buf_to_lds(w1b, off, lds0 + i * 1024);
        }
        for (int i = wave; i < p.n2; i += nthreads >> 6) {
            const int it = i * 64 + lane;
            unsigned off = it * 16u;
            if (gridDim.z > 1) {                                  // 16 NCO of the output channels: rows of q2 pieces
                const int k = (int)__umulhi((unsigned)it, p.inv2);
                off = (unsigned)((k * p.Cout + co0) * ES + (it - k * p.q2) * 16);
            }
            buf_to_lds(w2b, off + cs0 * p.Cout * ES, lds0 + p.off_w2 + i * 1024);
        }
        for (int q = tid; q * 4 < cw; q += nthreads) {
            float* dst = reinterpret_cast<float*>(smem + p.off_wd) + (q >> 2) * kTileFloats + 4 * (q & 3);
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            const f32x4 b1 = p.b1 ? *reinterpret_cast<const f32x4*>(p.b1 + cs0 + 4 * q) : zero;
            const f32x4 bd = p.bd ? *reinterpret_cast<const f32x4*>(p.bd + cs0 + 4 * q) : zero;
            if constexpr (BF16) {
                const unsigned short* src = (const unsigned short*)p.wd + cs0 + 4 * q;
                uint2 u[KS * KS];
#pragma unroll
                for (int t = 0; t < KS * KS; ++t) u[t] = *reinterpret_cast<const uint2*>(src + t * p.Cexp);
#pragma unroll
                for (int t = 0; t < KS * KS; ++t)
                    *reinterpret_cast<f32x4*>(dst + (2 + t) * 16) = f32x4{lo_bf16(u[t].x), hi_bf16(u[t].x), lo_bf16(u[t].y), hi_bf16(u[t].y)};
            } else {
                const float* src = (const float*)p.wd + cs0 + 4 * q;
                f32x4 u[KS * KS];
#pragma unroll
                for (int t = 0; t < KS * KS; ++t) u[t] = *reinterpret_cast<const f32x4*>(src + t * p.Cexp);
#pragma unroll
                for (int t = 0; t < KS * KS; ++t) *reinterpret_cast<f32x4*>(dst + (2 + t) * 16) = u[t];
            }
            *reinterpret_cast<f32x4*>(dst) = b1;
            *reinterpret_cast<f32x4*>(dst + 16) = bd;
        }
    };

    if constexpr (!CHUNKED) stage(cb, ce - cb);

    const int nwc = 1 << p.nwc_log, wu = wave >> p.nwc_log, wc = wave & (nwc - 1);
    const auto xb = buffer_of(p.x, p.x_bytes);
    // lane-constant pieces of the LDS addresses
    const lds_u8_t* w1_lane = BF16 ? lds + (4 * g + (j >> 2)) * p.p1 + (j & 3) * 8 : lds + 4 * g * p.p1 + j * 4;
    const lds_u8_t* w2_lane = lds + p.off_w2 + (BF16 ? (4 * g + (j >> 2)) * p.p2 + (j & 3) * 8 : 4 * g * p.p2 + j * 4);

    for (int ug = blockIdx.x; ug * p.nwu < p.units; ug += gridDim.x) {
        const int unit = ug * p.nwu + wu;                 // one past the end: its pixels are nowhere
        // unit -> (strip, row block); two segments: lanes 8 .. 15 take the next row block of the flattened list
        int rb = p.strips == 1 ? unit : (int)__umulhi((unsigned)unit, p.inv_strips), ox;
        if (p.segs == 2) { rb = 2 * rb + (j >> 3); ox = j & 7; }
        else ox = (unit - rb * p.strips) * G::VX + j - G::LH;
        const int n = p.yblocks == 1 ? rb : (int)__umulhi((unsigned)rb, p.inv_yblocks), oy0 = (rb - n * p.yblocks) * R;
        const bool rb_ok = rb < p.rowblocks;
        const bool slot_ok = rb_ok && (unsigned)ox < (unsigned)p.OW && (p.segs == 2 || (j >= G::LH && j < G::LH + G::VX));

        // input pixels: byte offset (kNowhere outside the image) and relu6's upper bound there
        unsigned xoff[ROWS][TILES];
        float hi[ROWS][TILES];
        {
            const int iy0 = oy0 * STRIDE - PAD, ix0 = ox * STRIDE, row_bytes = p.W * p.Cin * ES;
            unsigned row = (unsigned)((n * p.H + iy0) * p.W + ix0) * (unsigned)(p.Cin * ES) + 4 * g * ES;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const bool row_ok = rb_ok && (unsigned)(iy0 + r) < (unsigned)p.H;
#pragma unroll
                for (int t = 0; t < TILES; ++t) {
                    const bool in = row_ok && (unsigned)(ix0 + t) < (unsigned)p.W;
                    hi[r][t] = in ? 6.f : 0.f;
                    xoff[r][t] = in ? row + t * p.Cin * ES : kNowhere;
                }
                row += row_bytes;
            }
        }
        // operand fragment of step ks: bf16: channels 32 ks + 4 g .. + 3 and 16 further on; fp32: 16 ks + 4 g .. + 3
        auto load_x = [&](int r, int t, int ks) -> u32x4_b {
            const int left = p.Cin - ks * KG - 4 * g;
            if constexpr (BF16) {
                const u32x2_b lo = __builtin_amdgcn_raw_buffer_load_b64(xb, xoff[r][t] | (left > 0 ? 0 : kNowhere), ks * 64, 0);
                const u32x2_b up = __builtin_amdgcn_raw_buffer_load_b64(xb, xoff[r][t] | (left > 16 ? 0 : kNowhere), ks * 64 + 32, 0);
                return u32x4_b{lo[0], lo[1], up[0], up[1]};
            } else {
                return __builtin_amdgcn_raw_buffer_load_b128(xb, xoff[r][t] | (left > 0 ? 0 : kNowhere), ks * 64, 0);
            }
        };
        u32x4_b xf[XR ? ROWS * TILES * XR : 1];
        unsigned char* xs = smem + p.off_x + wu * ROWS * TILES * p.nk * 1024 + lane * 16;
        // accumulators: rows = output channels 16 o + 4 g .., columns = output columns; the first part starts from b2
        f32x4 acc[R][NCO];
        if (XR == 0 && ug != (int)blockIdx.x) __syncthreads();                    // the previous unit's fragments are no longer read
        if constexpr (XR > 0) {
#pragma unroll
            for (int ks = 0; ks < XR; ++ks)
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int t = 0; t < TILES; ++t) xf[(r * TILES + t) * XR + ks] = load_x(r, t, ks);
        } else {                                          // the parts of a unit share its fragments in LDS
            for (int ks = wc; ks < p.nk; ks += nwc) {
                u32x4_b v[ROWS][TILES];
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int t = 0; t < TILES; ++t) v[r][t] = load_x(r, t, ks);
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int t = 0; t < TILES; ++t) *reinterpret_cast<u32x4_b*>(xs + ((ks * ROWS + r) * TILES + t) * 1024) = v[r][t];
            }
        }
        {
            const auto bb = buffer_of(p.b2, p.b2 && p.nsplit == 1 && wc == 0 ? p.Cout * 4 : 0);
#pragma unroll
            for (int o = 0; o < NCO; ++o) {
                const f32x4 v = __builtin_bit_cast(f32x4, buf_ld16(bb, (co0 + o * 16 + 4 * g) * 4));
#pragma unroll
                for (int r = 0; r < R; ++r) acc[r][o] = v;
            }
        }
        if constexpr (!CHUNKED) {
            if (ug == (int)blockIdx.x) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's direct-to-LDS loads
            if (XR == 0 || ug == (int)blockIdx.x) __syncthreads();
        } else if (XR == 0 && p.residual) {
            __syncthreads();
        }
        // the residual: an output pixel's own input is among the fragments, in the accumulators' channel order
        if (STRIDE == 1 && p.residual && p.nsplit == 1 && wc == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int o = 0; o < NCO; ++o) {
                    const int ks = BF16 ? o / 2 : o;
                    u32x4_b v;
                    if constexpr (XR > 0) v = ks < XR ? xf[(r + PAD) * XR + (ks < XR ? ks : 0)] : u32x4_b{0, 0, 0, 0};
                    else v = *reinterpret_cast<const u32x4_b*>(xs + (min(co0 / KG + ks, p.nk - 1) * ROWS + r + PAD) * 1024);
                    if constexpr (BF16) {
                        const unsigned a = v[2 * (o & 1)], c = v[2 * (o & 1) + 1];
                        acc[r][o] += f32x4{lo_bf16(a), hi_bf16(a), lo_bf16(c), hi_bf16(c)};
                    } else {
                        acc[r][o] += __builtin_bit_cast(f32x4, v);
                    }
                }
        }

        auto walk = [&](int cw) {
        for (int ct = wc; ct * 16 < cw; ct += nwc) {      // 16 expanded channels at a time
            const float* tw = reinterpret_cast<const float*>(smem + p.off_wd) + ct * kTileFloats + 4 * g;
            const f32x4 b1 = *reinterpret_cast<const f32x4*>(tw);
            f32x4 e[ROWS][TILES];
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int t = 0; t < TILES; ++t) e[r][t] = b1;
            auto expand = [&](int ks, auto&& frag) {
                if constexpr (BF16) {
                    const bf16x8 w = invres_wfrag(w1_lane + ks * 32 * p.p1 + ct * 32, p.p1);
#pragma unroll
                    for (int r = 0; r < ROWS; ++r)
#pragma unroll
                        for (int t = 0; t < TILES; ++t)
                            e[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, __builtin_bit_cast(bf16x8, frag(r, t)), e[r][t], 0, 0, 0);
                } else {
                    float w[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        w[q] = *(const __attribute__((address_space(3))) float*)(w1_lane + (ks * 16 + q) * p.p1 + ct * 64);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int r = 0; r < ROWS; ++r)
#pragma unroll
                            for (int t = 0; t < TILES; ++t)
                                e[r][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q], __builtin_bit_cast(f32x4, frag(r, t))[q], e[r][t], 0, 0, 0);
                }
            };
            if constexpr (XR > 0) {
#pragma unroll
                for (int ks = 0; ks < XR; ++ks) expand(ks, [&](int r, int t) { return xf[(r * TILES + t) * XR + ks]; });
            } else {
                for (int ks = 0; ks < p.nk; ++ks)
                    expand(ks, [&](int r, int t) { return *reinterpret_cast<const u32x4_b*>(xs + ((ks * ROWS + r) * TILES + t) * 1024); });
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int t = 0; t < TILES; ++t)
#pragma unroll
                    for (int q = 0; q < 4; ++q) e[r][t][q] = __builtin_amdgcn_fmed3f(e[r][t][q], 0.f, hi[r][t]);
            // depthwise; the fences keep the taps' registers from piling up
            __builtin_amdgcn_sched_barrier(0);
            f32x4 d[R];
            {
                const f32x4 bd = *reinterpret_cast<const f32x4*>(tw + 16);
#pragma unroll
                for (int r = 0; r < R; ++r) d[r] = bd;
            }
            auto taps = [&](auto kxc) {
                constexpr int kx = decltype(kxc)::value, dx = kx - PAD;
                constexpr int t = STRIDE == 1 ? 0 : (dx & 1), sh = STRIDE == 1 ? dx : (dx - (dx & 1)) / 2;
#pragma unroll
                for (int ky = 0; ky < KS; ++ky) {
                    const f32x4 w = *reinterpret_cast<const f32x4*>(tw + (2 + ky * KS + kx) * 16);
#pragma unroll
                    for (int r = 0; r + 1 < R; r += 2)
                        dw_rows2<sh>(d[r], d[r + 1], e[r * STRIDE + ky][t], e[(r + 1) * STRIDE + ky][t], w);
                    if constexpr (R & 1) dw_row<sh>(d[R - 1], e[(R - 1) * STRIDE + ky][t], w);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            taps(std::integral_constant<int, 0>{}); taps(std::integral_constant<int, 1>{}); taps(std::integral_constant<int, 2>{});
            if constexpr (KS == 5) { taps(std::integral_constant<int, 3>{}); taps(std::integral_constant<int, 4>{}); }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) d[r][q] = __builtin_amdgcn_fmed3f(d[r][q], 0.f, 6.f);
            // projection of these 16 channels: a lane of group g brings channels 4 g .. + 3
            if constexpr (BF16) {
                bf16x4 db[R];
#pragma unroll
                for (int r = 0; r < R; ++r) db[r] = __builtin_bit_cast(bf16x4, u32x2_b{pack_bf16(d[r][0], d[r][1]), pack_bf16(d[r][2], d[r][3])});
#pragma unroll
                for (int o = 0; o < NCO; ++o) {
                    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
                    const bf16x4 w = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(w2_lane + ct * 16 * p.p2 + o * 32));
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r][o] = invres_mfma16(w, db[r], acc[r][o]);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int o = 0; o < NCO; ++o) {
                        const float w = *(const __attribute__((address_space(3))) float*)(w2_lane + (ct * 16 + q) * p.p2 + o * 64);
#pragma unroll
                        for (int r = 0; r < R; ++r) acc[r][o] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, d[r][q], acc[r][o], 0, 0, 0);
                    }
            }
        }
        };
        if constexpr (CHUNKED) {
            for (int cs = cb; cs < ce; cs += p.csplit) {
                if (cs > cb || ug != (int)blockIdx.x) __syncthreads();            // the previous chunk is no longer read
                stage(cs, min(p.csplit, ce - cs));
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                walk(min(p.csplit, ce - cs));
            }
        } else {
            walk(ce - cb);
        }

        // a lane holds 4 consecutive output channels of its output column, per row
        const unsigned out0 = (unsigned)(((n * p.OH + oy0) * p.OW + ox) * p.Cout + co0 + 4 * g);
        const int left = min(NCO * 16, p.Cout - co0) - 4 * g;
        const auto yb = p.nsplit > 1 ? buffer_of(p.part + (long)blockIdx.y * p.out_elems, p.out_elems * 4) : buffer_of(p.y, p.out_elems * ES);
        auto emit = [&](int r, int o, const f32x4& v) {
            const bool ok = slot_ok && oy0 + r < p.OH && 16 * o < left;
            const unsigned at = out0 + r * p.OW * p.Cout + o * 16;
            if (BF16 && p.nsplit == 1)
                __builtin_amdgcn_raw_buffer_store_b64(u32x2_b{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])}, yb, ok ? at * 2 : kNowhere, 0, 0);
            else
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_b, v), yb, ok ? at * 4 : kNowhere, 0, 0);
        };
        if (nwc == 1) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int o = 0; o < NCO; ++o) emit(r, o, acc[r][o]);
        } else {
            // partial projections of the parts -> LDS; part wc then finishes the pieces wc, wc + nwc, ...
            f32x4* red = reinterpret_cast<f32x4*>(smem + p.off_red) + (wu << p.nwc_log) * R * NCO * 64 + lane;
            __syncthreads();                              // weights and fragments may lie under it
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int o = 0; o < NCO; ++o) red[((wc * R + r) * NCO + o) * 64] = acc[r][o];
            __syncthreads();
            for (int i = wc; i < R * NCO; i += 2 * nwc) {  // two at a time: one's reads under the other's
                const int k = min(i + nwc, R * NCO - 1);
                f32x4 v = red[i * 64], w = red[k * 64];
                for (int q = 1; q < nwc; ++q) { v += red[(q * R * NCO + i) * 64]; w += red[(q * R * NCO + k) * 64]; }
                emit(i / NCO, i % NCO, v);
                if (i + nwc < R * NCO) emit(k / NCO, k % NCO, w);
            }
        }
    }
}

// Instantiations: output rows of a unit by stride and depthwise size, steps of the input fragments kept in registers
// (XR; 0: the fragments sit in LDS), 16-wide tiles of output channels.
constexpr int kRegR[2][2] = {{2, 4}, {1, 2}};             // [stride - 1][option]
constexpr int kRegNco[4] = {2, 4, 6, 10};

// one translation unit each (dtype, stride, depthwise size), so that they compile side by side
#define AGO_REG_DECL(NAME) hipError_t NAME(int ropt, int xr, int nco, const InvresRegParams& p, unsigned grid, unsigned threads, size_t smem, hipStream_t s);
AGO_REG_DECL(invres_reg_b13) AGO_REG_DECL(invres_reg_b15) AGO_REG_DECL(invres_reg_b23) AGO_REG_DECL(invres_reg_b25)
AGO_REG_DECL(invres_reg_f13) AGO_REG_DECL(invres_reg_f15) AGO_REG_DECL(invres_reg_f23) AGO_REG_DECL(invres_reg_f25)

template <bool BF16, int STRIDE, int KS, int R, int XR, int NCO, int WPE, bool CHUNKED>
static hipError_t invres_reg_start(const InvresRegParams& p, unsigned grid, unsigned threads, size_t smem, hipStream_t s) {
    if (hipError_t e = allow_dynamic_lds<invres_reg_kernel<BF16, STRIDE, KS, R, XR, NCO, WPE, CHUNKED>>(160 * 1024); e != hipSuccess) return e;
    hipLaunchKernelGGL((invres_reg_kernel<BF16, STRIDE, KS, R, XR, NCO, WPE, CHUNKED>),
                       dim3(grid, (unsigned)p.nsplit, (unsigned)((p.Cout + 16 * NCO - 1) / (16 * NCO))), dim3(threads), smem, s, p);
    return hipGetLastError();
}
// registers a variant needs, about: fragments, E, pixel offsets and bounds, D, projection tiles, and what the rest was seen
// to take.  Fragments that would not fit 256 beside the rest go through LDS; up to 168, three waves share a SIMD.
constexpr int reg_need(bool bf16, int stride, int ksize, int R, int xr, int nco) {
    const int frags = ((R - 1) * stride + ksize) * stride;
    return frags * (4 * xr + 4 + 2) + 4 * R + 4 * R * nco + (bf16 ? 36 + 2 * nco : 62);
}
constexpr int reg_waves(bool bf16, int stride, int ksize, int R, int xr, int nco) { return reg_need(bf16, stride, ksize, R, xr, nco) <= 168 ? 3 : 2; }
template <bool BF16, int STRIDE, int KS, int R, int XR, int NCO>
static hipError_t invres_reg_nco(int nco, const InvresRegParams& p, unsigned grid, unsigned threads, size_t smem, hipStream_t s) {
    if constexpr ((R <= 2 || (XR > 0 && NCO <= 4)) && reg_need(BF16, STRIDE, KS, R, XR, NCO) <= 256) {
        constexpr int WPE = reg_waves(BF16, STRIDE, KS, R, XR, NCO);
        if constexpr (R == kRegR[STRIDE - 1][0]) {
            if (nco == NCO && p.csplit < p.cspan) return invres_reg_start<BF16, STRIDE, KS, R, XR, NCO, WPE, true>(p, grid, threads, smem, s);
        }
        if (nco == NCO) return invres_reg_start<BF16, STRIDE, KS, R, XR, NCO, WPE, false>(p, grid, threads, smem, s);
    }
    if constexpr (NCO == 2) return invres_reg_nco<BF16, STRIDE, KS, R, XR, 4>(nco, p, grid, threads, smem, s);
    if constexpr (NCO == 4) return invres_reg_nco<BF16, STRIDE, KS, R, XR, 6>(nco, p, grid, threads, smem, s);
    if constexpr (NCO == 6) return invres_reg_nco<BF16, STRIDE, KS, R, XR, 10>(nco, p, grid, threads, smem, s);
    return hipErrorInvalidValue;
}
// fragment steps kept in registers: 1 .. 5 of 32 bf16 channels, 2 or 4 of 16 fp32 ones; 0: in LDS
template <bool BF16, int STRIDE, int KS, int R, int XR>
static hipError_t invres_reg_xr(int xr, int nco, const InvresRegParams& p, unsigned grid, unsigned threads, size_t smem, hipStream_t s) {
    if (xr == XR) return invres_reg_nco<BF16, STRIDE, KS, R, XR, 2>(nco, p, grid, threads, smem, s);
    constexpr int NEXT = XR + (BF16 ? 1 : 2);
    if constexpr (NEXT <= (BF16 ? 5 : 4)) return invres_reg_xr<BF16, STRIDE, KS, R, NEXT>(xr, nco, p, grid, threads, smem, s);
    return hipErrorInvalidValue;
}
template <bool BF16, int STRIDE, int KS>
static hipError_t invres_reg_run(int ropt, int xr, int nco, const InvresRegParams& p, unsigned grid, unsigned threads, size_t smem, hipStream_t s) {
    if (ropt == 0) return invres_reg_xr<BF16, STRIDE, KS, kRegR[STRIDE - 1][0], 0>(xr, nco, p, grid, threads, smem, s);
    return invres_reg_xr<BF16, STRIDE, KS, kRegR[STRIDE - 1][1], 0>(xr, nco, p, grid, threads, smem, s);
}

}  // namespace ago
