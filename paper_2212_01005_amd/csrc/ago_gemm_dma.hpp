// bf16 matrix product C[M][N] = act(A[M][K] W[K][N] + bias (+ R)), fp32 accumulation, K a multiple of 32.
//
// Both operands travel global -> LDS with the direct-to-LDS load (no registers, no LDS store instructions) through a
// ring of NST stages of 32 reduction steps; the waves multiply stage t while the stages behind it are in flight.  W is
// either row-major, read with the transposing LDS read, or packed into matrix-instruction fragments (pack_weight), read
// 16 bytes a lane; it is operand A of the matrix instruction, so a lane ends up with 4 consecutive columns of one row.
//
// Two forms: gemm_dma_kernel, whose waves divide the tile of C between them and meet at one barrier per stage (large
// products), and gemm_split_kernel, whose waves divide the reduction of one small tile (few rows or few columns).
//
// What bounds them, measured on an MI355X: large products run at 1.0 - 1.1 PFLOP/s (8192 x 1024 x 4096: 66 us, register-
// staged tiles of 128 x 192 before: 138 us), the matrix cores busy 55 - 60 % of the cycles, LDS a third, the rest is
// barrier skew and the start and end of each tile, which two workgroups to a compute unit hide in part; small ones by
// the launch, the first loads' latency (3.5 us together) and what a compute unit can pull out of the L2 (100 GB/s).
//
// LDS layouts in 16-byte chunks (the loads realise the permutation by choosing which global chunk a lane fetches):
//   A stage [BM rows][32 k]   64-byte rows,  chunk ^= (row >> 2) & 3
//   W stage [32 k][BN cols]   BN * 2-byte rows, 64-byte unit ^= k & 3 (rows a multiple of 256 bytes) or (k >> 1) & 1
// Both make the fragment reads bank-conflict free.
#pragma once
#include "ago_dev.hpp"
#include "ago_launch.hpp"
#include <type_traits>

namespace ago {

typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 lds_read_a(const lds_u8* p) {
    typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
    return *(const lds_bf16x8*)p;
}
// p: this lane's address in k-row (k0 + lane-dependent row) of a row-major W stage; stride: bytes per k-row
__device__ __forceinline__ bf16x8 lds_read_w(const lds_u8* p, int stride) {
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 4 * stride));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

struct GemmDmaParams {
    const bf16_t* a;
    const bf16_t *w0, *w1, *w2;  // siblings that share A (one for a plain product, three for the q / k / v projections)
    const float *b0, *b1, *b2;
    const bf16_t* r;             // residual, plain product only
    bf16_t *c0, *c1, *c2;
    int M, K, N;                 // N: columns of one sibling, a multiple of 8 (packed: 16)
    int tiles_m, tiles_n;        // tiles_n: column tiles of one sibling
    int siblings;
    int act;                     // read by the kActRuntime instantiations only
    int S, Hh, D;                // kEpHeadMajor: C is [B][Hh][S][D] instead of [M][N] = [B][S][Hh][D]; D % 8 == 0
};

// one wave: 64 lanes x 16 bytes from base + voff (per lane) to LDS at `lds` + 16 * lane.  Written as an instruction of
// its own because the compiler, which cannot tell the ring's stages apart, would wait for every outstanding load ahead
// of each LDS read; dma_wait() and the barrier order the two instead.  (m0, the LDS base of such loads, is a reserved
// register: nothing else in these kernels uses it.)
__device__ __forceinline__ void dma_16(const void* base, unsigned voff, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory");
}
__device__ __forceinline__ const unsigned char* uniform_ptr(const void* p) {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const unsigned char*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
// at most N of this wave's loads still in flight, all of its LDS reads returned; then the workgroup barrier
template <int N, bool BARRIER>
__device__ __forceinline__ void dma_wait() {
    if constexpr (BARRIER) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

struct GemmTile { int tm, sib, tn; };
// launch index -> tile: an XCD (index mod 8) takes a contiguous share of the tiles, ordered in bands of 8 row tiles so
// that what its workgroups read at one time fits its L2
__device__ __forceinline__ GemmTile gemm_tile_of(const GemmDmaParams& p, int bid) {
    const int TN = p.tiles_n * p.siblings, T = p.tiles_m * TN;
    const int q = T >> 3, r = T & 7, x = bid & 7;
    const int id = x * q + min(x, r) + (bid >> 3);
    const int band = id / (8 * TN), in = id - band * 8 * TN, rows = min(8, p.tiles_m - band * 8);
    const int tnn = in / rows, sib = tnn / p.tiles_n;
    return {band * 8 + (in - tnn * rows), sib, tnn - sib * p.tiles_n};
}
// byte offset, from row m0 of A, of lane's 16 bytes of load instruction q (16 rows x 64 bytes) of an A stage
__device__ __forceinline__ unsigned gemm_a_voff(int q, int lane, int last_row, int K) {
    const int row = q * 16 + (lane >> 2);
    return (unsigned)((long)min(row, last_row) * K * 2 + (((lane & 3) ^ ((row >> 2) & 3)) << 4));
}
// swizzle of 16-byte chunks in k-row k of a W stage with BN columns: four consecutive k-rows of 32 columns then cover
// the 64 banks once (rows of 64 or 192 bytes mod 256 do by themselves)
template <int BN>
__device__ __forceinline__ int gemm_w_swz(int k) {
    return BN * 2 % 256 == 0 ? (k & 3) << 2 : BN * 2 % 256 == 128 ? ((k >> 1) & 1) << 2 : 0;
}
// the same for load instruction q of a W stage: 64 chunks of the [32][BN] tile in row order, or one packed fragment
template <int BN, bool PACKED>
__device__ __forceinline__ unsigned gemm_w_voff(int q, int lane, int n0, int N) {
    if constexpr (PACKED) {
        return (unsigned)(min(n0 / 16 + q, N / 16 - 1) * 1024 + lane * 16);
    } else {
        constexpr int CPR = BN / 8;
        const int c = q * 64 + lane, k = c / CPR, pc = c % CPR;
        return (unsigned)(((long)k * N + min(n0 + ((pc ^ gemm_w_swz<BN>(k)) << 3), N - 8)) * 2);
    }
}
// byte offset inside a W stage of lane's fragment of 32-column tile nt, first half step (packed: the second is 512 bytes
// on; else 16 k-rows on)
template <int BN, bool PACKED>
__device__ __forceinline__ int gemm_w_frag(int lane, int nt) {
    if constexpr (PACKED) return (2 * nt + ((lane & 31) >> 4)) * 1024 + (lane >> 5) * 256 + (lane & 15) * 16;
    const int g = lane >> 4, s = lane & 15, k = 8 * (g >> 1) + (s >> 2);
    const int chunk = nt * 4 + 2 * (g & 1) + ((s & 3) >> 1);
    return k * BN * 2 + ((chunk ^ gemm_w_swz<BN>(k)) << 4) + 8 * (s & 1);
}

template <int BM_, int BN_, int WM_, int WN_, int NST_>
struct GemmDmaCfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NST = NST_, BK = 32;
    static constexpr int WAVES = WM * WN, THREADS = WAVES * 64;
    static constexpr int MT = BM / WM / 32, NT = BN / WN / 32;
    static constexpr int A_BYTES = BM * 64, W_ROW = BN * 2, W_BYTES = 32 * W_ROW, STAGE = A_BYTES + W_BYTES;
    static constexpr int A_LD = A_BYTES / 1024, W_LD = W_BYTES / 1024;       // load instructions per stage
    static constexpr int LD = (A_LD + W_LD + WAVES - 1) / WAVES;             // per wave; the last may be repeated
    static_assert(A_LD % WAVES == 0 && BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "whole 32 x 32 tiles");
    static constexpr int EP_ROW = NT * 64 + 16;                              // epilogue: bytes per row of a parked 32-row tile
    static constexpr int EP_BYTES = WAVES * 32 * EP_ROW;
    static constexpr int SMEM = NST * STAGE > EP_BYTES ? NST * STAGE : EP_BYTES;
    static_assert(SMEM <= 160 * 1024, "LDS");
};

// The multiply loop of both kernels below, over `steps` reduction steps of 32 that pass through a ring of NST LDS stages
// at `ring`.  A load instruction u of a stage reads 16 bytes per lane at (u < LDA ? ap : wp) + voff[u] and lands at stage
// offset ldst[u]; ap / wp move by a_step / w_step bytes per stage, and past the end stay on the last step (loaded again,
// never used).  SHARED: the ring belongs to the workgroup (barriers), else to the wave.
//
// Two half steps of 16 per stage, fragments read one half step ahead.  In the middle of stage t the reader holds its last
// fragments of it: its slot then takes stage t + NST (the first half of the loads at once, the others in the first half
// of stage t + 1), and stage t + 1, which has landed, may be read.  The loads are spread between the matrix instructions:
// a wave that issues them in a row waits for the address unit (16 clocks a load, shared by the compute unit's waves).
template <int MT, int NT, int NST, int STAGE, int LD, int LDA, int W_ROW, bool PACKED, bool SHARED>
__device__ __forceinline__ void gemm_ring(f32x16 (&acc)[MT][NT], const lds_u8* ring, const unsigned char* ap, const unsigned char* wp,
                                          long a_step, long w_step, const unsigned (&voff)[LD], const unsigned (&ldst)[LD], int a_off,
                                          const int (&w_off)[NT], int steps) {
    constexpr int LD1 = LD / 2, TILES = MT * NT;
    const unsigned ring0 = (unsigned)(uintptr_t)ring;
    int left = steps - 1;
    auto issue_one = [&](unsigned slot, int u) { dma_16(u < LDA ? ap : wp, voff[u], ring0 + slot + ldst[u]); };
    auto advance = [&] { if (left > 0) { ap += a_step; wp += w_step; --left; } };
    struct Frags { bf16x8 a[MT], w[NT]; };
    auto fetch = [&](Frags& f, const lds_u8* st, int ks) {
#pragma unroll
        for (int n = 0; n < NT; ++n) f.w[n] = PACKED ? lds_read_a(st + w_off[n] + ks * 512) : lds_read_w(st + w_off[n] + ks * 16 * W_ROW, W_ROW);
#pragma unroll
        for (int m = 0; m < MT; ++m) f.a[m] = lds_read_a(st + (a_off ^ (ks * 32)) + m * 2048);
    };
    auto mma = [&](const Frags& f, unsigned slot, auto u0c, auto u1c) {
        constexpr int U0 = decltype(u0c)::value, U1 = decltype(u1c)::value;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int i = m * NT + n;
                acc[m][n] = mfma32(f.w[n], f.a[m], acc[m][n]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = U0 + i * (U1 - U0) / TILES; u < U0 + (i + 1) * (U1 - U0) / TILES; ++u) issue_one(slot, u);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    typedef std::integral_constant<int, 0> C0;
    typedef std::integral_constant<int, LD1> C1;
    typedef std::integral_constant<int, LD> C2;
#pragma unroll
    for (int t = 0; t < NST; ++t) {
#pragma unroll
        for (int u = 0; u < (t + 1 < NST ? LD : LD1); ++u) issue_one(t * STAGE, u);
        if (t + 1 < NST) advance();
    }
    dma_wait<(NST - 2) * LD + LD1, SHARED>();
    Frags f0, f1;
    fetch(f0, ring, 0);
    int slot = 0, prev = (NST - 1) * STAGE;
    for (int t = 0; t < steps; ++t) {
        const int next = slot == (NST - 1) * STAGE ? 0 : slot + STAGE;
        fetch(f1, ring + slot, 1);
        __builtin_amdgcn_sched_barrier(0);
        mma(f0, prev, C1{}, C2{});
        advance();
        dma_wait<(NST - 2) * LD, SHARED>();
        fetch(f0, ring + next, 0);                     // past the end: the repeated last step, dropped
        __builtin_amdgcn_sched_barrier(0);
        mma(f1, slot, C0{}, C1{});
        prev = slot;
        slot = next;
    }
    dma_wait<0, true>();                               // nothing in flight, every wave is done reading: LDS is free
}

enum GemmEpilogue { kEpPlain = 0, kEpResidual = 1, kEpHeadMajor = 2 };
constexpr int kActRuntime = -1;
template <int ACT>
__device__ __forceinline__ float gemm_act(float v, int act) {
    if constexpr (ACT == kActRuntime) return apply_act_rt(v, act);
    else return apply_act<ACT>(v);
}

template <typename G, int ACT, int EP, bool PACKED>
__global__ __launch_bounds__(G::THREADS, 2) void gemm_dma_kernel(const GemmDmaParams p) {
    constexpr int BM = G::BM, BN = G::BN, MT = G::MT, NT = G::NT, WN = G::WN;
    extern __shared__ __align__(16) unsigned char smem[];
    lds_u8* lds = (lds_u8*)smem;
    const unsigned lds0 = (unsigned)(uintptr_t)lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int j = lane & 31, h = lane >> 5;

    const GemmTile tile = gemm_tile_of(p, blockIdx.x);
    const int sib = tile.sib, m0 = tile.tm * BM, n0 = tile.tn * BN;
    const bf16_t* W = sib == 0 ? p.w0 : sib == 1 ? p.w1 : p.w2;

    // per-lane global offsets of this wave's load instructions (bytes from the operand's base, first reduction step)
    unsigned voff[G::LD], ldst[G::LD];
#pragma unroll
    for (int u = 0; u < G::LD; ++u) {
        const int q = min(wave + u * G::WAVES, G::A_LD + G::W_LD - 1);      // instruction index inside the stage: A first, then W
        ldst[u] = q * 1024;
        voff[u] = u < G::A_LD / G::WAVES ? gemm_a_voff(q, lane, p.M - 1 - m0, p.K)
                                         : gemm_w_voff<BN, PACKED>(q - G::A_LD, lane, n0, p.N);
    }
    // the next stage to request: uniform base addresses, moved on by one reduction step per stage; past the end they stay
    // on the last step (loaded again, never read)
    const unsigned char* ap = uniform_ptr(p.a + (long)m0 * p.K);
    const unsigned char* wp = uniform_ptr(W);
    const long w_step = (long)32 * p.N * 2;            // bytes between reduction steps, packed or not
    const int nk = p.K / 32;
    // fragment addresses inside a stage
    const int a_off = (wm * MT * 32 + j) * 64 + ((h ^ ((j >> 2) & 3)) << 4);
    int w_off[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) w_off[n] = G::A_BYTES + gemm_w_frag<BN, PACKED>(lane, wn * NT + n);
    f32x16 acc[MT][NT];
    zero_acc(acc);
    gemm_ring<MT, NT, G::NST, G::STAGE, G::LD, G::A_LD / G::WAVES, G::W_ROW, PACKED, true>(
        acc, lds, ap, wp, 64, w_step, voff, ldst, a_off, w_off, nk);

    // epilogue, one 32-row tile of the wave at a time: bias, residual, activation in fp32, rounded, through the wave's
    // own piece of LDS so that the global stores are whole 16-byte chunks of consecutive columns
    typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) u32x2_t lds_u32x2;
    typedef __attribute__((address_space(3))) u32x4_t lds_u32x4;
    const float* bias = sib == 0 ? p.b0 : sib == 1 ? p.b1 : p.b2;
    bf16_t* C = sib == 0 ? p.c0 : sib == 1 ? p.c1 : p.c2;
    lds_u8* ep = lds + wave * 32 * G::EP_ROW;
    const int nw0 = n0 + wn * NT * 32, mw0 = m0 + wm * MT * 32;
    f32x4 bv[NT][4];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            bv[n][g] = bias ? *reinterpret_cast<const f32x4*>(bias + min(nw0 + n * 32 + 8 * g + 4 * h, p.N - 4)) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        u32x2_t res[NT][4];
        if constexpr (EP == kEpResidual) {
            const bf16_t* r = p.r + (long)min(mw0 + m * 32 + j, p.M - 1) * p.N;
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int g = 0; g < 4; ++g) res[n][g] = *reinterpret_cast<const u32x2_t*>(r + min(nw0 + n * 32 + 8 * g + 4 * h, p.N - 4));
        }
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[m][n][4 * g + e] + bv[n][g][e];
                if constexpr (EP == kEpResidual) {
                    v[0] += lo_bf16(res[n][g][0]); v[1] += hi_bf16(res[n][g][0]);
                    v[2] += lo_bf16(res[n][g][1]); v[3] += hi_bf16(res[n][g][1]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = gemm_act<ACT>(v[e], p.act);
                *(lds_u32x2*)(ep + j * G::EP_ROW + n * 64 + g * 16 + h * 8) = u32x2_t{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            }
        __builtin_amdgcn_wave_barrier();
        constexpr int CPR = NT * 4;
#pragma unroll
        for (int it = 0; it < 2 * NT; ++it) {
            const int u = it * 64 + lane, rr = u / CPR, c = u % CPR;
            const u32x4_t v = *(const lds_u32x4*)(ep + rr * G::EP_ROW + c * 16);
            const int grow = mw0 + m * 32 + rr, gcol = nw0 + c * 8;
            if (grow < p.M && gcol < p.N) {
                long off = (long)grow * p.N + gcol;
                if constexpr (EP == kEpHeadMajor) {
                    const int bi = grow / p.S, s = grow - bi * p.S, hh = gcol / p.D, d = gcol - hh * p.D;
                    off = (((long)bi * p.Hh + hh) * p.S + s) * p.D + d;
                }
                *reinterpret_cast<u32x4_t*>(C + off) = v;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Products with too few tiles for the kernel above: the WAVES waves of a workgroup share one BM x BN tile and split its
// reduction, each with a private ring of NST stages in LDS (no barrier until the end) holding its own 32-deep pieces of A
// and W.  Wave w takes the reduction steps w, w + WAVES, ...; the partial tiles meet in LDS in wave order.
template <int BM_, int BN_, int WAVES_, int NST_>
struct GemmSplitCfg {
    static constexpr int BM = BM_, BN = BN_, WAVES = WAVES_, NST = NST_, THREADS = WAVES * 64;
    static constexpr int MT = BM / 32, NT = BN / 32;
    static constexpr int A_BYTES = BM * 64, W_ROW = BN * 2, STAGE = A_BYTES + 32 * W_ROW;
    static constexpr int A_LD = BM / 16, W_LD = BN / 16, LD = A_LD + W_LD;
    static constexpr int PARK_ROW = BN * 4 + 16, PARK = 32 * PARK_ROW;       // one 32-row tile of a wave
    static constexpr int SMEM = WAVES * NST * STAGE > WAVES * PARK ? WAVES * NST * STAGE : WAVES * PARK;
    static_assert(BM % 32 == 0 && BN % 32 == 0 && SMEM <= 160 * 1024, "LDS");
};

template <typename G, int ACT, int EP, bool PACKED>
__global__ __launch_bounds__(G::THREADS) void gemm_split_kernel(const GemmDmaParams p) {
    constexpr int BM = G::BM, BN = G::BN, MT = G::MT, NT = G::NT;
    extern __shared__ __align__(16) unsigned char smem[];
    lds_u8* lds = (lds_u8*)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 31, h = lane >> 5;
    const GemmTile tile = gemm_tile_of(p, blockIdx.x);
    const int sib = tile.sib, m0 = tile.tm * BM, n0 = tile.tn * BN;
    const bf16_t* W = sib == 0 ? p.w0 : sib == 1 ? p.w1 : p.w2;

    unsigned voff[G::LD], ldst[G::LD];
#pragma unroll
    for (int u = 0; u < G::LD; ++u) {
        ldst[u] = u * 1024;
        voff[u] = u < G::A_LD ? gemm_a_voff(u, lane, p.M - 1 - m0, p.K) : gemm_w_voff<BN, PACKED>(u - G::A_LD, lane, n0, p.N);
    }
    const int nk = p.K / 32, steps = (nk - wave + G::WAVES - 1) / G::WAVES;       // this wave's steps; none: loads step nk - 1, unused
    const unsigned char* ap = uniform_ptr((const unsigned char*)(p.a + (long)m0 * p.K) + (long)min(wave, nk - 1) * 64);
    const unsigned char* wp = uniform_ptr((const unsigned char*)W + (long)min(wave, nk - 1) * 32 * p.N * 2);
    const int a_off = j * 64 + ((h ^ ((j >> 2) & 3)) << 4);
    int w_off[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) w_off[n] = G::A_BYTES + gemm_w_frag<BN, PACKED>(lane, n);
    f32x16 acc[MT][NT];
    zero_acc(acc);
    gemm_ring<MT, NT, G::NST, G::STAGE, G::LD, G::A_LD, G::W_ROW, PACKED, false>(
        acc, lds + wave * G::NST * G::STAGE, ap, wp, 64 * G::WAVES, (long)32 * p.N * 2 * G::WAVES, voff, ldst, a_off, w_off, steps);

    // partial tiles -> LDS as [row][column] fp32, 32 rows at a time; every thread then adds the copies of its 4-column
    // pieces in wave order
    const float* bias = sib == 0 ? p.b0 : sib == 1 ? p.b1 : p.b2;
    bf16_t* C = sib == 0 ? p.c0 : sib == 1 ? p.c1 : p.c2;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        if (m) __syncthreads();
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4*>(smem + wave * G::PARK + j * G::PARK_ROW + (n * 32 + 8 * g + 4 * h) * 4) =
                    make_float4(acc[m][n][4 * g], acc[m][n][4 * g + 1], acc[m][n][4 * g + 2], acc[m][n][4 * g + 3]);
        __syncthreads();
        for (int u = tid; u < 32 * BN / 4; u += G::THREADS) {
            const int rr = u / (BN / 4), c4 = u % (BN / 4) * 4, row = m0 + m * 32 + rr, col = n0 + c4;
            if (row >= p.M || col >= p.N) continue;
            const unsigned char* src = smem + rr * G::PARK_ROW + c4 * 4;
            float4 v = *reinterpret_cast<const float4*>(src);
#pragma unroll
            for (int q = 1; q < G::WAVES; ++q) {
                const float4 x = *reinterpret_cast<const float4*>(src + q * G::PARK);
                v.x += x.x; v.y += x.y; v.z += x.z; v.w += x.w;
            }
            if (bias) {
                const float4 b = *reinterpret_cast<const float4*>(bias + col);
                v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
            }
            if constexpr (EP == kEpResidual) {
                const uint2 x = *reinterpret_cast<const uint2*>(p.r + (long)row * p.N + col);
                v.x += lo_bf16(x.x); v.y += hi_bf16(x.x); v.z += lo_bf16(x.y); v.w += hi_bf16(x.y);
            }
            long off = (long)row * p.N + col;
            if constexpr (EP == kEpHeadMajor) {
                const int bi = row / p.S, s = row - bi * p.S, hh = col / p.D, d = col - hh * p.D;
                off = (((long)bi * p.Hh + hh) * p.S + s) * p.D + d;
            }
            *reinterpret_cast<uint2*>(C + off) = make_uint2(pack_bf16(gemm_act<ACT>(v.x, p.act), gemm_act<ACT>(v.y, p.act)),
                                                             pack_bf16(gemm_act<ACT>(v.z, p.act), gemm_act<ACT>(v.w, p.act)));
        }
    }
}

// The tilings, in the order of the time model in ago_gemm_dma.hip: BM, BN, then waves along M and N (or waves that split
// the reduction) and ring stages.
#define AGO_GEMM_TILINGS(SHARED, SPLIT)                                                                          \
    SHARED(0, 128, 256, 1, 4, 3) SHARED(1, 128, 256, 2, 4, 6) SHARED(2, 128, 192, 2, 2, 4)                       \
    SHARED(3, 128, 128, 2, 2, 4) SHARED(4, 64, 128, 1, 4, 4)                                                     \
    SPLIT(5, 64, 96, 4, 4) SPLIT(6, 64, 64, 8, 2) SPLIT(7, 64, 32, 8, 3) SPLIT(8, 32, 32, 8, 4) SPLIT(9, 32, 64, 8, 3)
constexpr int kGemmTilings = 10;

template <typename G, int ACT, int EP, bool PACKED>
static hipError_t gemm_dma_start(GemmDmaParams p, hipStream_t s) {
    if (hipError_t e = allow_dynamic_lds<gemm_dma_kernel<G, ACT, EP, PACKED>>(G::SMEM); e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_dma_kernel<G, ACT, EP, PACKED>), dim3((unsigned)(p.tiles_m * p.tiles_n * p.siblings)), dim3(G::THREADS),
                       G::SMEM, s, p);
    return hipGetLastError();
}
template <typename G, int ACT, int EP, bool PACKED>
static hipError_t gemm_split_start(GemmDmaParams p, hipStream_t s) {
    if (hipError_t e = allow_dynamic_lds<gemm_split_kernel<G, ACT, EP, PACKED>>(G::SMEM); e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_split_kernel<G, ACT, EP, PACKED>), dim3((unsigned)(p.tiles_m * p.tiles_n * p.siblings)), dim3(G::THREADS),
                       G::SMEM, s, p);
    return hipGetLastError();
}
template <int ACT, int EP, bool PACKED>
static hipError_t gemm_dma_tiling(int tiling, GemmDmaParams p, hipStream_t s) {
    switch (tiling) {
#define AGO_GEMM_SHARED(ID, BM, BN, WM, WN, NST)                                                                 \
    case ID:                                                                                                     \
        p.tiles_m = (p.M + BM - 1) / BM; p.tiles_n = (p.N + BN - 1) / BN;                                        \
        return gemm_dma_start<GemmDmaCfg<BM, BN, WM, WN, NST>, ACT, EP, PACKED>(p, s);
#define AGO_GEMM_SPLIT(ID, BM, BN, WAVES, NST)                                                                   \
    case ID:                                                                                                     \
        p.tiles_m = (p.M + BM - 1) / BM; p.tiles_n = (p.N + BN - 1) / BN;                                        \
        return gemm_split_start<GemmSplitCfg<BM, BN, WAVES, NST>, ACT, EP, PACKED>(p, s);
        AGO_GEMM_TILINGS(AGO_GEMM_SHARED, AGO_GEMM_SPLIT)
#undef AGO_GEMM_SHARED
#undef AGO_GEMM_SPLIT
        default: return hipErrorInvalidValue;
    }
}

// one translation unit each, so that they compile side by side
hipError_t gemm_dma_rows(int tiling, const GemmDmaParams& p, hipStream_t s);         // row-major W, plain epilogue
hipError_t gemm_dma_packed(int tiling, const GemmDmaParams& p, hipStream_t s);       // packed W, plain epilogue
hipError_t gemm_dma_special(int tiling, const GemmDmaParams& p, bool head_major, hipStream_t s);   // row-major W, residual or head-major store

}  // namespace ago
