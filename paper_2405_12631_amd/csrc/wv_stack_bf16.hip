// A whole coding-step stack of the context model (Sec. 3.2: the conv stack of one
// (subband type, step) and its mixture head) in one kernel, BF16 operands and
// activations, FP32 accumulation.  Model shape: 64 channels, three conv3x3
// layers with ReLU (the first one also reads the coded symbols of the earlier
// steps when step >= 1) and the head conv.
//
// Why fused: one 64 -> 64 BF16 conv layer does 288 FLOP per byte of activations
// it reads and writes, below the chip's ~312 FLOP/B balance, so a layer-by-layer
// stack is bound by HBM round trips of its intermediate activations.  Here they
// never leave LDS: a workgroup walks a strip of 58 output columns of one plane
// down its rows and keeps, for each layer input, a ring of 4 rows x 66 columns
// (64 BF16 channels per position).  Only the step's input l_i and the symbols
// come from HBM and only the parameters of the step's positions go back.
//
// Work split (8 waves, two per SIMD; wave w runs on SIMD w mod 4).  A row step is 12 units of matrix
// work (3 layers x 4 blocks of 16 output channels, 64 positions each), 3 per SIMD:
//   waves 0-1 layer 0 and waves 2-3 layer 2, two blocks each (pair_run);
//   waves 4-7 layer 1, one block each, with 16 positions of the head, a quarter of ring 0's input rows
//   and of the mixture parameters, and wave 7 the symbol operands (single_run).
// Each wave keeps its blocks' weight fragments in registers for the whole launch (72 VGPRs per block:
// 18 K steps of 32 input channels), so LDS carries only activations.  A row step ends with one LDS-only
// workgroup barrier.  In step t layer l computes row y0 - 3 - 2 l + t (two rows behind layer l - 1), the
// loads bring input row y0 - 1 + t, the head finishes row y0 - 9 + t and the parameters of row
// y0 - 10 + t leave.  Every read of a step therefore sees rows finished in earlier steps, and with
// 4-row rings no slot written in a step is one read in it.
//
// What bounds it: the matrix cores are busy 55 % of the time (3680 of 6700 cycles of a row step, 1.3
// PFLOP/s with the strips' overlap and the head's padding).  The two K loops alone take 4000 cycles; the
// head's chain after layer 1 adds 600, the layers' epilogues 700, mixture and loads 300, and items'
// starts 10 % of the launch.  Twelve images of 512 x 768: 541-554 us per launch with symbols and 541-561
// without, where the split it replaces (layers 1 and 2 whole on SIMDs 2-3, the head on SIMD 0, loads
// through registers on SIMD 1: 4608 cycles of matrix work on the fullest SIMD) took 632 and 666.  What
// made the difference, in turn: the even split 612 / 597; input rows straight into LDS 602 / 592; layer 1
// summing three output rows at once, so that each fragment is read from LDS once and not three times (612
// KB of fragment reads per step were 87 % of the LDS's rate, now 408 KB) 548 / 559.  Slower: 32 x 32 x 16
// products (668), layers 0 and 2 writing a row one step later (565), the head's products inside layer 1's
// loop (585), 12 waves of 16 channels (736).
//
// Bits: every output is accumulated with the same MFMA sequence as the
// layer-by-layer kernel (taps 0..8, 32-channel chunks in order, the symbol
// chunk last; the same fragment layout), then the same bias, ReLU and BF16
// rounding, and the head the same epilogue, so both forms give identical
// parameters.
#include "wv_device.h"
#include "wv_internal.h"
#include "wv_rows.h"

#include <type_traits>

namespace wv {
namespace {

constexpr int SW = 64;             // positions a layer computes per row (4 blocks of 16)
constexpr int SLOTS = SW + 2;      // ring columns; slot k is image column c0 - 4 + k
constexpr int PSTR = 128;          // bytes per slot: 64 BF16 channels in 8 chunks of 16 bytes
constexpr int RROW = SLOTS * PSTR;
constexpr int RING = 4 * RROW;
constexpr int NT = 512;            // threads: 8 waves
constexpr int NCH = 64;            // channels of every layer input
constexpr int CC = NCH / 32;       // K chunks per tap
constexpr int NK = 9 * CC;         // K steps per layer

struct Item {
    int n, y0, R, c0;
};

__device__ __forceinline__ bool next_item(const StackSeg* segs, int nseg, long long it, long long total, int& si,
                                          Item& I) {
    if (it >= total) return false;
    int lo = 0, hi = nseg;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (segs[mid].item0 <= it) lo = mid; else hi = mid;
    }
    si = lo;
    const StackSeg& S = segs[lo];
    long long local = it - S.item0;
    const int sx = (int)(local % S.strips_x);
    local /= S.strips_x;
    const int sy = (int)(local % S.segs_y);
    I.n = (int)(local / S.segs_y);
    I.y0 = sy * S.seg_rows;
    I.R = min(S.seg_rows, S.h - I.y0);
    I.c0 = sx * (SW - 6);
    return true;
}

// f(integral constant I) for I = A .. B - 1: a loop whose index is a constant in the body.
template <int A, int B, class F>
__device__ __forceinline__ void static_for(const F& f) {
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        static_for<A + 1, B>(f);
    }
}
// The same value, unknown to the optimiser: what is computed from it in a loop (LDS addresses) is
// recomputed there instead of being kept in registers.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

struct Smem {
    uint8_t ring[4][RING];      // inputs of layers 0..2 and the head: row r in slot r & 3
    uint4 rec[2][SW][2];        // symbol operands of layer 0's output row r in slot r & 1: taps 0-7, tap 8
    uint4 wsym[4][64];          // symbol weights of layer 0
    float bias[3][64], hb[16];  // of the layers and the head
    float head_st[SW][17];      // raw head outputs of a row
};

// 16 bytes per active lane from byte voff of the row at `row` (of `bytes` bytes; the buffer's bounds
// check gives zeros outside them) straight into LDS at lds + 16 lane.  The caller waits (wait_vm) before
// the barrier that publishes them; in the builtin's place, the compiler would wait before the next LDS
// read of any kind.  The LDS address is an operand in m0, which the compiler sets and so knows of; the
// s_nop covers the wait states after writes of m0 and of the descriptor.
__device__ __forceinline__ void row_to_lds(const void* row, uint32_t bytes, uint32_t voff, uint32_t lds) {
    typedef int int4v __attribute__((ext_vector_type(4)));
    const uint64_t a = (uint64_t)row;
    const int4v rsrc = {__builtin_amdgcn_readfirstlane((int)a), __builtin_amdgcn_readfirstlane((int)(a >> 32) & 0xffff),
                        __builtin_amdgcn_readfirstlane((int)bytes), 0x00027000};
    asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 ::"{m0}"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(voff), "s"(rsrc)
                 : "memory");
}

// K loop of one row of a layer: positions 0..63 of output row x (slots 1..64) from the input ring's
// rows x - 1, x, x + 1; two column blocks of weights in registers.
__device__ __forceinline__ void pair_mfma(const uint8_t* rin, int x, const uint4 (&wr)[NK][2], floatx4 (&acc)[4][2],
                                          int lane) {
    constexpr int PF = 2;   // K steps read ahead
    const int m = lane & 15;
    const int kk = lane >> 4;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};
    uint4 a[PF + 1][4];
    auto load_a = [&](int st) {
        const int tap = st / CC, cc = st % CC;
        // blocks mb are 16 slots apart, which keeps slot & 7 and so the chunk swizzle
        const uint8_t* p = rin + ((x - 1 + tap / 3) & 3) * RROW + swz(m + tap % 3, cc * 4 + kk);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) a[st % (PF + 1)][mb] = *reinterpret_cast<const uint4*>(p + mb * 16 * PSTR);
    };
#pragma unroll
    for (int i = 0; i < PF; ++i) load_a(i);
    __builtin_amdgcn_sched_group_barrier(0x100, PF * 4, 0);
#pragma unroll
    for (int st = 0; st < NK; ++st) {
        if (st + PF < NK) load_a(st + PF);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = mfma_bf16(wr[st][nb], a[st % (PF + 1)][mb], acc[mb][nb]);
        // Keep the fragment reads ahead of this step's MFMAs: the latency of an LDS read is then
        // covered by PF steps of MFMAs.
        if (st + PF < NK) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
    }
}

// Input row `rin` into the sums of the output rows below (A0, its last taps), at (A1) and above it
// (A2, its first taps) for one column block: each fragment is read once and feeds three MFMAs.
__device__ __forceinline__ void single_mfma(const uint8_t* rin, const uint4 (&wr)[NK], floatx4 (&A0)[4][1],
                                            floatx4 (&A1)[4][1], floatx4 (&A2)[4][1], int lane) {
    constexpr int LA = 4;      // fragments read ahead
    const int m = lane & 15, kk = lane >> 4;
    const floatx4 zero = floatx4{0.f, 0.f, 0.f, 0.f};
    uint4 f[LA + 1];
    auto load = [&](auto gi) {
        constexpr int dx = gi / 4 / CC, cc = gi / 4 % CC, mb = gi % 4;
        f[gi % (LA + 1)] = *reinterpret_cast<const uint4*>(rin + swz(m + dx, cc * 4 + kk) + mb * 16 * PSTR);
    };
    static_for<0, LA>(load);
    static_for<0, 24>([&](auto gi) {
        constexpr int st = gi / 4, mb = gi % 4;   // K step of the first tap row; the others follow at 6, 12
        if constexpr (gi + LA < 24) load(std::integral_constant<int, gi + LA>{});
        const uint4 v = f[gi % (LA + 1)];
        A0[mb][0] = mfma_bf16(wr[12 + st], v, st == 0 ? A1[mb][0] : A0[mb][0]);
        A1[mb][0] = mfma_bf16(wr[6 + st], v, st == 0 ? A2[mb][0] : A1[mb][0]);
        A2[mb][0] = mfma_bf16(wr[st], v, st == 0 ? zero : A2[mb][0]);
        __builtin_amdgcn_sched_barrier(0);
    });
}

// The same for 16 positions of the head, of which every other row is wanted: the middle taps of hacc,
// or with LAST its last taps and the first ones of hnew.
template <bool LAST>
__device__ __forceinline__ void head_mfma(const uint8_t* rin, const uint4 (&wh)[NK], floatx4& hacc, floatx4& hnew, int lane) {
    const int m = lane & 15, kk = lane >> 4;
    uint4 f[6];
#pragma unroll
    for (int st = 0; st < 6; ++st) f[st] = *reinterpret_cast<const uint4*>(rin + swz(m + st / CC, st % CC * 4 + kk));
    if (LAST) hnew = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < 6; ++st) {
        hacc = mfma_bf16(wh[(LAST ? 12 : 6) + st], f[st], hacc);
        if (LAST) hnew = mfma_bf16(wh[st], f[st], hnew);
    }
}

// Bias, ReLU and BF16 of a row into a ring row; positions outside the plane are zero (the next
// layer's padding).  Lane: position p = 16 mb + lane % 16, channels 16 (nb0 + nb) + 4 (lane / 16)
// .. + 3, i.e. 8 bytes of chunk 2 (nb0 + nb) + lane / 32 at byte 8 ((lane / 16) & 1), swizzled by
// slot 1 + p (block mb adds 16 slots: swizzle unchanged).
template <int NBL>
__device__ __forceinline__ void write_row(uint8_t* row, const floatx4 (&acc)[4][NBL], const float* bias, int nb0,
                                          int c0, int w, bool rok, int ln) {
    const int pm = ln & 15, sl = 1 + pm;
    uint8_t* orow = row + sl * PSTR + ((ln >> 4) & 1) * 8;
    floatx4 b[NBL];
#pragma unroll
    for (int nb = 0; nb < NBL; ++nb)
        b[nb] = *reinterpret_cast<const floatx4*>(bias + 16 * (nb0 + nb) + 4 * (ln >> 4));
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
        const int c = c0 - 3 + mb * 16 + pm;
        const bool ok = rok && c >= 0 && c < w;
#pragma unroll
        for (int nb = 0; nb < NBL; ++nb) {
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = fmaxf(acc[mb][nb][k] + b[nb][k], 0.f);
            uint2 u = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
            if (!ok) u = make_uint2(0u, 0u);
            const int chunk = 2 * (nb0 + nb) + (ln >> 5);
            *reinterpret_cast<uint2*>(orow + mb * 16 * PSTR + ((chunk ^ (sl & 7)) << 4)) = u;
        }
    }
}

// Layers 0 and 2: two output blocks from nb0.
template <bool SYM, int L>
__device__ __forceinline__ void pair_run(const StackSeg* __restrict__ segs, int nseg, long long total, int nb0,
                                         Smem& M) {
    const int lane = lane_id();
    uint4 wr[NK][2];
    const uint16_t* wcur = nullptr;
    long long it = blockIdx.x;
    int si;
    Item I;
    while (next_item(segs, nseg, it, total, si, I)) {
        const StackSeg& S = segs[si];
        if (S.w16[L] != wcur) {   // every item of a launch uses one step's weights
            wcur = S.w16[L];
            const uint4* wg = reinterpret_cast<const uint4*>(wcur);
#pragma unroll
            for (int st = 0; st < NK; ++st)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) wr[st][nb] = ld_g(wg + (st * 4 + nb0 + nb) * 64 + lane);
            // read by this wave alone, after the barrier below
            if (lane < 32) M.bias[L][16 * nb0 + lane] = gmem(S.bias[L])[16 * nb0 + lane];
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                if (SYM && L == 0)
                    M.wsym[nb0 + nb][lane] = ld_g(reinterpret_cast<const uint4*>(S.wsym) + (nb0 + nb) * 64 + lane);
        }
        wait_vm();
        lds_barrier();
        const int T = I.R + 10;
        for (int t = 0; t < T; ++t) {
            const int x = I.y0 - 3 - 2 * L + t;
            if (t >= 3 * L && t <= I.R + 5 + L) {
                floatx4 acc[4][2];
                const bool rok = x >= 0 && x < S.h;
                if (rok) {
                    pair_mfma(M.ring[L], x, wr, acc, lane);
                    if (SYM && L == 0) {   // the symbol chunk comes after the taps; lane groups 2, 3 hold zeros
                        const int ln = opaque(lane), kk = ln >> 4;
                        const uint4 ws[2] = {M.wsym[nb0][ln], M.wsym[nb0 + 1][ln]};
#pragma unroll
                        for (int mb = 0; mb < 4; ++mb) {
                            uint4 e = M.rec[x & 1][16 * mb + (ln & 15)][kk & 1];
                            if (kk > 1) e = make_uint4(0, 0, 0, 0);
#pragma unroll
                            for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = mfma_bf16(ws[nb], e, acc[mb][nb]);
                        }
                    }
                }
                write_row<2>(M.ring[L + 1] + (x & 3) * RROW, acc, M.bias[L], nb0, I.c0, S.w, rok, opaque(lane));
            }
            lds_barrier();
        }
        it += gridDim.x;
    }
}

// Layer 1's output block hw, the head of positions 16 hw .. + 15, the input rows, symbol operands and
// mixture parameters.
template <bool SYM>
__device__ __forceinline__ void single_run(const StackSeg* __restrict__ segs, int nseg, long long total, int hw,
                                           Smem& M) {
    const int lane = lane_id();
    uint4 wr[NK], wh[NK];
    const floatx4 zero = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 A0[4][1], A1[4][1], A2[4][1], hacc = zero, hnew = zero;   // sums of this step's rows, see single_mfma
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) A0[mb][0] = A1[mb][0] = A2[mb][0] = zero;
    const uint16_t* wcur = nullptr;
    long long it = blockIdx.x;
    int si;
    Item I;
    while (next_item(segs, nseg, it, total, si, I)) {
        const StackSeg& S = segs[si];
        if (S.w16[1] != wcur) {
            wcur = S.w16[1];
#pragma unroll
            for (int st = 0; st < NK; ++st) {
                wr[st] = ld_g(reinterpret_cast<const uint4*>(wcur) + (st * 4 + hw) * 64 + lane);
                wh[st] = ld_g(reinterpret_cast<const uint4*>(S.w16[3]) + st * 64 + lane);
            }
            if (lane < 16) M.bias[1][16 * hw + lane] = gmem(S.bias[1])[16 * hw + lane];
            if (hw == 0 && lane < 16) M.hb[lane] = gmem(S.bias[3])[lane];
        }
        // ---- rows of ring 0: slots 8 q .. + 7 by wave q mod 4, straight into LDS (lane: slot
        // 8 q + lane / 8, and the chunk that the swizzle puts at place lane % 8) ----
        const uint16_t* in = S.in16 + (long long)I.n * S.in_ps;
        const uint32_t voff = (uint32_t)((I.c0 - 4 + 8 * hw + (lane >> 3)) * PSTR + ((lane & 7) ^ (lane >> 3)) * 16);
        const uint32_t ring0 = (uint32_t)(uint64_t)(__attribute__((address_space(3))) uint8_t*)&M.ring[0][0];
        auto fetch = [&](int row) {
            const bool rok = row >= 0 && row < S.h;
            const void* src = in + (long long)(rok ? row : 0) * S.w * NCH;
            const uint32_t bytes = rok ? (uint32_t)S.w * PSTR : 0u;
            const uint32_t dst = ring0 + (row & 3) * RROW + 1024 * hw;
            row_to_lds(src, bytes, voff, dst);
            row_to_lds(src, bytes, voff + 32 * PSTR, dst + 4096);
            if (hw == 0 && lane < 16) row_to_lds(src, bytes, voff + 64 * PSTR, dst + 8192);
        };
        // ---- symbol operands, by the last wave, one lane per position ----
        const auto sp = gmem(SYM ? S.sym + (long long)I.n * S.sym_ps : reinterpret_cast<const int16_t*>(S.in16));
        int16_t sv[3] = {0, 0, 0};
        auto sym_load = [&](int row) {
            const auto rp = sp + (long long)min(max(row, 0), S.h - 1) * S.w;
#pragma unroll
            for (int d = 0; d < 3; ++d) sv[d] = rp[(uint32_t)min(max(I.c0 - 4 + lane + d, 0), S.w - 1)];
        };
        auto sym_step = [&](int row) {   // the loaded symbols of row `row` complete the record of row - 1
            const int ln = opaque(lane);
            uint32_t e[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int c = I.c0 - 4 + ln + d;
                const bool ok = row >= 0 && row < S.h && c >= 0 && c < S.w && (2 * (row & 1) + (c & 1)) < S.step;
                e[d] = f2bf(ok ? (float)sv[d] : 0.f);
            }
            // the two older rows come from the record before, one row up
            const uint4 o = M.rec[row & 1][ln][0];
            const uint32_t o8 = M.rec[row & 1][ln][1].x;
            M.rec[(row - 1) & 1][ln][0] = make_uint4((o.y >> 16) | (o.z << 16), (o.z >> 16) | (o.w << 16),
                                                     (o.w >> 16) | (o8 << 16), e[0] | (e[1] << 16));
            M.rec[(row - 1) & 1][ln][1].x = e[2];
        };
        for (int r = I.y0 - 4; r <= I.y0 - 2; ++r) fetch(r);
        if (SYM && hw == 3) {
            for (int r = I.y0 - 4; r <= I.y0 - 2; ++r) {
                sym_load(r);
                sym_step(r);
            }
            sym_load(I.y0 - 1);
        }
        wait_vm();
        lds_barrier();
        const int gr = S.step >> 1, gc = S.step & 1;
        const int T = I.R + 10;
        for (int t = 0; t < T; ++t) {
            // symbols first: a wait for them behind the fetch would wait for the fetch too
            if (SYM && hw == 3) {
                if (t <= I.R + 4) sym_step(I.y0 - 1 + t);
                if (t <= I.R + 3) sym_load(I.y0 + t);
            }
            if (t <= I.R + 4) fetch(I.y0 - 1 + t);
            // ---- mixture parameters of the head row finished in the previous step, one lane per
            // (position of this coding step, component): two of the four waves ----
            const int xm = I.y0 - 10 + t;
            if (xm >= I.y0 && (xm & 1) == gr && ((xm >> 1) & 1) == (hw & 1)) {
                const int ln = opaque(lane), K = S.K;
                const int p0 = 3 + ((I.c0 ^ gc) & 1);
                const int np = (min(SW - 3 - p0, S.w - (I.c0 - 3 + p0)) + 1) >> 1;   // at most 29
                const int wg2 = (S.w - gc + 1) >> 1, hg = (S.h - gr + 1) >> 1;
                float* o = S.params + (((long long)I.n * hg + (xm >> 1)) * wg2 + ((I.c0 - 3 + p0) >> 1)) * 3 * K;
                const int q = ln & 31, k = 2 * (hw >> 1) + (ln >> 5);
                if (q < np && k < K)
                    mixture_head_part(&M.head_st[p0 + 2 * q][0], K, k, S.sigma_min, gmem(o + q * 3 * K));
            }
            // ---- layer 1: input row x + 1 finishes output row x; the head: input row xh + 1 finishes
            // row xh, or is the middle one of row xh + 1 ----
            const int x = I.y0 - 5 + t, xh = I.y0 - 9 + t;
            const int ln = opaque(lane);
            const uint8_t* rin = M.ring[1] + ((x + 1) & 3) * RROW;
            const uint8_t* rhd = M.ring[3] + ((xh + 1) & 3) * RROW + hw * 16 * PSTR;
            if (t >= 1 && t <= I.R + 6) single_mfma(rin, wr, A0, A1, A2, ln);
            if (t >= 3 && t <= I.R + 6)
                write_row<1>(M.ring[2] + (x & 3) * RROW, A0, M.bias[1], hw, I.c0, S.w, x >= 0 && x < S.h, ln);
            if (t >= 7 && t <= I.R + 8) {
                if ((xh & 1) == gr) {
                    const floatx4 hbias = *reinterpret_cast<const floatx4*>(M.hb + 4 * (ln >> 4));
                    head_mfma<true>(rhd, wh, hacc, hnew, ln);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        M.head_st[16 * hw + (ln & 15)][4 * (ln >> 4) + k] = hacc[k] + hbias[k];
                    hacc = hnew;
                } else {
                    head_mfma<false>(rhd, wh, hacc, hnew, ln);
                }
            }
            wait_vm();   // the fetched row
            lds_barrier();
        }
        it += gridDim.x;
    }
}

template <bool SYM>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void stack_bf16_k(
    const StackSeg* __restrict__ segs, int nseg, long long total) {
    __shared__ __attribute__((aligned(16))) Smem M;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: role values in scalar registers
    // Ring edge slots 0 and 65 of the layer outputs are never written; they feed only outputs outside
    // the strip's kept columns, but keep them finite.  The symbol records' unused elements stay zero.
    for (int k = tid; k < 16 * 2 * (PSTR / 4); k += NT) {
        const int e = k % (2 * (PSTR / 4)), r = k / (2 * (PSTR / 4));
        const int slot = e < PSTR / 4 ? 0 : SLOTS - 1;
        reinterpret_cast<uint32_t*>(M.ring[0] + r * RROW + slot * PSTR)[e % (PSTR / 4)] = 0u;   // rings are contiguous
    }
    for (int k = tid; k < 2 * SW * 2; k += NT) (&M.rec[0][0][0])[k] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    switch (wave) {   // wave w runs on SIMD w mod 4 (see the work split above)
        case 0:
        case 1: pair_run<SYM, 0>(segs, nseg, total, 2 * wave, M); break;
        case 2:
        case 3: pair_run<SYM, 2>(segs, nseg, total, 2 * (wave - 2), M); break;
        default: single_run<SYM>(segs, nseg, total, wave - 4, M); break;
    }
}

}  // namespace

hipError_t launch_stack_bf16(const StackSeg* segs, int nseg, long long total, int has_sym, int grid,
                             hipStream_t s) {
    if (total <= 0 || nseg <= 0) return hipSuccess;
    if (grid < 1) grid = 1;
    if (has_sym)
        hipLaunchKernelGGL(stack_bf16_k<true>, dim3(grid), dim3(NT), 0, s, segs, nseg, total);
    else
        hipLaunchKernelGGL(stack_bf16_k<false>, dim3(grid), dim3(NT), 0, s, segs, nseg, total);
    return hipGetLastError();
}

}  // namespace wv
