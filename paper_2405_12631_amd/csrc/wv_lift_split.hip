// One predict/update filter application of the synthesis transform (Sec. 3.1), 32 channels, of a model
// made with WV_LIFT_SPLIT (every synthesis of it; the FP32 forms are lift_fused_k and lift_rows_k):
//   out = A + sign * f,  f = z + N(z) (predict) or z/2 + N(z) (update),
//   N = conv3x3(32 -> 1) . tanh . conv3x3(32 -> 32) . tanh . conv3x3(1 -> 32),
// every conv zero-padded at the array border, with all three convs on the 16-bit matrix units
// at no less than FP32 accuracy: each FP32 operand is split into 16-bit parts whose products are
// exact in the FP32 accumulator, and the products that matter are all taken (three BF16 parts: Henry,
// Tang, Heinecke, ARITH 2019; two FP16 parts with power-of-two scaling: Ootomo, Yokota, IJHPCA 2022).
//   layer 1: z and w as three BF16 parts each (24 bits, the FP32 range); 8 of the 9 products, one
//            tap per wave half: 5 MFMAs for 9 taps;
//   layer 2: the tanh outputs (in [-1, 1], scaled by 2^10) and the weights (scaled by a power of
//            two) as two FP16 parts each (22-23 bits); high x high + low x high + high x low: 6
//            MFMAs of K = 16 per tap;
//   layer 3: the same split; the MFMA's rows are the nine taps (T[tap][position]), and an output
//            is the sum of nine of them.
// Error against 64 bits over a 512 x 768 and a 1088 x 1920 synthesis: 3.48e-8 and 4.30e-8 of the
// norm, the same as with the FP32 matrix units (lift_fused_k, lift_rows_k), and at most 0.6 % above
// theirs for filters of other scales (tests/test_gpu_lift_accuracy.py).
//
// What bounds it.  Per 32 positions 63 v_mfma_f32_32x32x16 (32 cycles each) against 578 FP32
// MFMA-equivalents before, and about 240 vector instructions, 64 of them exponentials and
// reciprocals.  A wave issues about one instruction per 5 cycles, so the 32 x 32 form (half the
// instructions of 16 x 16 for the same work) and vector work placed between the MFMAs are what
// counts.  1088 x 1920 x 8 planes: the matrix pipe is busy 71 % of a wave pair's time, at 1.9 GHz
// (the chip lowers its clock: all-zero input runs 12 % faster); synthesis 10.0 -> 2.99 ms, one
// 512 x 768 x 3 image 1.18 -> 0.47 ms (its smaller launches are bound by the pipeline's length).
// Tried and slower: 16 x 16 x 32 MFMAs (3.44 ms; 3.28 with vector work between them), layers 1
// and 2 in separate blocks, low weight parts in registers (spills).
//
// Row streaming: the waves of a strip walk 32 G positions (32 G - 4 output columns) down a
// segment of rows; a wave owns 32 positions in every stage, and the stages of consecutive rows
// are one step apart.  In step t: layer 1 on row y0 - 5 + t; the layer-1 row x = y0 - 6 + t into
// the layer-2 sums of rows x - 1, x, x + 1, which stay in registers, so that a layer-1 value is
// read from LDS once per column tap instead of nine times; tanh and layer 3 of the layer-2 row
// y0 - 8 + t finished in the step before; output row y0 - 10 + t; z row y0 - 3 + t stored.
// A strip of 4 waves (124 of 128 positions used) has one LDS-only barrier per step; a strip of one
// wave (28 of 32) needs none and wastes less of a narrow array (the choice: split_cut).
// The weights' high parts stay in registers for the whole launch, the low parts in LDS.  With
// the weights as the MFMA's first operand a lane ends with 16 channels of one position, which are,
// in that channel order, both the 16-byte LDS records that layer 2 reads and layer 3's operand: no
// shuffles between the layers.
//
// Every output takes the same operations in the same order wherever it lies in a strip or a
// segment, so results do not depend on the launch geometry or on the other planes.
#include "wv_device.h"
#include "wv_internal.h"
#include "wv_pieces.h"
#include "wv_rows.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace wv {
namespace {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int NW = 4;             // waves of a workgroup; G of them share a strip
// Layer 1 takes z clamped to this, so that no product or sum of its split parts overflows (weights are
// at most 2^24): infinite z saturates the tanhs that its weights' signs say, where an FP32 sum of
// opposite infinities is NaN.  (A weight below 1e-28 does not saturate its tanh at the clamp.)
constexpr float ZMAX = 7.9e28f;

template <int G>
struct Strip {
    static constexpr int NP = 32 * G;      // positions of layers 1 and 2 per row; position p is column c0 - 2 + p
    static constexpr int OUTW = NP - 4;    // output columns
    static constexpr int SL = NP + 2;      // slots: z slot s is column c0 - 3 + s, the others' slot s position s - 1
    uint4 zv[4][SL];                       // z as {z0,z0 | z0,z1 | z1,z2 | z1,z2} BF16 parts
    float zf[8][SL];                       // z
    uint4 ah[2][2][SL][2];                 // layer 1, high parts: [row][c][slot][lane half], 8 channels each
    uint4 al[2][2][SL][2];                 // low parts
    float sx[2][4][SL];                    // layer-3 sums by column tap (the fourth row takes unused lanes' writes)
};
template <int G>
struct Smem {
    Strip<G> strip[NW / G];
    uint4 w2l[9][2][64];                   // layer-2 weights, low parts
    uint4 w1[5][64];
    uint4 w3[2][64];
    float b1[32], b2[32];
};

__device__ __forceinline__ floatx16 mfma_f16(uint4 a, uint4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0,
                                                  0);
}
__device__ __forceinline__ floatx16 mfma_bf16w(uint4 a, uint4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf(a), as_bf(b), c, 0, 0, 0);
}
// v - (float)low / high half of hw, in one instruction (exact: hw holds the rounded v).
__device__ __forceinline__ float sub_lo(uint32_t hw, float v) {
    float d;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(d) : "v"(hw), "v"(v));
    return d;
}
__device__ __forceinline__ float sub_hi(uint32_t hw, float v) {
    float d;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(hw), "v"(v));
    return d;
}
// The float `off` bytes after a uniform global address.
template <class P>
__device__ __forceinline__ auto& at(P base, uint32_t off) {
    typedef __attribute__((address_space(1))) char Byte;
    return *(P)((Byte*)base + off);
}
// f(integral constant I) for I = A .. B - 1: a loop whose index is a constant in the body.
template <int A, int B, class F>
__device__ __forceinline__ void static_for(const F& f) {
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        static_for<A + 1, B>(f);
    }
}
// Keeps the instruction that made x where it stands: pure instructions are otherwise free to move
// past the scheduling barriers.  No code.
template <class V>
__device__ __forceinline__ void pin(V& x) {
    asm volatile("" : "+v"(x));
}
__device__ __forceinline__ void keep(const floatx16& acc) { asm volatile("" ::"v"(acc)); }
__device__ __forceinline__ uint32_t pack_h2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){a, b}, halfx2));
}

// A step's LDS writes are visible to the strip's waves in the next step: a workgroup barrier, or
// for a strip of one wave program order alone (a wave's LDS accesses are performed in order).
template <int G>
__device__ __forceinline__ void strip_sync() {
    if constexpr (G == 1) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        lds_barrier();
    }
}

template <int G>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void lift_split_k(
    const LiftSplit L, const LiftIO io0, const LiftIO io1, int N, int h, int w, int nstrips, int nseg, int seg_rows,
    int predict, float sign, unsigned total) {
    static_assert(G == 1 || G == NW, "the barrier is the workgroup's");
    using St = Strip<G>;
    constexpr int NP = St::NP, OUTW = St::OUTW, SL = St::SL;
    __shared__ Smem<G> W;
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    if (tid < 32) {
        W.b1[tid] = gmem(L.b1)[tid];
        W.b2[tid] = gmem(L.b2)[tid];
    }
    // edge slots: read for positions whose results are never used, but kept finite
    const int sub = G == 1 ? wv : 0, wg = G == 1 ? 0 : wv;   // this wave's strip, and its place in it
    St& S = W.strip[sub];
    if (wg == 0 && lane < 16) {
        const int sl = lane & 1 ? SL - 1 : 0;
        S.ah[(lane >> 3) & 1][(lane >> 2) & 1][sl][(lane >> 1) & 1] = make_uint4(0, 0, 0, 0);
        S.al[(lane >> 3) & 1][(lane >> 2) & 1][sl][(lane >> 1) & 1] = make_uint4(0, 0, 0, 0);
        S.sx[(lane >> 3) & 1][(lane >> 1) & 3][sl] = 0.f;
    }
    const uint4* g1 = reinterpret_cast<const uint4*>(L.w1);
    const uint4* g2 = reinterpret_cast<const uint4*>(L.w2);   // high parts, then low parts
    const uint4* g3 = reinterpret_cast<const uint4*>(L.w3);
    for (int i = tid; i < 9 * 2 * 64; i += 64 * NW) (&W.w2l[0][0][0])[i] = ld_g(g2 + 9 * 2 * 64 + i);
    for (int i = tid; i < 5 * 64; i += 64 * NW) (&W.w1[0][0])[i] = ld_g(g1 + i);
    if (tid < 128) (&W.w3[0][0])[tid] = ld_g(g3 + tid);
    uint4 w2h[9][2];
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int c = 0; c < 2; ++c) w2h[tap][c] = ld_g(g2 + (tap * 2 + c) * 64 + lane);
    const float b3 = gmem(L.b3)[0];
    __syncthreads();
    const int p = 32 * wg + (lane & 31);   // this lane's position
    for (unsigned it = blockIdx.x * (NW / G) + sub; it < total; it += gridDim.x * (NW / G)) {
        const int strip = (int)(it % (unsigned)nstrips);
        const unsigned rest = it / (unsigned)nstrips;
        const int seg = (int)(rest % (unsigned)nseg);
        int n = (int)(rest / (unsigned)nseg);
        const bool second = n >= N;
        n -= second ? N : 0;
        const int y0 = seg * seg_rows, R = min(seg_rows, h - y0), c0 = strip * OUTW;
        const auto zp = gmem(second ? io1.z.p : io0.z.p) + (long long)n * (second ? io1.z.ps : io0.z.ps);
        const auto ap = gmem(second ? io1.A.p : io0.A.p) + (long long)n * (second ? io1.A.ps : io0.A.ps);
        const auto op = gmem(second ? io1.out.p : io0.out.p) + (long long)n * (second ? io1.out.ps : io0.out.ps);
        const int zrs = second ? io1.z.rs : io0.z.rs, zcs = second ? io1.z.cs : io0.z.cs;
        const int ars = second ? io1.A.rs : io0.A.rs, acs = second ? io1.A.cs : io0.A.cs;
        const int ors = second ? io1.out.rs : io0.out.rs, ocs = second ? io1.out.cs : io0.out.cs;
        // z slot loaded by this lane: its own position's (both wave halves; the same value), and the
        // strip's last two slots by two lanes of its first wave
        const int zs = wg == 0 && (lane == 32 || lane == 33) ? NP + lane - 32 : p;
        const int zc = c0 - 3 + zs;
        const bool zcol = zc >= 0 && zc < w;
        const uint32_t zo = 4u * (uint32_t)(min(max(zc, 0), w - 1) * zcs);   // byte offsets within a row
        const int pc = c0 - 2 + p;                       // this position's column
        const bool inc = pc >= 0 && pc < w;
        const uint32_t ao = 4u * (uint32_t)(min(max(pc, 0), w - 1) * acs);
        const uint32_t oo = 4u * (uint32_t)(max(pc, 0) * ocs);
        const bool live = c0 - 2 + 32 * wg < w;          // the wave has a position inside the array
        const bool owner = half == 0 && inc && p >= 2 && p < NP - 2;
        // unconditional loads from clamped rows and columns; what lies outside is zeroed after
        auto row = [&](int r) { return (long long)min(max(r, 0), h - 1); };
        auto zat = [&](int r) { return at(zp + row(r) * zrs, zo); };
        auto zput = [&](int r, float z) {
            z = zcol && r >= 0 && r < h ? z : 0.f;
            S.zf[r & 7][zs] = z;
            const float zc1 = z == z ? fminf(fmaxf(z, -ZMAX), ZMAX) : z;
            const uint32_t z0 = f2bf(zc1);
            const float e1 = zc1 - __builtin_bit_cast(float, z0 << 16);
            const uint32_t z1 = f2bf(e1);
            const uint32_t z2 = f2bf(e1 - __builtin_bit_cast(float, z1 << 16));
            const uint32_t q = z1 | (z2 << 16);
            S.zv[r & 3][zs] = make_uint4(z0 | (z0 << 16), z0 | (z1 << 16), q, q);
        };
        // The first three z rows together, before the steps.
        const float zi[3] = {zat(y0 - 3), zat(y0 - 2), zat(y0 - 1)};
        float zn = zat(y0), an = 0.f, pend = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) zput(y0 - 3 + k, zi[k]);
        strip_sync<G>();
        // Layer-2 sums: A0 the row finished in the previous step, A1 and A2 the next two rows'.
        floatx16 A0, A1, A2;
#pragma unroll
        for (int i = 0; i < 16; ++i) A0[i] = A1[i] = A2[i] = 0.f;
        float ua0 = 0.f, ua1 = 0.f, ub0 = 0.f, ub1 = 0.f;   // layer-3 sums of the next two output rows
        auto step = [&](int t, auto on) {   // on: layers 1 and 2 run
            if (t >= 11 && owner) at(op + (long long)(y0 - 11 + t) * ors, oo) = pend;
            // z row y0 - 3 + t, loaded in the previous step; then the next step's z and A
            auto turn = [&](float s, float zz) {
                const float zcur = zn, acur = an;
                zn = zat(y0 - 2 + t);
                an = at(ap + row(y0 - 9 + t) * ars, ao);
                zput(y0 - 3 + t, zcur);
                pend = acur + sign * ((predict ? zz : 0.5f * zz) + fmaf(s, L.s3, b3));
            };
            const int r1 = y0 - 5 + t;   // layer-1 row
            const int x = r1 - 1;        // layer-1 row that layer 2 takes
            const int r2 = x - 2;        // layer-2 row finished in the previous step
            if (!live) {
                turn(0.f, 0.f);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    S.ah[r1 & 1][c][1 + p][half] = make_uint4(0, 0, 0, 0);
                    S.al[r1 & 1][c][1 + p][half] = make_uint4(0, 0, 0, 0);
                }
                S.sx[r2 & 1][half][1 + p] = 0.f;
                S.sx[r2 & 1][2 + half][1 + p] = 0.f;
            } else {
                // One straight block: 63 MFMAs with the vector work of the finished layer-2 row and of
                // layer 1 between them.  Steps outside a stage's rows compute values that no needed row
                // takes; the last two steps have neither layer 1 nor layer 2 (`on`).
                const int r = y0 - 10 + t;   // output row, from the layer-3 sums of the previous step
                const float(*Sr)[SL] = S.sx[(r2 - 1) & 1];
                float s0 = Sr[0][p], s1 = Sr[1][p + 1], s2 = Sr[2][p + 2];
                const float zz = S.zf[r & 7][p + 1];
                uint4 fh[2], fl[2], wl[3], zf1[2], wf1[2], w3f[2], hi[2], lo[2];
                auto load_hi = [&](int dx) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) fh[c] = S.ah[x & 1][c][p + dx][half];
                };
                auto load_lo = [&](int dx) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) fl[c] = S.al[x & 1][c][p + dx][half];
                };
                // operands of layer 1's MFMA q: tap 2 q + half (tap 9: zero weights, reads tap 8)
                const uint4 *zm = S.zv[(r1 - 1) & 3], *z0 = S.zv[r1 & 3], *zq = S.zv[(r1 + 1) & 3];
                auto load_1 = [&](auto q) {
                    if constexpr (q == 0) zf1[0] = zm[p + half];
                    if constexpr (q == 1) zf1[1] = *(half ? z0 + p : zm + p + 2);
                    if constexpr (q == 2) zf1[0] = z0[p + half + 1];
                    if constexpr (q == 3) zf1[1] = zq[p + half];
                    if constexpr (q == 4) zf1[0] = zq[p + 2];
                    wf1[q % 2] = W.w1[q][lane];
                };
                floatx16 a1, tt;
                float v[16], bb[16];
                auto load_b2 = [&](int q) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) bb[4 * q + i] = W.b2[8 * q + 4 * half + i];
                };
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) a1[4 * q + i] = W.b1[8 * q + 4 * half + i];
                load_b2(0);
                load_b2(1);
                load_1(std::integral_constant<int, 0>{});
                load_1(std::integral_constant<int, 1>{});
                const bool ok2 = inc && r2 >= 0 && r2 < h, ok1 = inc && r1 >= 0 && r1 < h;
                const float kb2 = ok2 ? 1024.f : 0.f, ka2 = -2.f * kb2;   // zeros outside the array
                const float kb1 = ok1 ? 1024.f : 0.f, ka1 = -2.f * kb1;
                uint32_t hw[8], lw[8];
                // Vector work in units: 0 .. 79 the finished layer-2 row (A0 -> hi, lo), 80 .. 159 layer 1.
                // tanh x = 1 - 2 / (1 + e^{2x}) times 2^10; the sums are 2 x log2 e.
                auto unit = [&](auto unit_k) {
                    constexpr bool l1 = unit_k >= 80;
                    constexpr int u = unit_k % 80;
                    if constexpr (u < 16) {
                        v[u] = __builtin_amdgcn_exp2f(l1 ? a1[u] : fmaf(A0[u], L.s2, bb[u]));
                        pin(v[u]);
                    } else if constexpr (u < 32) {
                        v[u - 16] = __builtin_amdgcn_rcpf(1.f + v[u - 16]);
                        pin(v[u - 16]);
                    } else if constexpr (u < 48) {
                        v[u - 32] = fmaf(l1 ? ka1 : ka2, v[u - 32], l1 ? kb1 : kb2);
                        pin(v[u - 32]);
                    } else if constexpr (u < 56) {
                        hw[u - 48] = pack_h2(v[2 * (u - 48)], v[2 * (u - 48) + 1]);
                        pin(hw[u - 48]);
                    } else if constexpr (u < 72) {
                        v[u - 56] = (u & 1) ? sub_hi(hw[(u - 56) >> 1], v[u - 56]) : sub_lo(hw[(u - 56) >> 1], v[u - 56]);
                        pin(v[u - 56]);
                    } else {
                        lw[u - 72] = pack_h2(v[2 * (u - 72)], v[2 * (u - 72) + 1]);
                        pin(lw[u - 72]);
                    }
                };
                static_for<0, 59>([&](auto slot) {
                    constexpr int sl = slot;
                    // operands are read from LDS several slots before their MFMAs
                    if constexpr (sl == 1 || sl == 2) load_b2(sl + 1);
                    if constexpr (on && sl == 3) load_hi(0);
                    if constexpr (on && sl >= 5) {
                        constexpr int i = sl - 5, dx = i / 18, j = i % 18;
                        if constexpr (j < 3 || (j >= 6 && j < 9)) wl[j % 3] = W.w2l[3 * (2 - j % 3) + dx][j / 6][lane];
                        if constexpr (j == 5) load_lo(dx);
                        if constexpr (j == 13 && dx < 2) load_hi(dx + 1);
                    }
                    if constexpr (sl == 27) {
                        w3f[0] = W.w3[0][lane];
                        w3f[1] = W.w3[1][lane];
                    }
                    if constexpr (sl < 5) {
                        if constexpr (on) a1 = mfma_bf16w(wf1[sl % 2], zf1[sl % 2], a1);
                        pin(a1);
                        if constexpr (on && sl < 3) load_1(std::integral_constant<int, sl + 2>{});
                    } else if constexpr (on) {
                        constexpr int i = sl - 5, dx = i / 18, j = i % 18, g = j / 3, k = j % 3;
                        // K chunk 0's high x high and low x high, chunk 1's, then both high x low
                        constexpr int pr = g >= 4 ? 2 : g & 1, c = g >= 4 ? g - 4 : g >> 1;
                        constexpr int tap = 3 * (2 - k) + dx;
                        const uint4 wt = pr == 1 ? wl[k] : w2h[tap][c];
                        const uint4 f = pr == 2 ? fl[c] : fh[c];
                        // the first MFMA of each row takes the row's sums over from the previous step
                        const floatx16 zero = {0.f};
                        floatx16& d = k == 0 ? A0 : k == 1 ? A1 : A2;
                        d = mfma_f16(wt, f, i >= 3 ? d : k == 0 ? A1 : k == 1 ? A2 : zero);
                        // (kept alive past it, so that the sum moves in the MFMA and not by copies)
                        if constexpr (i < 2) keep(i == 0 ? A1 : A2);
                        pin(d);
                    }
                    // layer-2 tanh inputs are all read in the first five slots, before A0 is overwritten
                    constexpr int u0 = sl < 5 ? (16 * sl) / 5 : sl < 30 ? 16 + (64 * (sl - 5)) / 25 : 80 + (80 * (sl - 30)) / 29;
                    constexpr int e = sl + 1;
                    constexpr int u1 = e < 5 ? (16 * e) / 5 : e < 30 ? 16 + (64 * (e - 5)) / 25 : 80 + (80 * (e - 30)) / 29;
                    static_for<u0, u1>([&](auto k) {
                        if constexpr (k < 80 || on) unit(k);
                    });
                    if constexpr (sl == 6) s0 = (s0 + s1) + s2;
                    if constexpr (sl == 44) turn(s0, zz);
                    if constexpr (sl == 30) {
                        hi[0] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                        hi[1] = make_uint4(hw[4], hw[5], hw[6], hw[7]);
                        lo[0] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
                        lo[1] = make_uint4(lw[4], lw[5], lw[6], lw[7]);
                        const floatx16 zero = {0.f};
                        tt = mfma_f16(w3f[0], hi[0], zero);
                    }
                    if constexpr (sl == 31) tt = mfma_f16(w3f[1], hi[1], tt);
                    if constexpr (sl == 32) tt = mfma_f16(w3f[0], lo[0], tt);
                    if constexpr (sl == 33) tt = mfma_f16(w3f[1], lo[1], tt);
                    if constexpr (sl == 38) {   // rows 0-2 (and 16-18: the weights' low parts) of the wave half: a column's taps
                        float* so = &S.sx[r2 & 1][half][1 + p];
                        so[0] = ua0 + (tt[2] + tt[10]);
                        ua0 = ua1 + (tt[1] + tt[9]);
                        ua1 = tt[0] + tt[8];
                        so[2 * SL] = ub0 + (tt[6] + tt[14]);
                        ub0 = ub1 + (tt[5] + tt[13]);
                        ub1 = tt[4] + tt[12];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if (!on) continue;
                    S.ah[r1 & 1][c][1 + p][half] = make_uint4(hw[4 * c], hw[4 * c + 1], hw[4 * c + 2], hw[4 * c + 3]);
                    S.al[r1 & 1][c][1 + p][half] = make_uint4(lw[4 * c], lw[4 * c + 1], lw[4 * c + 2], lw[4 * c + 3]);
                }
            }
            strip_sync<G>();
        };
        for (int t = 3; t <= R + 7; ++t) step(t, std::true_type{});
        step(R + 8, std::false_type{});
        step(R + 9, std::false_type{});
        if (owner) at(op + (long long)(y0 + R - 1) * ors, oo) = pend;
    }
}

template <int G>
int split_resident() {   // resident workgroups, cached per device (256 if unknown: the cut, not the results, depends on it)
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cache[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        int per_cu = 0, cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, lift_split_k<G>, 64 * NW, 0) != hipSuccess ||
            per_cu < 1)
            return 256;
        n = per_cu * cus;
        cache[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// How a launch is cut: strips of G waves, segments of seg_rows rows.  An item pays about 6 steps of
// pipeline fill, a launch takes as many rounds of the resident strips as its items need, and a step
// is about a quarter shorter where a wave has its SIMD to itself: the segment length with the least.
struct Cut {
    int nstrips, seg_rows, nseg, grid;
    long long total, cost;
};
template <int G>
Cut split_cut(int h, int w, long long planes) {
    Cut c{};
    const long long slots = (long long)split_resident<G>() * (NW / G);
    c.nstrips = (w + Strip<G>::OUTW - 1) / Strip<G>::OUTW;
    const long long cols = c.nstrips * planes;
    each_segment_rows(h, [&](int r) {
        const long long items = cols * ((h + r - 1) / r);
        const long long cost = (items + slots - 1) / slots * (r + 6) * (2 * items <= slots ? 3 : 4);
        if (c.cost == 0 || cost < c.cost) {
            c.cost = cost;
            c.seg_rows = r;
        }
    });
    c.nseg = (h + c.seg_rows - 1) / c.seg_rows;
    c.total = cols * c.nseg;
    c.grid = (int)((std::min(c.total, slots) + NW / G - 1) / (NW / G));
    return c;
}

}  // namespace

hipError_t launch_lift_split(const LiftSplit& L, const LiftIO& io0, const LiftIO& io1, int sets, int N, int h, int w,
                             int predict, float sign, hipStream_t s) {
    if ((long long)N * h * w == 0) return hipSuccess;
    if (sets < 1 || sets > 2) return hipErrorInvalidValue;
    const Cut c1 = split_cut<1>(h, w, (long long)N * sets), c4 = split_cut<NW>(h, w, (long long)N * sets);
    if (c1.total >= 1ll << 31 || c4.total >= 1ll << 31) return hipErrorInvalidValue;
    if (c1.cost < c4.cost)
        hipLaunchKernelGGL(lift_split_k<1>, dim3(c1.grid), dim3(64 * NW), 0, s, L, io0, io1, N, h, w, c1.nstrips,
                           c1.nseg, c1.seg_rows, predict, sign, (unsigned)c1.total);
    else
        hipLaunchKernelGGL(lift_split_k<NW>, dim3(c4.grid), dim3(64 * NW), 0, s, L, io0, io1, N, h, w, c4.nstrips,
                           c4.nseg, c4.seg_rows, predict, sign, (unsigned)c4.total);
    return hipGetLastError();
}

}  // namespace wv
