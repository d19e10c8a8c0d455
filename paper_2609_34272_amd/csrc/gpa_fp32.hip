// Fused FP32 attention baseline on gfx950: BF16 inputs and outputs, every
// product and accumulation in FP32 (appendix "Comparison Methods", "Fused
// FP32 baseline").  The forward saves FP32 O and three FP32 row statistics --
// the LSE, the row maximum and the inverse normaliser -- and the backward
// rebuilds P = exp(s - rowmax) * (1/l) from the last two, which keeps the
// normalisation exact to FP32 where large logits leave the LSE short of
// resolution.  No N x N matrix is stored.
//
// The paper's kernel is SIMT FP32 because the Hopper tensor cores round FP32
// operands to TF32.  Here the contractions run on the bf16 matrix cores without
// rounding an operand: Q K^T and dO V^T multiply BF16 inputs, whose products are
// exact in FP32, and the FP32 factors P and dS enter as three BF16 parts that
// add up to them exactly (split3), so P V, P^T dO, dS K and dS^T Q are three
// exact products into the same FP32 accumulator.  The softmax, its statistics
// and the score gradient run on the vector ALU in FP32.  Against FP64 the errors
// are those of the FP32 matrix cores (v_mfma_f32_16x16x4_f32: FP32 operands)
// or smaller, because a 32-wide product rounds the accumulator once where the
// 4-wide FP32 one rounds it eight times: FP32 output 1.7e-7 to 1.3e-5 (2.6e-7 to
// 1.5e-5) relative over N = 77 to 5000, d = 64 and 128, causal and not, key
// bias 0 to 64; LSE 3.0e-8 to 4.3e-8 (3.1e-8 to 4.9e-8).  What bounds the
// kernels now is the vector ALU (the split is 5.5 instructions per pair and FP32
// factor, of 11 to 20): forward / query pass / key pass 369 / 537 / 659 us on the
// FP32 matrix cores, 80 / 91 / 135 us here (16 heads of 4096 causal tokens, d =
// 64; 1552 and 306 us in all).
//
// MFMA layouts as in the BF16 kernels (16x16x32, wave64): lane (c16 = lane & 15,
// g = lane >> 4) supplies 8 values along k of row (A) or column (B) c16; the
// accumulator holds D[4g + i][c16].  The accumulator of S^T = K Q^T (or S = Q
// K^T) leaves each lane the values of rows 4g + i of its column, which is the
// k-layout the LDS transpose read delivers from a row-major BF16 tile, so P and
// dS never pass through LDS.
//
// Work split: a workgroup has 4 waves and owns 64 rows (queries in the
// forward and the query-major pass, keys in the key-major pass), 16 per wave;
// it streams 64-row tiles of the other side through a double-buffered LDS
// ring filled with the LDS DMA load.  At d = 64 a unit holds 5 workgroups of the
// forward, 4 of the query pass and 3 of the key pass, and those rounds are dealt out
// in snake order (map_block): without and with it, 92 / 101 / 143 us and 80 / 91 /
// 135 us (16 heads of 4096), 82 / 77 / 115 and 66 / 55 / 83 (5 of 4160); no
// difference at d = 128.
#include "gpa_device.h"
#include "gpa_launch.h"

#include <type_traits>

namespace gpa {
namespace {

// Per query tile, the key-major pass reads three 64-float blocks: the scaled
// row maximum (+inf beyond N, so P = 0 there), the inverse normaliser (0
// beyond N) and D = rowsum(dO O32) (0 beyond N).
constexpr int kF32Stat = 3 * kTile;

// A row of a [N, D] BF16 tensor as an MFMA operand along d (zero beyond N
// through the buffer resource): chunk kc holds columns 32 kc + 8 g .. + 7.
template <int D>
__device__ __forceinline__ void ld_row_chunks(rsrc_t r, int row, int g, bf16x8 (&out)[D / 32]) {
#pragma unroll
    for (int kc = 0; kc < D / 32; ++kc)
        out[kc] = __builtin_bit_cast(bf16x8, ld_row16<D>(r, row, 32 * kc + 8 * g));
}

// One 16 x 16 block X_rows . Y^T over d: the A side comes from a swizzled LDS
// tile (rows r0 + c16), the B side from registers.  Both are BF16 inputs, so
// every product is exact.
template <int D>
__device__ __forceinline__ f32x4 block_dot(const uint16_t* X, int r0, const bf16x8 (&y)[D / 32],
                                           int c16, int g) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < D / 32; ++kc)
        acc = mfma_16x16x32(ld_b128(X + tile_off<D>(r0 + c16, 32 * kc + 8 * g)), y[kc], acc);
    return acc;
}

// The three BF16 parts of 8 FP32 values, x = hi + mid + lo exactly (24 bits of
// significand in three times 8): each part is the upper half of what the parts
// before it leave, which an FP32 subtraction gives exactly.  Five vector
// instructions per value and a half.  A value that is not finite gives a mid part
// that is a NaN; EXACT_INF gives it as its hi part alone.
struct Split {
    bf16x8 hi, mid, lo;
};
__device__ __forceinline__ bool is_finite(float x) {
    return (__float_as_uint(x) & 0x7F800000u) != 0x7F800000u;
}
__device__ __forceinline__ float upper(float x) {
    return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
}
__device__ __forceinline__ uint32_t uppers(float a, float b) {  // b's upper half above a's
    return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}
template <bool EXACT_INF>
__device__ __forceinline__ Split split3(const f32x4& x0, const f32x4& x1) {
    u32x4 h, m, l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float r[2], q[2];
        const float x[2] = {j < 2 ? x0[2 * j] : x1[2 * j - 4], j < 2 ? x0[2 * j + 1] : x1[2 * j - 3]};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            r[e] = x[e] - upper(x[e]);
            if (EXACT_INF && !is_finite(x[e])) r[e] = 0.f;
            q[e] = r[e] - upper(r[e]);
        }
        h[j] = uppers(x[0], x[1]);
        m[j] = uppers(r[0], r[1]);
        l[j] = uppers(q[0], q[1]);
    }
    return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

// acc[mb] += X^T[d][rows] . B[rows][col] for the 64 tile rows, where the FP32
// values b[kb][i] belong to row 16 kb + 4 g + i and X is a row-major swizzled
// BF16 tile: the transpose read gives lane (c16, g) X[32 kb2 + 4 g + r][16 mb +
// c16] and X[32 kb2 + 16 + 4 g + r][...] for r = 0..3.
//
// A factor whose mid or lo part is 0 turns an infinity of X into a NaN, and so does
// an infinite factor.  A wave that ends with a NaN in its accumulators therefore
// forms them again with EXACT_INF: values of X that are not finite then meet the hi
// part alone, which has the factor's sign and is 0 where it is, so the products are
// the infinities and NaNs of one FP32 product, and all others what they were.
template <int D, bool EXACT_INF>
__device__ __forceinline__ void tr_accumulate(const uint16_t* X, const f32x4 (&b)[4],
                                              f32x4 (&acc)[D / 16], int c16, int g) {
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2) {
        const Split p = split3<EXACT_INF>(b[2 * kb2], b[2 * kb2 + 1]);
#pragma unroll
        for (int mb = 0; mb < D / 16; ++mb) {
            const bf16x8 t = ld_tr_operand<D>(X, 32 * kb2, 16 * mb, c16, g);
            bf16x8 f = t;
            if constexpr (EXACT_INF)
#pragma unroll
                for (int i = 0; i < 8; ++i) f[i] = is_finite(bf16_to_f32(t[i])) ? t[i] : (__bf16)0.f;
            acc[mb] = mfma_16x16x32(f, p.lo, acc[mb]);
            acc[mb] = mfma_16x16x32(f, p.mid, acc[mb]);
            acc[mb] = mfma_16x16x32(t, p.hi, acc[mb]);
        }
    }
}

// Whether an accumulator of the wave may be a NaN: their sum is one then (and where
// infinities or an overflow meet, for which the second walk is merely superfluous).
template <int MB>
__device__ __forceinline__ float nan_sum(const f32x4 (&acc)[MB]) {
    f32x4 t = acc[0];
#pragma unroll
    for (int mb = 1; mb < MB; ++mb) t += acc[mb];
    return (t[0] + t[1]) + (t[2] + t[3]);
}
__device__ __forceinline__ bool wave_nan(float x) {
    return __builtin_amdgcn_ballot_w64((__float_as_uint(x) & 0x7FFFFFFFu) > 0x7F800000u) != 0;
}

// Stages a tile for one wave alone, which has the LDS tile `dst` to itself: what it
// read there before has arrived, and the tile is there on return.
template <int D>
__device__ __forceinline__ void stage_alone(int lane, const uint16_t* head, uint16_t* dst, int row0,
                                            int N) {
    asm volatile("" : "+v"(lane));  // the offsets are formed here, and kept nowhere
    TileDma<D, 64> dma;
    dma.init(lane, 0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    dma.load(head, dst, row0, N);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// ------------------------------------------------------------------ forward
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 5 : 2) void f32_fwd_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, float* __restrict__ O32, uint16_t* __restrict__ O,
    float* __restrict__ LSE, float* __restrict__ Mrow, float* __restrict__ Linv, int BH, int N,
    int causal, float scale) {
    constexpr int KC = D / 32, MB = D / 16;
    __shared__ __attribute__((aligned(16))) uint16_t KV0[2][kTile * D];
    __shared__ __attribute__((aligned(16))) uint16_t KV1[2][kTile * D];
    const int T = (N + kTile - 1) / kTile;
    int bh, tile;
    map_block(blockIdx.x, BH, T, causal != 0, &bh, &tile, D == 64 ? 5 : 0, true);
    const size_t hoff = (size_t)bh * N * D;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c16 = lane & 15;
    const int q0w = tile * kTile + 16 * wave;
    const int qrow = q0w + c16;

    bf16x8 qf[KC];
    ld_row_chunks<D>(make_rsrc(Q + hoff, (uint32_t)N * (2 * D)), qrow, g, qf);

    const KeyRange kr = key_range(tile, N, 0, causal);
    const int nkv = kr.nkv, nplain = kr.nplain;
    const float lg = kLog2e;
    float mrun = -INFINITY, lrun = 0.f;  // scaled running maximum; this lane's share of l
    f32x4 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    TileDma<D> dma;
    dma.init(lane, wave);
    dma.load(K + hoff, KV0[0], 0, N);
    dma.load(V + hoff, KV0[1], 0, N);
    wait_vm_lgkm0<0>();
    __syncthreads();

    // P of tile kt into s, with the running maximum and sum and the rescaled output
    auto probs = [&](auto masked, int kt, const uint16_t* Kc, f32x4 (&s)[4]) {
        constexpr bool MASK = decltype(masked)::value;
        float tmax = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            s[kb] = block_dot<D>(Kc, 16 * kb, qf, c16, g);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v = scale * s[kb][i];
                if constexpr (MASK) {
                    const int key = kt * kTile + 16 * kb + 4 * g + i;
                    v = (key < N && (!causal || key <= qrow)) ? v : -INFINITY;
                }
                s[kb][i] = v;
                tmax = fmaxf(tmax, v);
            }
        }
        const float mnew = fmaxf(mrun, xor_max(tmax));
        // a row that has seen no key yet keeps m = -inf; its factors are 1, 0
        const float corr = mnew == -INFINITY ? 1.f : fexp2((mrun - mnew) * lg);
        const float msub = mnew == -INFINITY ? 0.f : mnew;
        mrun = mnew;
        float lsum = 0.f;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float p = fexp2((s[kb][i] - msub) * lg);
                s[kb][i] = p;
                lsum += p;
            }
        lrun = lrun * corr + lsum;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] *= corr;
    };
    auto step = [&](auto masked, int kt, const uint16_t* Kc, const uint16_t* Vc, uint16_t* Kn,
                    uint16_t* Vn) {
        if (kt + 1 < nkv) {
            dma.load(K + hoff, Kn, (kt + 1) * kTile, N);
            dma.load(V + hoff, Vn, (kt + 1) * kTile, N);
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x4 s[4];
        probs(masked, kt, Kc, s);
        tr_accumulate<D, false>(Vc, s, acc, c16, g);
        wait_vm_lgkm0<0>();
        __syncthreads();
    };
    const std::false_type plain;
    const std::true_type masked;
    // Two steps a turn, each with its buffers: the accumulators then stay where they
    // are over the loop's edge, and no copy of them can come too early (mfma_settle).
    int kt = 0;
    for (; kt + 1 < nplain; kt += 2) {
        step(plain, kt, KV0[0], KV0[1], KV1[0], KV1[1]);
        step(plain, kt + 1, KV1[0], KV1[1], KV0[0], KV0[1]);
    }
    if (kt < nplain) {
        step(plain, kt, KV0[0], KV0[1], KV1[0], KV1[1]);
        ++kt;
    }
    // Tile kt lives in buffer kt mod 2.
    // At most one tile needs masks: the diagonal one, or the key tail.
    if (kt < nkv) {
        if (kt & 1) step(masked, kt, KV1[0], KV1[1], KV0[0], KV0[1]);
        else step(masked, kt, KV0[0], KV0[1], KV1[0], KV1[1]);
    }
    mfma_settle();
    if (__builtin_expect(wave_nan(nan_sum(acc)), 0)) {
        // again with EXACT_INF, this wave alone: each wave has one of the four tiles
        uint16_t* buf = wave < 2 ? KV0[wave] : KV1[wave - 2];
        mrun = -INFINITY;
        lrun = 0.f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int t = 0; t < nkv; ++t) {
            f32x4 s[4];
            stage_alone<D>(lane, K + hoff, buf, t * kTile, N);
            probs(masked, t, buf, s);
            stage_alone<D>(lane, V + hoff, buf, t * kTile, N);
            tr_accumulate<D, true>(buf, s, acc, c16, g);
            mfma_settle();
        }
    }

    const float l = xor_sum(lrun);
    if (qrow < N) {
        const float inv = 1.f / l;
        float* orow = O32 + hoff + (size_t)qrow * D;
        uint16_t* brow = O + hoff + (size_t)qrow * D;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            f32x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = acc[mb][i] / l;
            *reinterpret_cast<f32x4*>(orow + 16 * mb + 4 * g) = o;
            st_bf16x4(brow + 16 * mb + 4 * g, o[0], o[1], o[2], o[3]);
        }
        if (g == 0) {
            const size_t r = (size_t)bh * N + qrow;
            LSE[r] = mrun + logf(l);
            Mrow[r] = mrun;
            Linv[r] = inv;
        }
    }
}

// ------------------------------------------------------- query-major pass
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 4 : 2) void f32_dq_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, const uint16_t* __restrict__ dO,
    const float* __restrict__ O32, const float* __restrict__ Mrow,
    const float* __restrict__ Linv, float* __restrict__ TS, uint16_t* __restrict__ dQ, int BH,
    int N, int causal, float scale) {
    constexpr int KC = D / 32, MB = D / 16;
    __shared__ __attribute__((aligned(16))) uint16_t KV0[2][kTile * D];
    __shared__ __attribute__((aligned(16))) uint16_t KV1[2][kTile * D];
    const int T = (N + kTile - 1) / kTile;
    int bh, tile;
    map_block(blockIdx.x, BH, T, causal != 0, &bh, &tile, D == 64 ? 4 : 0, true);
    const size_t hoff = (size_t)bh * N * D;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c16 = lane & 15;
    const int qrow = tile * kTile + 16 * wave + c16;
    const bool qok = qrow < N;

    const uint32_t tb = (uint32_t)N * (2 * D);
    bf16x8 qf[KC], uf[KC];
    ld_row_chunks<D>(make_rsrc(Q + hoff, tb), qrow, g, qf);
    ld_row_chunks<D>(make_rsrc(dO + hoff, tb), qrow, g, uf);
    // D_i = sum_d dO_id O32_id (the saved FP32 output), this lane's d subset
    // then the other three lanes of the query.
    float dpart = 0.f;
    if (qok) {
        const float* orow = O32 + hoff + (size_t)qrow * D;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const f32x4 o = *reinterpret_cast<const f32x4*>(orow + 32 * kc + 8 * g + 4 * p);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    dpart = fmaf(bf16_to_f32(uf[kc][4 * p + e]), o[e], dpart);
            }
    }
    const float Di = xor_sum(dpart);
    const size_t srow = (size_t)bh * N + qrow;
    const float mi = qok ? Mrow[srow] : INFINITY;  // rows beyond N: P = 0
    const float li = qok ? Linv[srow] : 0.f;
    const float lg = kLog2e;

    const KeyRange kr = key_range(tile, N, 0, causal);
    const int nkv = kr.nkv, nplain = kr.nplain;
    f32x4 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    TileDma<D> dma;
    dma.init(lane, wave);
    wait_vm_lgkm0<0>();
    dma.load(K + hoff, KV0[0], 0, N);
    dma.load(V + hoff, KV0[1], 0, N);
    wait_vm_lgkm0<0>();
    __syncthreads();

    // dS of key block kb of tile kt from its S and dP
    auto grads = [&](auto masked, int kt, int kb, const f32x4& s, const f32x4& dp, f32x4& ds) {
        constexpr bool MASK = decltype(masked)::value;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float p = fexp2((scale * s[i] - mi) * lg) * li;
            if constexpr (MASK) {
                const int key = kt * kTile + 16 * kb + 4 * g + i;
                p = (key < N && (!causal || key <= qrow)) ? p : 0.f;
            }
            ds[i] = p * (dp[i] - Di);
            if constexpr (MASK) ds[i] = p != 0.f ? ds[i] : 0.f;
        }
    };
    auto step = [&](auto masked, int kt, const uint16_t* Kc, const uint16_t* Vc, uint16_t* Kn,
                    uint16_t* Vn) {
        if (kt + 1 < nkv) {
            dma.load(K + hoff, Kn, (kt + 1) * kTile, N);
            dma.load(V + hoff, Vn, (kt + 1) * kTile, N);
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x4 ds[4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            const f32x4 s = block_dot<D>(Kc, 16 * kb, qf, c16, g);
            const f32x4 dp = block_dot<D>(Vc, 16 * kb, uf, c16, g);
            grads(masked, kt, kb, s, dp, ds[kb]);
        }
        tr_accumulate<D, false>(Kc, ds, acc, c16, g);
        wait_vm_lgkm0<0>();
        __syncthreads();
    };
    const std::false_type plain;
    const std::true_type masked;
    // Two steps a turn, each with its buffers: the accumulators then stay where they
    // are over the loop's edge, and no copy of them can come too early (mfma_settle).
    int kt = 0;
    for (; kt + 1 < nplain; kt += 2) {
        step(plain, kt, KV0[0], KV0[1], KV1[0], KV1[1]);
        step(plain, kt + 1, KV1[0], KV1[1], KV0[0], KV0[1]);
    }
    if (kt < nplain) {
        step(plain, kt, KV0[0], KV0[1], KV1[0], KV1[1]);
        ++kt;
    }
    // Tile kt lives in buffer kt mod 2.
    // At most one tile needs masks: the diagonal one, or the key tail.
    if (kt < nkv) {
        if (kt & 1) step(masked, kt, KV1[0], KV1[1], KV0[0], KV0[1]);
        else step(masked, kt, KV0[0], KV0[1], KV1[0], KV1[1]);
    }
    mfma_settle();
    if (__builtin_expect(wave_nan(nan_sum(acc)), 0)) {  // again, as in the forward
        uint16_t* buf = wave < 2 ? KV0[wave] : KV1[wave - 2];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int t = 0; t < nkv; ++t) {
            f32x4 s[4], ds[4];
            stage_alone<D>(lane, K + hoff, buf, t * kTile, N);
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) s[kb] = block_dot<D>(buf, 16 * kb, qf, c16, g);
            stage_alone<D>(lane, V + hoff, buf, t * kTile, N);
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const f32x4 dp = block_dot<D>(buf, 16 * kb, uf, c16, g);
                if (t < nplain) grads(plain, t, kb, s[kb], dp, ds[kb]);
                else grads(masked, t, kb, s[kb], dp, ds[kb]);
            }
            stage_alone<D>(lane, K + hoff, buf, t * kTile, N);
            tr_accumulate<D, true>(buf, ds, acc, c16, g);
            mfma_settle();
        }
    }

    if (qok) {
        uint16_t* drow = dQ + hoff + (size_t)qrow * D;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            st_bf16x4(drow + 16 * mb + 4 * g, scale * acc[mb][0], scale * acc[mb][1],
                      scale * acc[mb][2], scale * acc[mb][3]);
    }
    // the tile's statistics for the key-major pass
    if (g == 0) {
        float* ts = TS + ((size_t)bh * T + tile) * kF32Stat + 16 * wave + c16;
        ts[0] = mi;
        ts[kTile] = li;
        ts[2 * kTile] = qok ? Di : 0.f;
    }
}

// --------------------------------------------------------- key-major pass
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void f32_dkdv_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, const uint16_t* __restrict__ dO,
    const float* __restrict__ TS, uint16_t* __restrict__ dK, uint16_t* __restrict__ dV, int BH,
    int N, int causal, float scale) {
    constexpr int KC = D / 32, MB = D / 16;
    __shared__ __attribute__((aligned(16))) uint16_t QU0[2][kTile * D];
    __shared__ __attribute__((aligned(16))) uint16_t QU1[2][kTile * D];
    __shared__ __attribute__((aligned(16))) float ST0[kF32Stat];
    __shared__ __attribute__((aligned(16))) float ST1[kF32Stat];
    const int T = (N + kTile - 1) / kTile;
    int bh, tile;
    map_block(blockIdx.x, BH, T, false, &bh, &tile, D == 64 ? 3 : 0, true);
    const size_t hoff = (size_t)bh * N * D;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c16 = lane & 15;
    const int krow = tile * kTile + 16 * wave + c16;

    const uint32_t tb = (uint32_t)N * (2 * D);
    bf16x8 kf[KC], vf[KC];
    ld_row_chunks<D>(make_rsrc(K + hoff, tb), krow, g, kf);
    ld_row_chunks<D>(make_rsrc(V + hoff, tb), krow, g, vf);
    const float lg = kLog2e;
    const float* tsh = TS + (size_t)bh * T * kF32Stat;

    f32x4 accV[MB], accK[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        accV[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
        accK[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int qt0 = causal ? tile : 0;  // the diagonal tile first, masked

    TileDma<D> dma;
    dma.init(lane, wave);
    // Query tile qt's Q and dO tiles and its statistics block (waves 0..2 each
    // move one 256-byte third of it with a 4-byte LDS DMA), issued through the
    // vector-memory path the closing vmcnt(0) waits for: no load in the loop
    // is visible to the compiler's own wait counting.
    auto fill = [&](int qt, uint16_t (*QU)[kTile * D], float* ST) {
        dma.load(Q + hoff, QU[0], qt * kTile, N);
        dma.load(dO + hoff, QU[1], qt * kTile, N);
        if (wave < 3)
            lds_dma4(buf_desc(tsh + (size_t)qt * kF32Stat + wave * kTile, kTile * 4),
                     lds_addr(ST + wave * kTile), (uint32_t)lane * 4u);
    };
    wait_vm_lgkm0<0>();
    fill(qt0 < T ? qt0 : 0, QU0, ST0);
    wait_vm_lgkm0<0>();
    __syncthreads();

    // P and dS of query block qb of tile qt from its S and dP and the tile's statistics
    auto grads = [&](auto masked, int qt, int qb, const float* st, const f32x4& s, const f32x4& dp,
                     f32x4& p, f32x4& ds) {
        constexpr bool MASK = decltype(masked)::value;
        const f32x4 mq = *reinterpret_cast<const f32x4*>(st + 16 * qb + 4 * g);
        const f32x4 lq = *reinterpret_cast<const f32x4*>(st + kTile + 16 * qb + 4 * g);
        const f32x4 dq = *reinterpret_cast<const f32x4*>(st + 2 * kTile + 16 * qb + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float pv = fexp2((scale * s[i] - mq[i]) * lg) * lq[i];
            if constexpr (MASK) {
                const int query = qt * kTile + 16 * qb + 4 * g + i;
                pv = (!causal || krow <= query) ? pv : 0.f;
            }
            p[i] = pv;
            ds[i] = pv * (dp[i] - dq[i]);
            if constexpr (MASK) ds[i] = pv != 0.f ? ds[i] : 0.f;
        }
    };
    auto step = [&](auto masked, int qt, uint16_t (*QUc)[kTile * D], const float* st,
                    uint16_t (*QUn)[kTile * D], float* STn) {
        const uint16_t* Qc = QUc[0];
        const uint16_t* Uc = QUc[1];
        if (qt + 1 < T) fill(qt + 1, QUn, STn);
        __builtin_amdgcn_sched_barrier(0);
        f32x4 p[4], ds[4];
#pragma unroll
        for (int qb = 0; qb < 4; ++qb) {
            const f32x4 s = block_dot<D>(Qc, 16 * qb, kf, c16, g);
            const f32x4 dp = block_dot<D>(Uc, 16 * qb, vf, c16, g);
            grads(masked, qt, qb, st, s, dp, p[qb], ds[qb]);
        }
        tr_accumulate<D, false>(Uc, p, accV, c16, g);
        tr_accumulate<D, false>(Qc, ds, accK, c16, g);
        wait_vm_lgkm0<0>();
        __syncthreads();
    };
    const std::false_type plain;
    const std::true_type masked;
    int qt = qt0;
    // The first tile (there always is one) is staged in slot 0 whatever its index:
    // slots alternate with the step count from qt0.
    if (causal) step(masked, qt, QU0, ST0, QU1, ST1);
    else step(plain, qt, QU0, ST0, QU1, ST1);
    ++qt;
    // two steps a turn, as in the passes above
    for (; qt + 1 < T; qt += 2) {
        step(plain, qt, QU1, ST1, QU0, ST0);
        step(plain, qt + 1, QU0, ST0, QU1, ST1);
    }
    if (qt < T) step(plain, qt, QU1, ST1, QU0, ST0);
    mfma_settle();
    if (__builtin_expect(wave_nan(nan_sum(accV) + nan_sum(accK)), 0)) {  // again, as in the forward
        uint16_t* buf = wave < 2 ? QU0[wave] : QU1[wave - 2];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            accV[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
            accK[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 1
        for (int t = qt0; t < T; ++t) {
            f32x4 s[4], p[4], ds[4];
            stage_alone<D>(lane, Q + hoff, buf, t * kTile, N);
#pragma unroll
            for (int qb = 0; qb < 4; ++qb) s[qb] = block_dot<D>(buf, 16 * qb, kf, c16, g);
            stage_alone<D>(lane, dO + hoff, buf, t * kTile, N);
            const float* st = tsh + (size_t)t * kF32Stat;
#pragma unroll
            for (int qb = 0; qb < 4; ++qb) {
                const f32x4 dp = block_dot<D>(buf, 16 * qb, vf, c16, g);
                if (t == qt0) grads(masked, t, qb, st, s[qb], dp, p[qb], ds[qb]);
                else grads(plain, t, qb, st, s[qb], dp, p[qb], ds[qb]);
            }
            tr_accumulate<D, true>(buf, p, accV, c16, g);
            stage_alone<D>(lane, Q + hoff, buf, t * kTile, N);
            tr_accumulate<D, true>(buf, ds, accK, c16, g);
            mfma_settle();
        }
    }

    if (krow < N) {
        uint16_t* vrow = dV + hoff + (size_t)krow * D;
        uint16_t* krw = dK + hoff + (size_t)krow * D;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            st_bf16x4(vrow + 16 * mb + 4 * g, accV[mb][0], accV[mb][1], accV[mb][2], accV[mb][3]);
            st_bf16x4(krw + 16 * mb + 4 * g, scale * accK[mb][0], scale * accK[mb][1],
                      scale * accK[mb][2], scale * accK[mb][3]);
        }
    }
}

}  // namespace

hipError_t launch_f32_fwd(const uint16_t* Q, const uint16_t* K, const uint16_t* V, float* O32,
                          uint16_t* O, float* LSE, float* Mrow, float* Linv, const Shape& s,
                          hipStream_t st) {
    const int T = (s.N + kTile - 1) / kTile;
    dim3 grid((unsigned)(s.BH * T)), block(kThreads);
    if (s.d == 64)
        launch_kernel(f32_fwd_kernel<64>, grid, block, st, Q, K, V, O32, O, LSE, Mrow, Linv, s.BH,
                      s.N, s.causal, s.scale);
    else
        launch_kernel(f32_fwd_kernel<128>, grid, block, st, Q, K, V, O32, O, LSE, Mrow, Linv, s.BH,
                      s.N, s.causal, s.scale);
    return hipGetLastError();
}

hipError_t launch_f32_dq(const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                         const uint16_t* dO, const float* O32, const float* Mrow,
                         const float* Linv, float* TS, uint16_t* dQ, const Shape& s,
                         hipStream_t st) {
    const int T = (s.N + kTile - 1) / kTile;
    dim3 grid((unsigned)(s.BH * T)), block(kThreads);
    if (s.d == 64)
        launch_kernel(f32_dq_kernel<64>, grid, block, st, Q, K, V, dO, O32, Mrow, Linv, TS, dQ,
                      s.BH, s.N, s.causal, s.scale);
    else
        launch_kernel(f32_dq_kernel<128>, grid, block, st, Q, K, V, dO, O32, Mrow, Linv, TS, dQ,
                      s.BH, s.N, s.causal, s.scale);
    return hipGetLastError();
}

hipError_t launch_f32_dkdv(const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                           const uint16_t* dO, const float* TS, uint16_t* dK, uint16_t* dV,
                           const Shape& s, hipStream_t st) {
    const int T = (s.N + kTile - 1) / kTile;
    dim3 grid((unsigned)(s.BH * T)), block(kThreads);
    if (s.d == 64)
        launch_kernel(f32_dkdv_kernel<64>, grid, block, st, Q, K, V, dO, TS, dK, dV, s.BH, s.N,
                      s.causal, s.scale);
    else
        launch_kernel(f32_dkdv_kernel<128>, grid, block, st, Q, K, V, dO, TS, dK, dV, s.BH, s.N,
                      s.causal, s.scale);
    return hipGetLastError();
}

}  // namespace gpa
