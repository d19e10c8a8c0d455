// FA3-SBS attention forward on gfx950 bf16 MFMA (appendix "Implemented
// Arithmetic and Rounding", eq. gproj-forward): the exponent argument is
// fl32[ sub32(x, xmax) * fl32(alpha log2 e) ] with the unscaled logit x and the
// unscaled running row maximum xmax, so the largest logit maps to exactly
// exp2(0) = 1.
//
// Schedule: one workgroup per (batch*head, 64-query tile); 4 waves.  Wave w
// owns 32 of the 64 queries (two 16-query MFMA blocks sharing every LDS
// fragment) and half of each 64-key tile; the two waves with the same queries
// merge their online-softmax states at the end with the same rescale rule.  K
// and V tiles are loaded straight into LDS (row-major, swizzled, double
// buffered); V is read back transposed with the LDS transpose load.  A wave
// computes S^T = K Q^T with v_mfma_f32_16x16x32_bf16, so each lane holds the
// logits of ONE query (its column): the row maximum and sum are in-lane except
// for a 4-way exchange.  The probabilities are then already in the B-operand
// layout of O^T += V^T P^T, whose accumulator again keeps one query per lane,
// so the online-softmax rescale is a per-lane scalar.
#include "gpa_device.h"
#include "gpa_launch.h"

#include <algorithm>
#include <type_traits>

namespace gpa {
namespace {

// Exponent argument of z = exp2(arg).  FA3-SBS (the path's forward):
// fl32[fl32(x - m) * c].  FMA (diagnostic only): the historical rounding
// fma(x, c, -fl32(m * c)), whose result is the rounding error of x*c rather
// than 0 when x = m (appendix on the source of the saved-output error, eq.
// historical-fma).
template <bool FMA>
__device__ __forceinline__ float exp_arg(float x, float m, float c) {
    if constexpr (FMA) {
#pragma clang fp contract(off)
        const float mc = m * c;
        return __builtin_fmaf(x, c, -mc);
    } else {
#pragma clang fp contract(off)
        return (x - m) * c;
    }
}

// How a forward kernel takes the packed sequences that few_sequence (gpa_launch.h)
// names: like the others (kNone), by splits of their keys that leave their states in a
// workspace (kSplit), or by the same splits one after the other (kWalk).
enum class Few { kNone, kSplit, kWalk };
struct FewArgs {
    float* Oacc = nullptr;  // states: FP32 O^T accumulators [Hkv, rows, D],
    float* ML = nullptr;    // row maxima and sums [Hkv, rows, 2]
    int64_t rows = 0;       // state rows of a key/value head
    int blocks = 0;         // workgroups that take them, before the others
    int places = 0;         // (row tile, split) places of a (sequence, key/value head)
    uint32_t items = 0;     // places in all
};

// Weights of a row's state (maximum m) and of the next split's (maximum mi) under
// their common maximum, by the rescale rule that the forward uses between tiles.
__device__ __forceinline__ void few_weights(float& m, float mi, float c, float& w, float& wi) {
    const float mn = fmaxf(m, mi);
    const float ms = (mn == -INFINITY) ? 0.f : mn;
    w = fexp2((m - ms) * c);
    wi = fexp2((mi - ms) * c);
    m = mn;
}

// Few queries against long key runs.  A workgroup of the kernels below would fill
// a few of its 64 query rows and walk every key tile alone, and each query head
// would read its group's K and V again.  Here the rows of a (sequence, key/value
// head) are all G heads' queries (row r: head r / nq, query r % nq), so K and V are
// read once per row tile, and the key tiles are split (few_chunk).  Per (query, key)
// the arithmetic is fwd_sbs_q16_kernel's; every split has an unnormalised state (O^T
// accumulator, row maximum, row sum; FP32) of its own, and the states of a row are
// taken together in split order, by fwd_few_merge_kernel or (kWalk) right here.
// These workgroups run in the launch of the pack's other sequences, in front of
// them: a launch of their own would leave the chip to short sequences that take as
// long.  What bounds it: the latency of each split's few tiles, then HBM.  8
// sequences of 4 queries on 406 to 5115 keys, 16 heads on 4, d = 128 (47 MB of K and
// V): 68 us in the ordinary forward, 14.8 us here and 4.3 us for the merge; 24 of 1
// on 1292 to 8192 keys, 32 heads on 8 (466 MB): 270 us, 84 and 4.6 us (5.5 TB/s).
template <int D, Few FEW>
__device__ __forceinline__ void few_rows(
    uint16_t (&KV0)[2][kTile * D], uint16_t (&KV1)[2][kTile * D], int bid,
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, uint16_t* __restrict__ O, float* __restrict__ LSE, int Nmax,
    int causal, float scale, int G, const int* __restrict__ cu, int Hq, int total,
    const int* __restrict__ cu_k, int total_k, int Nkmax, const FewArgs& few) {
    constexpr int MB = D / 16;
    constexpr int KC = D / 32;
    const int Hkv = Hq / G;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c16 = lane & 15;
    const float c = scale * kLog2e;
    TileDma<D> dma;
    dma.init(lane, wave);

    // items [sequence][key/value head][place]
    for (uint32_t item = bid; item < few.items; item += few.blocks) {
        const int prob = (int)(item / few.places);
        const int place = (int)(item - (uint32_t)prob * few.places);
        const int seq = prob / Hkv, kvh = prob - seq * Hkv;
        const SeqRows sr = seq_rows(cu, cu_k, seq * Hq + kvh * G, Nmax, Nkmax, G, Hq, total, total_k);
        const int N = sr.nq, Nk = sr.nk;
        if (N == 0 || !few_sequence(N, Nk, G)) continue;
        const int rows = G * N;
        const int RT = (rows + kTile - 1) / kTile, tiles = (Nk + kTile - 1) / kTile;
        const int chunk = few_chunk(RT, tiles);
        const int S = (tiles + chunk - 1) / chunk;
        // Each problem's places begin elsewhere, so that problems that fill few of them
        // are spread over the XCDs all the same.
        const int w = (int)(((uint32_t)place + 3u * (uint32_t)prob) % (uint32_t)few.places);
        const int rt = FEW == Few::kWalk ? w : w / S, first = FEW == Few::kWalk ? 0 : w % S;
        if (rt >= RT) continue;
        const int last = FEW == Few::kWalk ? S : first + 1;
        const int off = Nk - N;
        const size_t kvoff = sr.kv0 * D;
        const int r = rt * kTile + 16 * wave + c16;         // this lane's row
        const bool active = rt * kTile + 16 * wave < rows;  // the wave has a row
        const int hg = r / N, qi = r - hg * N;       // its head in the group and query
        const size_t qrow = sr.q0 + (size_t)hg * total + qi;  // its row of Q, O and LSE

        // the first tile's loads go out before the operands'
        auto fill = [&](int kt, uint16_t (&KV)[2][kTile * D]) {
            dma.load(K + kvoff, KV[0], kt * kTile, Nk);
            dma.load(V + kvoff, KV[1], kt * kTile, Nk);
        };
        wait_vm_lgkm0<0>();
        fill(first * chunk, KV0);
        bf16x8 qf[KC];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            u32x4 w = {0u, 0u, 0u, 0u};
            if (r < rows) w = *reinterpret_cast<const u32x4*>(Q + qrow * D + kc * 32 + 8 * g);
            qf[kc] = __builtin_bit_cast(bf16x8, w);
        }
        // the first tile that needs masks: every query sees the keys up to the
        // first query's last one
        const int nplain = min(causal ? max(floor_div(off + 1, kTile), 0) : Nk / kTile, Nk / kTile);

        float mrow = -INFINITY, lrow = 0.f;  // kWalk: the row's state so far
        f32x4 orow[MB];
        if constexpr (FEW == Few::kWalk)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) orow[mb] = f32x4{0.f, 0.f, 0.f, 0.f};

        for (int split = first; split < last; ++split) {
            float mrun = -INFINITY, lrun = 0.f;
            f32x4 acc[MB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int kt0 = split * chunk, kt1 = min(kt0 + chunk, tiles);

            if (split > first) fill(kt0, KV0);
            wait_vm_lgkm0<0>();
            __syncthreads();

            auto compute = [&](auto masked, int kt, const uint16_t* Kc, const uint16_t* Vc) {
                constexpr bool MASK = decltype(masked)::value;
                f32x4 s[4];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    s[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kc = 0; kc < KC; ++kc)
                        s[kb] = mfma_16x16x32(
                            ld_b128(Kc + tile_off<D>(kb * 16 + c16, kc * 32 + 8 * g)), qf[kc], s[kb]);
                }
                if constexpr (MASK) {
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int key = kt * kTile + kb * 16 + 4 * g + i;
                            const bool ok = key < Nk && (!causal || key <= qi + off);
                            s[kb][i] = ok ? s[kb][i] : -INFINITY;
                        }
                }
                float mx = s[0][0];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[kb][i]);
                mx = xor_max(mx);
                const float mnew = fmaxf(mrun, mx);
                const float ms = (mnew == -INFINITY) ? 0.f : mnew;
                if (__builtin_amdgcn_ballot_w64(mnew != mrun) != 0) {
                    const float corr = fexp2((mrun - ms) * c);
                    lrun *= corr;
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc[mb] *= corr;
                }
                bf16x8 pf[2];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float z = fexp2(exp_arg<false>(s[kb][i], ms, c));
                        lrun += z;
                        pf[kb >> 1][(kb & 1) * 4 + i] = to_bf16(z);
                    }
                mrun = mnew;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[mb] = mfma_16x16x32(ld_tr_operand<D>(Vc, 32 * j, mb * 16, c16, g), pf[j],
                                                acc[mb]);
                mfma_settle();
            };
            auto step = [&](int kt, const uint16_t (&KV)[2][kTile * D],
                            uint16_t (&next)[2][kTile * D]) {
                if (kt + 1 < kt1) fill(kt + 1, next);
                __builtin_amdgcn_sched_barrier(0);
                if (active) {
                    if (kt < nplain) compute(std::false_type{}, kt, KV[0], KV[1]);
                    else compute(std::true_type{}, kt, KV[0], KV[1]);
                }
                wait_vm_lgkm0<0>();
                __syncthreads();
            };
            for (int kt = kt0; kt < kt1; kt += 2) {
                step(kt, KV0, KV1);
                if (kt + 1 < kt1) step(kt + 1, KV1, KV0);
            }

            const float ltot = xor_sum(lrun);
            if constexpr (FEW == Few::kWalk) {
                // l = 0: the split saw none of the row's keys (on the bits, as in
                // the kernels below), and its accumulator may hold anything
                if (__float_as_uint(ltot) != 0u) {
                    float w, wi;
                    few_weights(mrow, mrun, c, w, wi);
                    lrow = __builtin_fmaf(ltot, wi, lrow * w);
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            orow[mb][i] = __builtin_fmaf(acc[mb][i], wi, orow[mb][i] * w);
                }
            } else if (r < rows) {
                const size_t p = (size_t)kvh * few.rows +
                                 few_base(seq, sr.q0 - (size_t)kvh * G * total,
                                          sr.kv0 - (size_t)kvh * total_k, G) +
                                 (size_t)split * rows + r;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    *reinterpret_cast<f32x4*>(few.Oacc + p * D + mb * 16 + 4 * g) = acc[mb];
                if (g == 0) {
                    few.ML[2 * p] = mrun;
                    few.ML[2 * p + 1] = ltot;
                }
            }
        }
        if constexpr (FEW == Few::kWalk) {
            if (r < rows) {
                const bool empty = __float_as_uint(lrow) == 0u;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = empty ? 0.f : orow[mb][i] / lrow;
                    st_bf16x4(O + qrow * D + mb * 16 + 4 * g, v[0], v[1], v[2], v[3]);
                }
                if (g == 0) {
#pragma clang fp contract(off)
                    const float lse = scale * mrow + logf(lrow);
                    LSE[qrow] = empty ? INFINITY : lse;
                }
            }
        }
    }
}

template <int D, bool FMA, bool UNEVEN, Few FEW>
__global__ __launch_bounds__(kThreads, FEW == Few::kWalk ? 1 : GPA_FWD_OCC) void fwd_sbs_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, uint16_t* __restrict__ O, float* __restrict__ LSE,
    int BH, int Nmax, int causal, float scale, int G, const int* __restrict__ cu, int Hq,
    int total, const int* __restrict__ cu_k, int total_k, int Nkmax, FewArgs few) {
    constexpr int MB = D / 16;
    constexpr int KC = D / 32;
    constexpr int PER_NB = MB * 4 + 2;  // acc, m, l of one query block
    // K and V tiles, double-buffered in two separate LDS objects so the
    // compiler can tell the tile being read from the one the DMA is filling.
    __shared__ __attribute__((aligned(16))) uint16_t KV0[2][kTile * D];
    __shared__ __attribute__((aligned(16))) uint16_t KV1[2][kTile * D];

    int bid = blockIdx.x;
    if constexpr (FEW != Few::kNone) {
        if (bid < few.blocks) {
            few_rows<D, FEW>(KV0, KV1, bid, Q, K, V, O, LSE, Nmax, causal, scale, G, cu, Hq, total,
                             cu_k, total_k, Nkmax, few);
            return;
        }
        bid -= few.blocks;
    }
    const int T = (Nmax + kTile - 1) / kTile;  // tiles of the longest problem
    int bh, tile;
    if constexpr (UNEVEN) {
        if (!map_packed(bid, BH, Hq, Nmax, cu, total, causal != 0, &bh, &tile)) return;
    } else map_block(bid, BH, T, causal != 0, &bh, &tile, 2);
    const SeqRows sr = seq_rows(cu, cu_k, bh, Nmax, Nkmax, G, Hq, total, total_k);
    const int N = sr.nq, Nk = sr.nk;
    if (tile * kTile >= N) return;  // a shorter sequence has no such tile
    if constexpr (FEW != Few::kNone)
        if (few_sequence(N, Nk, G)) return;  // taken by few_rows
    const int off = Nk - N;           // causal: query i sees key j iff j <= i + off
    const size_t hoff = sr.q0 * D;    // query head: Q, O
    const size_t kvoff = sr.kv0 * D;  // its key/value head
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c16 = lane & 15;
    const int qh = wave & 1;   // which 32 of the workgroup's 64 queries
    const int kh = wave >> 1;  // which 32 of each 64-key tile
    const int q0w = tile * kTile + 32 * qh;

    // Q^T as the B operand: column = this lane's query of block nb, k = d.
    const rsrc_t rq = make_rsrc(Q + hoff, (uint32_t)N * (2 * D));
    bf16x8 qf[2][KC];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
            qf[nb][kc] = __builtin_bit_cast(bf16x8, ld_row16<D>(rq, q0w + nb * 16 + c16, kc * 32 + 8 * g));

    const float c = scale * kLog2e;  // fl32(alpha log2 e)
    float mrun[2] = {-INFINITY, -INFINITY};  // running maximum of the unscaled logits
    float lrun[2] = {0.f, 0.f};              // this lane's share of the running sum of z
    f32x4 acc[2][MB];                        // O^T[dv][query]
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Only the last one or two key tiles need masks (the causal diagonal, the
    // key tail).
    const KeyRange kr = key_range(tile, Nk, off, causal);
    const int nkv = kr.nkv, nplain = kr.nplain;

    // Zero both buffers once, so that every value a product can read is finite
    // whatever the DMA leaves in the slots of rows beyond Nk (it writes zeros
    // there, but the tail does not depend on it).
    {
        u32x4* z0 = reinterpret_cast<u32x4*>(&KV0[0][0]);
        u32x4* z1 = reinterpret_cast<u32x4*>(&KV1[0][0]);
        constexpr int n16 = (int)(sizeof(KV0) / 16);
#pragma unroll
        for (int i = tid; i < n16; i += kThreads) {
            z0[i] = u32x4{0u, 0u, 0u, 0u};
            z1[i] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    __syncthreads();

    TileDma<D> dma;
    dma.init(lane, wave);
    dma.load(K + kvoff, KV0[0], 0, Nk);
    dma.load(V + kvoff, KV0[1], 0, Nk);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    auto step = [&](auto masked, int kt, const uint16_t* Kc, const uint16_t* Vc, uint16_t* Kn,
                    uint16_t* Vn) {
        constexpr bool MASK = decltype(masked)::value;
        const int k0 = kt * kTile;
        if (kt + 1 < nkv) {
            dma.load(K + kvoff, Kn, k0 + kTile, Nk);
            dma.load(V + kvoff, Vn, k0 + kTile, Nk);
        }
        // Keep the loads of the next tile at the top of the step: left alone,
        // the scheduler sinks them next to the closing wait, which exposes
        // their whole latency.
        __builtin_amdgcn_sched_barrier(0);
        // S^T[key][query] for this wave's 32 keys x 32 queries; s[nb][kb]
        // holds keys 4g+i of key block kb for query block nb.  The wave raises
        // its issue priority while it feeds the matrix core, so that the other
        // wave on the SIMD runs its exponentials meanwhile (h16_n4096_d128
        // forward 6 % faster; neutral on the batched d = 128 workload).
        __builtin_amdgcn_s_setprio(1);
        f32x4 s[2][2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            s[0][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
            s[1][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const bf16x8 ka = ld_b128(Kc + tile_off<D>(32 * kh + kb * 16 + c16, kc * 32 + 8 * g));
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) s[nb][kb] = mfma_16x16x32(ka, qf[nb][kc], s[nb][kb]);
            }
        }
        if constexpr (MASK) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int key = k0 + 32 * kh + kb * 16 + 4 * g + i;
                        const int qrow = q0w + nb * 16 + c16;
                        const bool ok = key < Nk && (!causal || key <= qrow + off);
                        s[nb][kb][i] = ok ? s[nb][kb][i] : -INFINITY;
                    }
        }
        __builtin_amdgcn_s_setprio(0);
        bf16x8 pf[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            float mx = s[nb][0][0];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[nb][kb][i]);
            mx = xor_max(mx);
            const float mnew = fmaxf(mrun[nb], mx);
            // A wave half may not have seen a visible key yet (mnew = -inf);
            // then every z is 0 and nothing is rescaled.
            const float ms = (mnew == -INFINITY) ? 0.f : mnew;
            // Rescale by exp2(fl32[fl32(mold - mnew) * c]): the same rule as z;
            // skipped when no query of the wave has a new maximum (corr is then
            // exactly 1).
            if (__builtin_amdgcn_ballot_w64(mnew != mrun[nb]) != 0) {
                const float corr = fexp2((mrun[nb] - ms) * c);
                lrun[nb] *= corr;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[nb][mb] *= corr;
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float z = fexp2(exp_arg<FMA>(s[nb][kb][i], ms, c));
                    lrun[nb] += z;
                    pf[nb][kb * 4 + i] = to_bf16(z);
                }
            mrun[nb] = mnew;
        }
        // O^T[dv][query] += V^T[dv][key] P^T[key][query].
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const bf16x8 va = ld_tr_operand<D>(Vc, 32 * kh, mb * 16, c16, g);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) acc[nb][mb] = mfma_16x16x32(va, pf[nb], acc[nb][mb]);
        }
        if constexpr (MASK) mfma_settle();  // the loop over these steps copies acc
        __builtin_amdgcn_s_waitcnt(0);  // this wave's loads of the next tile
        __syncthreads();
    };
    const std::false_type plain;
    const std::true_type masked;
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
    for (; kt < nkv; ++kt) {
        if (kt & 1)
            step(masked, kt, KV1[0], KV1[1], KV0[0], KV0[1]);
        else
            step(masked, kt, KV0[0], KV0[1], KV1[0], KV1[1]);
    }

    // Merge the two key halves of each query (waves w and w + 2): waves 2, 3
    // park (acc, m, l) in LDS, waves 0, 1 combine them with the same rescale
    // rule and finish.
    // Query block nb goes through buffer object nb (each holds 2 x 64 x PER_NB
    // floats).
    static_assert(sizeof(KV0) >= 2 * 64 * PER_NB * sizeof(float), "merge space");
    float* const scratch[2] = {reinterpret_cast<float*>(&KV0[0][0]),
                               reinterpret_cast<float*>(&KV1[0][0])};
    if (wave >= 2) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            float* p = scratch[nb] + (wave - 2) * 64 * PER_NB + lane;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) p[(mb * 4 + i) * 64] = acc[nb][mb][i];
            p[(MB * 4) * 64] = mrun[nb];
            p[(MB * 4 + 1) * 64] = lrun[nb];
        }
    }
    __syncthreads();
    if (wave >= 2) return;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const float* p = scratch[nb] + wave * 64 * PER_NB + lane;
        const float mo = p[(MB * 4) * 64];
        const float lo = p[(MB * 4 + 1) * 64];
        const float mt = fmaxf(mrun[nb], mo);
        const float ms = (mt == -INFINITY) ? 0.f : mt;
        const float fa = fexp2((mrun[nb] - ms) * c);
        const float fb = fexp2((mo - ms) * c);
        const float ltot = xor_sum(lrun[nb] * fa + lo * fb);
        const int qrow = q0w + nb * 16 + c16;
        if (qrow < N) {
            // A query that sees no key (l = 0; a visible key adds z = 1) gets
            // O = 0 and LSE = +inf, so the backward's P is 0 on its row.  l is
            // +0 exactly then; the test is on the bits so that a NaN row (NaN
            // l) keeps NaN outputs whatever the compiler assumes about NaNs.
            const bool empty = __float_as_uint(ltot) == 0u;
            uint16_t* orow = O + hoff + (size_t)qrow * D;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[i] = empty ? 0.f : (acc[nb][mb][i] * fa + p[(mb * 4 + i) * 64] * fb) / ltot;
                st_bf16x4(orow + mb * 16 + 4 * g, v[0], v[1], v[2], v[3]);
            }
            if (g == 0) {
#pragma clang fp contract(off)
                const float lse = scale * mt + logf(ltot);
                LSE[sr.q0 + qrow] = empty ? INFINITY : lse;
            }
        }
    }
}

// Variant with one 16-query block per wave: each of the 4 waves owns 16 of
// the workgroup's 64 queries and runs them against the whole 64-key tile, so
// the online-softmax bookkeeping (row maximum, rescale of the output
// accumulator, correction factor) is paid once per 64 keys and no merge of
// partial states is needed; the price is that every K and V fragment read from
// LDS feeds one MFMA instead of two.  Fewer registers per wave allow more
// waves per SIMD.  The arithmetic per (query, key) is that of fwd_sbs_kernel.
template <int D, bool FMA, bool UNEVEN, Few FEW>
__global__ __launch_bounds__(kThreads, FEW == Few::kWalk ? 2 : GPA_FWD16_OCC) void fwd_sbs_q16_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, uint16_t* __restrict__ O, float* __restrict__ LSE,
    int BH, int Nmax, int causal, float scale, int G, const int* __restrict__ cu, int Hq,
    int total, const int* __restrict__ cu_k, int total_k, int Nkmax, FewArgs few) {
    constexpr int MB = D / 16;
    constexpr int KC = D / 32;
    __shared__ __attribute__((aligned(16))) uint16_t KV0[2][kTile * D];
    __shared__ __attribute__((aligned(16))) uint16_t KV1[2][kTile * D];

    int bid = blockIdx.x;
    if constexpr (FEW != Few::kNone) {
        if (bid < few.blocks) {
            few_rows<D, FEW>(KV0, KV1, bid, Q, K, V, O, LSE, Nmax, causal, scale, G, cu, Hq, total,
                             cu_k, total_k, Nkmax, few);
            return;
        }
        bid -= few.blocks;
    }
    const int T = (Nmax + kTile - 1) / kTile;  // tiles of the longest problem
    int bh, tile;
    if constexpr (UNEVEN) {
        if (!map_packed(bid, BH, Hq, Nmax, cu, total, causal != 0, &bh, &tile)) return;
    } else map_block(bid, BH, T, causal != 0, &bh, &tile, 5, true);
    const SeqRows sr = seq_rows(cu, cu_k, bh, Nmax, Nkmax, G, Hq, total, total_k);
    const int N = sr.nq, Nk = sr.nk;
    if (tile * kTile >= N) return;  // a shorter sequence has no such tile
    if constexpr (FEW != Few::kNone)
        if (few_sequence(N, Nk, G)) return;  // taken by few_rows
    const int off = Nk - N;  // causal: query i sees key j iff j <= i + off
    const size_t hoff = sr.q0 * D;
    const size_t kvoff = sr.kv0 * D;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c16 = lane & 15;
    const int qrow = tile * kTile + 16 * wave + c16;  // this lane's query

    const rsrc_t rq = make_rsrc(Q + hoff, (uint32_t)N * (2 * D));
    bf16x8 qf[KC];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
        qf[kc] = __builtin_bit_cast(bf16x8, ld_row16<D>(rq, qrow, kc * 32 + 8 * g));

    const float c = scale * kLog2e;
    float mrun = -INFINITY, lrun = 0.f;
    f32x4 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const KeyRange kr = key_range(tile, Nk, off, causal);
    const int nkv = kr.nkv, nplain = kr.nplain;

    TileDma<D> dma;
    dma.init(lane, wave);
    wait_vm_lgkm0<0>();
    dma.load(K + kvoff, KV0[0], 0, Nk);
    dma.load(V + kvoff, KV0[1], 0, Nk);
    wait_vm_lgkm0<0>();
    __builtin_amdgcn_s_barrier();

    auto step = [&](auto masked, int kt, const uint16_t* Kc, const uint16_t* Vc, uint16_t* Kn,
                    uint16_t* Vn) {
        constexpr bool MASK = decltype(masked)::value;
        const int k0 = kt * kTile;
        if (kt + 1 < nkv) {
            dma.load(K + kvoff, Kn, k0 + kTile, Nk);
            dma.load(V + kvoff, Vn, k0 + kTile, Nk);
        }
        __builtin_amdgcn_sched_barrier(0);
        // S^T[key][query]: s[kb] holds keys 16 kb + 4g + i for this lane's query.
        f32x4 s[4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            s[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
                s[kb] = mfma_16x16x32(ld_b128(Kc + tile_off<D>(kb * 16 + c16, kc * 32 + 8 * g)),
                                      qf[kc], s[kb]);
        }
        if constexpr (MASK) {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int key = k0 + kb * 16 + 4 * g + i;
                    const bool ok = key < Nk && (!causal || key <= qrow + off);
                    s[kb][i] = ok ? s[kb][i] : -INFINITY;
                }
        }
        float mx = s[0][0];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[kb][i]);
        mx = xor_max(mx);
        const float mnew = fmaxf(mrun, mx);
        const float ms = (mnew == -INFINITY) ? 0.f : mnew;
        // Rescale only when some query of the wave has a new maximum: otherwise
        // corr is exactly 1 in every lane and multiplying by it changes nothing.
        if (__builtin_amdgcn_ballot_w64(mnew != mrun) != 0) {
            const float corr = fexp2((mrun - ms) * c);
            lrun *= corr;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[mb] *= corr;
        }
        // pf[j]: B operand of keys 32 j .. 32 j + 31 (k-layout {4g+i, 16+4g+i}).
        bf16x8 pf[2];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float z = fexp2(exp_arg<FMA>(s[kb][i], ms, c));
                lrun += z;
                pf[kb >> 1][(kb & 1) * 4 + i] = to_bf16(z);
            }
        mrun = mnew;
        // O^T[dv][query] += V^T[dv][key] P^T[key][query].
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[mb] = mfma_16x16x32(ld_tr_operand<D>(Vc, 32 * j, mb * 16, c16, g), pf[j],
                                        acc[mb]);
        if constexpr (MASK) mfma_settle();  // the loop over these steps copies acc
        wait_vm_lgkm0<0>();
        __builtin_amdgcn_s_barrier();
    };
    const std::false_type plain;
    const std::true_type masked;
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
    for (; kt < nkv; ++kt) {
        if (kt & 1)
            step(masked, kt, KV1[0], KV1[1], KV0[0], KV0[1]);
        else
            step(masked, kt, KV0[0], KV0[1], KV1[0], KV1[1]);
    }

    const float ltot = xor_sum(lrun);
    if (qrow < N) {
        // A query that sees no key (l = 0; a visible key adds z = 1) gets O = 0
        // and LSE = +inf, so the backward's P is 0 on its row.  l is +0 exactly
        // then; the test is on the bits so that a NaN row (NaN l) keeps NaN
        // outputs whatever the compiler assumes about NaNs.
        const bool empty = __float_as_uint(ltot) == 0u;
        uint16_t* orow = O + hoff + (size_t)qrow * D;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = empty ? 0.f : acc[mb][i] / ltot;
            st_bf16x4(orow + mb * 16 + 4 * g, v[0], v[1], v[2], v[3]);
        }
        if (g == 0) {
#pragma clang fp contract(off)
            const float lse = scale * mrun + logf(ltot);
            LSE[sr.q0 + qrow] = empty ? INFINITY : lse;
        }
    }
}

// Takes the states of every row together, in split order, and finishes as the
// kernels above do.  D/4 lanes share a row, 4 columns each: they read the
// accumulators of all splits, and a split's row maximum and sum per lane, which LDS
// hands round, before they wait once (about 4 us, whatever S).  items [sequence][key/value head][chunk of rows].
template <int D>
__global__ __launch_bounds__(256) void fwd_few_merge_kernel(
    const float* __restrict__ Oacc, const float* __restrict__ ML, uint16_t* __restrict__ O,
    float* __restrict__ LSE, int Nmax, float scale, int G, const int* __restrict__ cu, int Hq,
    int total, const int* __restrict__ cu_k, int total_k, int Nkmax, int64_t state_rows,
    int probs, int chunks) {
    constexpr int LPR = D / 4;      // lanes of a row
    constexpr int RPB = 256 / LPR;  // rows of a workgroup
    __shared__ float M[RPB][kFewMaxSplits];
    __shared__ float L[RPB][kFewMaxSplits];
    const int rl = threadIdx.x / LPR, j = threadIdx.x - rl * LPR;
    const int col = 4 * j;
    const int Hkv = Hq / G;
    const float c = scale * kLog2e;
    for (uint32_t item = blockIdx.x; item < (uint32_t)probs * (uint32_t)chunks; item += gridDim.x) {
        const int prob = (int)(item / (uint32_t)chunks);
        const int seq = prob / Hkv, kvh = prob - seq * Hkv;
        const SeqRows sr = seq_rows(cu, cu_k, seq * Hq + kvh * G, Nmax, Nkmax, G, Hq, total, total_k);
        const int N = sr.nq, Nk = sr.nk;
        const int rows = G * N;
        const int r0 = (int)(item - (uint32_t)prob * (uint32_t)chunks) * RPB, r = r0 + rl;
        if (!few_sequence(N, Nk, G) || r0 >= rows) continue;
        const int tiles = (Nk + kTile - 1) / kTile;
        const int chunk = few_chunk((rows + kTile - 1) / kTile, tiles);
        const int S = (tiles + chunk - 1) / chunk;
        const bool have = r < rows;
        const size_t p = (size_t)kvh * state_rows +
                         few_base(seq, sr.q0 - (size_t)kvh * G * total,
                                  sr.kv0 - (size_t)kvh * total_k, G) + r;
        static_assert(kFewMaxSplits <= LPR, "a lane per split");
        const bool mine = have && j < S;
        const float mj = mine ? ML[2 * (p + (size_t)j * rows)] : 0.f;
        const float lj = mine ? ML[2 * (p + (size_t)j * rows) + 1] : 0.f;
        f32x4 x[kFewMaxSplits];
#pragma unroll
        for (int i = 0; i < kFewMaxSplits; ++i) {
            x[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (have && i < S)
                x[i] = *reinterpret_cast<const f32x4*>(Oacc + (p + (size_t)i * rows) * D + col);
        }
        if (j < kFewMaxSplits) {
            M[rl][j] = mj;
            L[rl][j] = lj;
        }
        __syncthreads();
        if (have) {
            float m = -INFINITY, l = 0.f;
            f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < kFewMaxSplits; ++i) {
                if (i >= S) break;
                const float li = L[rl][i];
                if (__float_as_uint(li) == 0u) continue;  // none of the row's keys
                float w, wi;
                few_weights(m, M[rl][i], c, w, wi);
                l = __builtin_fmaf(li, wi, l * w);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(x[i][e], wi, o[e] * w);
            }
            const size_t qrow = sr.q0 + (size_t)(r / N) * total + r % N;
            const bool empty = __float_as_uint(l) == 0u;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = empty ? 0.f : o[i] / l;
            st_bf16x4(O + qrow * D + col, v[0], v[1], v[2], v[3]);
            if (j == 0) {
#pragma clang fp contract(off)
                const float lse = scale * m + logf(l);
                LSE[qrow] = empty ? INFINITY : lse;
            }
        }
        __syncthreads();  // M and L have been read
    }
}

}  // namespace

namespace {

// Workgroups that take few-query items in turn: enough to fill the chip several
// times over, and few enough that a pack without such sequences does not wait for
// their exits.
constexpr int64_t kFewBlocks = 2048;

// Most rows that a (sequence, key/value head) with few queries has.
int few_most_rows(const Shape& s) {
    const int64_t rows = (int64_t)s.G * (s.N < kFewQueries ? s.N : kFewQueries);
    return (int)std::min<int64_t>(rows, std::max(kTile, s.Nk / kFewKeysPerRow));
}

// Places of a (sequence, key/value head): the most (row tile, split) pairs that any
// sequence within the longest runs has.
int few_places(const Shape& s, bool walk) {
    const int most = (few_most_rows(s) + kTile - 1) / kTile;
    const int tiles = (s.Nk + kTile - 1) / kTile;
    if (walk) return most;
    int places = 0;
    for (int RT = 1; RT <= most; ++RT)
        places = std::max(places, RT * std::min(kFewMaxSplits, (tiles + 4 * RT - 1) / (4 * RT)));
    return places;
}

template <int D, Few FEW>
hipError_t launch_fwd_as(const uint16_t* Q, const uint16_t* K, const uint16_t* V, uint16_t* O,
                         float* LSE, const Shape& s, hipStream_t st, FewArgs few) {
    const int T = (s.N + kTile - 1) / kTile;
    dim3 grid((unsigned)(s.BH * T)), block(kThreads);
    const bool uneven = uneven_pack(s, s.total, s.N);
    if (uneven) grid.x = packed_grid(s, s.total, s.N);
    if constexpr (FEW != Few::kNone) {
        few.places = few_places(s, FEW == Few::kWalk);
        few.items = (uint32_t)(s.BH / s.G) * (uint32_t)few.places;
        // a launch holds fewer than 2^32 threads, 2^24 workgroups of these
        const int64_t room = (int64_t)0xFFFFFF - grid.x;
        few.blocks = (int)std::max<int64_t>(1, std::min({(int64_t)few.items, kFewBlocks, room}));
        grid.x += (unsigned)few.blocks;
    }
    const int Nk = s.Nk > 0 ? s.Nk : s.N;
#define GPA_FWD(KERNEL, UN)                                                                    \
    launch_kernel(KERNEL<D, false, UN, FEW>, grid, block, st, Q, K, V, O, LSE, s.BH, s.N,      \
                  s.causal, s.scale, s.G, s.cu, s.Hq, s.total, s.cu_k, s.total_k, Nk, few)
    // d = 64: one 16-query block per wave (measured faster); d = 128: two
    // blocks per wave, whose halved LDS reads matter more there.
    if constexpr (D == 64) {
        if (uneven) GPA_FWD(fwd_sbs_q16_kernel, true);
        else GPA_FWD(fwd_sbs_q16_kernel, false);
    } else {
        if (uneven) GPA_FWD(fwd_sbs_kernel, true);
        else GPA_FWD(fwd_sbs_kernel, false);
    }
#undef GPA_FWD
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd(const uint16_t* Q, const uint16_t* K, const uint16_t* V, uint16_t* O,
                      float* LSE, const Shape& s, hipStream_t st, bool fma_forward) {
    if (!fma_forward)
        return s.d == 64 ? launch_fwd_as<64, Few::kNone>(Q, K, V, O, LSE, s, st, {})
                         : launch_fwd_as<128, Few::kNone>(Q, K, V, O, LSE, s, st, {});
    const int T = (s.N + kTile - 1) / kTile;  // dense batches only
    dim3 grid((unsigned)(s.BH * T)), block(kThreads);
#define GPA_FMA(KERNEL, DD)                                                                    \
    launch_kernel(KERNEL<DD, true, false, Few::kNone>, grid, block, st, Q, K, V, O, LSE, s.BH, \
                  s.N, s.causal, s.scale, s.G, s.cu, s.Hq, s.total, s.cu_k, s.total_k,         \
                  s.Nk > 0 ? s.Nk : s.N, FewArgs{})
    if (s.d == 64) GPA_FMA(fwd_sbs_q16_kernel, 64); else GPA_FMA(fwd_sbs_kernel, 128);
#undef GPA_FMA
    return hipGetLastError();
}

hipError_t launch_fwd_few(const uint16_t* Q, const uint16_t* K, const uint16_t* V, uint16_t* O,
                          float* LSE, float* Oacc, float* ML, const Shape& s, hipStream_t st) {
    FewArgs few;
    if (Oacc == nullptr)
        return s.d == 64 ? launch_fwd_as<64, Few::kWalk>(Q, K, V, O, LSE, s, st, few)
                         : launch_fwd_as<128, Few::kWalk>(Q, K, V, O, LSE, s, st, few);
    few.Oacc = Oacc;
    few.ML = ML;
    few.rows = few_base(s.BH / s.Hq, s.total, s.total_k, s.G);
    return s.d == 64 ? launch_fwd_as<64, Few::kSplit>(Q, K, V, O, LSE, s, st, few)
                     : launch_fwd_as<128, Few::kSplit>(Q, K, V, O, LSE, s, st, few);
}

hipError_t launch_fwd_few_merge(const float* Oacc, const float* ML, uint16_t* O, float* LSE,
                                const Shape& s, hipStream_t st) {
    // chunks of 1024 / d rows: no more than key tiles, so probs * chunks < 2^31
    const int chunks = (few_most_rows(s) * (s.d / 4) + 255) / 256;
    const int probs = s.BH / s.G;
    const int64_t items = (int64_t)probs * chunks;
    dim3 grid((unsigned)std::min(items, kFewBlocks)), block(256);
    const int64_t rows = few_base(s.BH / s.Hq, s.total, s.total_k, s.G);
#define GPA_MERGE(DD)                                                                          \
    launch_kernel(fwd_few_merge_kernel<DD>, grid, block, st, Oacc, ML, O, LSE, s.N, s.scale,   \
                  s.G, s.cu, s.Hq, s.total, s.cu_k, s.total_k, s.Nk, rows, probs, chunks)
    if (s.d == 64) GPA_MERGE(64); else GPA_MERGE(128);
#undef GPA_MERGE
    return hipGetLastError();
}

}  // namespace gpa
