// Device-side helpers shared by the gfx950 kernels of libgpa.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gpa_launch.h"

namespace gpa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// FP32 log2(e), rounded to FP32.
constexpr float kLog2e = 1.44269504088896340736f;

// Tile geometry shared by the MFMA kernels.  A wave owns 16 or 32 rows of its
// operand (queries in the forward and the query-major backward, keys in the
// key-major backward); a workgroup has 4 waves (the d = 128 query-major pass,
// 8).
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kTile = 64;  // rows per workgroup tile and per streamed tile

__device__ __forceinline__ f32x4 mfma_16x16x32(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 ld_b128(const uint16_t* p) {
    return *reinterpret_cast<const bf16x8*>(p);
}

// Two 8-byte reads joined into one MFMA operand: elements 0..3 from p0 and
// 4..7 from p1.
__device__ __forceinline__ bf16x8 ld_b64x2(const uint16_t* p0, const uint16_t* p1) {
    bf16x4 a = *reinterpret_cast<const bf16x4*>(p0);
    bf16x4 b = *reinterpret_cast<const bf16x4*>(p1);
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

typedef __bf16 bf16v4_t __attribute__((__vector_size__(8)));
typedef __attribute__((address_space(3))) bf16v4_t lds_bf16v4_t;

// LDS tiles hold 64 rows x D BF16 values, row-major without padding, with the
// 16-byte chunks of each row permuted: chunk c of row r lives at chunk
// c ^ swz<D>(r).  The gfx950 LDS has 64 banks of 4 bytes (256 bytes per cycle).
// An 8-byte read is served half a wave at a time, a 16-byte read in quarters
// that are not consecutive lanes: lanes 0-3, 12-15 and 20-27 together, lanes
// 4-11, 16-19 and 28-31 together, and the same in the upper half.  Two read
// patterns hit these tiles, and both have to meet 16 distinct 16-byte groups:
//   * 16-byte reads of chunk 4k + g of row c16 (lane 16 g + c16): the first
//     quarter takes rows 0-3 and 12-15 of an even chunk c and rows 4-11 of chunk
//     c + 1 = c ^ 1, so swz of rows 4-11 has to be closed under ^ 1;
//   * transpose reads of two adjacent chunks from 8 consecutive rows, so swz >> 1
//     has to differ over rows 0-7 and over rows 8-15.
// swz takes row bits 0-2 (d = 64, where two 128-byte rows share a 256-byte line
// and rows of equal parity have to differ: bits 1-2) above row bit 3, with the
// top of them inverted in rows 8-15: rows 8-11 then pair with rows 4-7.  Without
// that inversion the 16-byte reads conflict two ways (SQ_LDS_BANK_CONFLICT 25 to
// 40 % of the LDS cycles); with it the counter reads 0 in every kernel (0.2 to 0.5
// cycles an instruction in the atomic schedule's key pass, whose exchange tiles are
// its own).  Measured
// before and after, us: d = 128 query pass 145 and 138, key pass 181 and 173
// (h16_n4096_d128, gproj); 8560 and 8070, 10920 and 10660 (b8_h32_n8192_d128);
// d = 64 forward 667 and 655, query pass 932 and 920 (h16_n16384_d64); the FP32
// baseline 338 and 316.  swz<D>(r + 16) == swz<D>(r), so tiles can be addressed
// 16 rows at a time.  The staging writes fill whole 256-byte lines.
template <int D>
__device__ __forceinline__ int swz(int r) {
    static_assert(D == 64 || D == 128, "head dimension");
    if constexpr (D == 64)
        return ((((r >> 1) & 3) ^ ((r >> 2) & 2)) << 1) | ((r >> 3) & 1);
    else
        return (((r & 7) ^ ((r >> 1) & 4)) << 1) | ((r >> 3) & 1);
}

// Element offset of (row r, column col) in a swizzled tile; col % 4 == 0.
template <int D>
__device__ __forceinline__ int tile_off(int r, int col) {
    return r * D + (((col >> 3) ^ swz<D>(r)) << 3) + (col & 7);
}

// Raw buffer resource over the `bytes` bytes at `base` (stride 0, the gfx9
// data-format word).  The hardware range-checks every buffer load against
// `bytes`: a load at or beyond it returns zero and touches no memory, so tile
// tails need no clamping or masking of addresses.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// 16-byte buffer load at byte offset `off` (zero beyond the resource).
__device__ __forceinline__ u32x4 buf_ld16(rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// The same raw buffer resource as four words, for inline assembly.
__device__ __forceinline__ i32x4 buf_desc(const void* base, uint32_t bytes) {
    const uint64_t a = (uint64_t)(uintptr_t)base;
    return i32x4{(int32_t)(uint32_t)a, (int32_t)((uint32_t)(a >> 32) & 0xFFFFu), (int32_t)bytes,
                 0x00020000};
}

// 32-bit LDS address of a pointer into a __shared__ array.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)((__attribute__((address_space(3))) const char*)p);
}

// LDS DMA buffer loads (lane L writes 16 or 4 bytes at M0 + 16 L or M0 + 4 L;
// lanes out of the resource's range write zeros).  They are issued as inline
// assembly so that the compiler's wait-count insertion does not see them: its
// alias tracking of LDS DMA targets is imprecise and would wait for every
// outstanding tile load before each LDS read.  The kernels therefore order
// these loads themselves, with explicit vmcnt waits and barriers (volatile
// assembly keeps its place relative to those).  No memory clobber: nothing
// the compiler reads or writes in LDS overlaps an in-flight DMA target, and a
// clobber would pin every LDS read of the step between the pieces of a fill.
// The s_nop covers the M0-write to LDS-DMA hazard.
__device__ __forceinline__ void lds_dma16(i32x4 desc, uint32_t m0, uint32_t voff) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(m0), "v"(voff), "s"(desc));
#else
    (void)desc; (void)m0; (void)voff;
#endif
}
__device__ __forceinline__ void lds_dma4(i32x4 desc, uint32_t m0, uint32_t voff) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(m0), "v"(voff), "s"(desc));
#else
    (void)desc; (void)m0; (void)voff;
#endif
}

// Direct global -> LDS staging of one 64-row tile with the gfx950 LDS DMA load
// (buffer_load_dwordx4 ... lds): lane L of a wave writes 16 bytes at
// M0 + 16 L, so each wave call fills a contiguous 1 KB of the swizzled tile
// and every lane loads the global chunk that the swizzle places in its slot.
// No registers or LDS write instructions are involved; completion is tracked
// by vmcnt.  The resource of a call starts at the tile's first row and ends at
// the tensor's last row, so rows at or beyond N are range-checked away: their
// lanes read nothing and write zeros into their LDS slots (measured with an
// in-bounds probe).  The kernels do not rely on that for correctness: every
// probability of a row or key beyond the problem is exactly 0, and the masked
// steps select (not multiply) the operands that meet those rows.
template <int D, int NTHR = kThreads>
struct TileDma {
    static constexpr int NWAVES = NTHR / 64;
    static constexpr int CALLS = kTile * D * 2 / (NTHR * 16);
    uint32_t voff[CALLS];  // byte offset, inside the tile, of this lane's chunk in call k
    uint32_t lds[CALLS];   // byte offset of this wave's 1 KB block (wave-uniform)

    __device__ __forceinline__ void init(int lane, int wave) {
#pragma unroll
        for (int k = 0; k < CALLS; ++k) {
            const int b = (k * NWAVES + wave) * 1024 + 16 * lane;
            const int r = b / (2 * D);
            const int p = (b - r * 2 * D) / 16;
            voff[k] = (uint32_t)(r * 2 * D + ((p ^ swz<D>(r)) * 16));
            lds[k] = (uint32_t)((k * NWAVES + wave) * 1024);
        }
    }
    // Stage rows [row0, row0 + 64) of the [N, D] tensor at `head` into `dst`.
    // With valid == false nothing is read and the slot is filled with zeros
    // (every lane is then out of range), which keeps the number of
    // vector-memory instructions per step fixed.
    __device__ __forceinline__ void load(const uint16_t* head, uint16_t* dst, int row0, int N,
                                         bool valid = true) const {
        const int r0 = valid ? row0 : 0;
        const i32x4 desc =
            buf_desc(head + (size_t)r0 * D, valid ? (uint32_t)(N - r0) * (2 * D) : 0u);
        const uint32_t base = lds_addr(dst);
#pragma unroll
        for (int k = 0; k < CALLS; ++k) lds_dma16(desc, base + lds[k], voff[k]);
    }
    // Call k alone of load(): lets a kernel spread one tile's loads over a step.
    __device__ __forceinline__ void load_call(const uint16_t* head, uint16_t* dst, int row0, int N,
                                              bool valid, int k) const {
        const int r0 = valid ? row0 : 0;
        const i32x4 desc =
            buf_desc(head + (size_t)r0 * D, valid ? (uint32_t)(N - r0) * (2 * D) : 0u);
        lds_dma16(desc, lds_addr(dst) + lds[k], voff[k]);
    }
};

// Per query tile, the key-major pass reads the tile's row statistics from a
// 512-byte block: 64 log2-scaled LSE values, then 64 values of D (FP32).
constexpr int kStatFloats = 2 * kTile;

// LDS DMA of the statistics one wave needs: its 32 query rows (half `qh` of
// the tile) of log2-LSE and of D, 4 bytes per lane, into the 256 bytes at
// `dst` ([32 log2-LSE][32 D]).  A 4-byte LDS DMA writes lane L at M0 + 4 L, so
// the wave's footprint is exactly those 256 bytes.  valid == false writes
// zeros and reads nothing.
__device__ __forceinline__ void stat_dma(const float* tile_stats, float* dst, int lane, int qh,
                                         bool valid) {
    const i32x4 desc = buf_desc(tile_stats, valid ? kStatFloats * 4 : 0);
    const uint32_t row = (uint32_t)(32 * qh + (lane & 31)) + (lane < 32 ? 0u : (uint32_t)kTile);
    lds_dma4(desc, lds_addr(dst), row * 4u);
}

// s_waitcnt with vmcnt <= VM (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] |
// lgkmcnt[11:8] | vmcnt[5:4] at bits 15:14), lgkmcnt = 0, expcnt untouched.
template <int VM>
__device__ __forceinline__ void wait_vm_lgkm0() {
    static_assert(VM >= 0 && VM < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | ((VM >> 4) << 14));
}

// Where control flow parts or meets right behind matrix products.  A vector
// instruction may touch the registers of a 16x16x32 product eight wait states after
// it at the earliest; the compiler keeps that within a block, but over an edge it has
// been seen to count a branch that is not on the path, and to copy or overwrite them
// one or two states too early (with wrong values in one kernel).  No instruction moves
// over this, and the eight states pass here.
__device__ __forceinline__ void mfma_settle() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7");
    __builtin_amdgcn_sched_barrier(0);
}

// Transposed MFMA operand read straight from a row-major LDS tile X[k][n]
// with the gfx950 LDS transpose load ds_read_b64_tr_b16.  Within each 16-lane
// group, that instruction hands lane j element j of the 4 x 16 block formed by
// the 8-byte reads of lanes 4r+q (row r, columns 4q..4q+3).  Addressing rows
// k0+4g+r and columns n0+4q therefore gives lane (c16, g) the values
// X[k0 + 4g + r][n0 + c16], r = 0..3; a second read 16 rows further down fills
// elements 4..7.  This is the k-layout {4g+r, 16+4g+r} that the 16x16
// accumulator of the preceding product leaves in each lane.
template <int D>
__device__ __forceinline__ bf16x8 ld_tr_operand(const uint16_t* X, int k0, int n0, int c16,
                                                int g) {
    const int row = k0 + 4 * g + (c16 >> 2);
    const uint16_t* p0 = X + tile_off<D>(row, n0 + 4 * (c16 & 3));
    const uint16_t* p1 = p0 + 16 * D;  // row + 16 has the same swizzle
    const bf16x4 a =
        __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16v4_t*)p0));
    const bf16x4 b =
        __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16v4_t*)p1));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ __bf16 to_bf16(float x) { return static_cast<__bf16>(x); }
__device__ __forceinline__ float bf16_to_f32(__bf16 x) { return static_cast<float>(x); }

__device__ __forceinline__ uint16_t bf16_bits(float x) {
    return __builtin_bit_cast(uint16_t, static_cast<__bf16>(x));
}

// Store 4 floats as 4 consecutive BF16 values (8 bytes).
__device__ __forceinline__ void st_bf16x4(uint16_t* p, float a, float b, float c, float d) {
    bf16x4 v;
    v[0] = to_bf16(a); v[1] = to_bf16(b); v[2] = to_bf16(c); v[3] = to_bf16(d);
    *reinterpret_cast<bf16x4*>(p) = v;
}

// BF16 halves of a packed 32-bit word, widened exactly to FP32.
__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// 16-byte load of row `row` at column `col` of a [N, D] tensor whose buffer
// resource `r` covers exactly its N rows: rows at or beyond N read as zero.
template <int D>
__device__ __forceinline__ u32x4 ld_row16(rsrc_t r, int row, int col) {
    return buf_ld16(r, (uint32_t)(row * D + col) * 2u);
}

// MFMA A operand whose row 0 is all ones and rows 1..15 zero: multiplying it
// into a B operand gives the column sums of B in accumulator row 0.
__device__ __forceinline__ bf16x8 ones_row0(int c16) {
    const __bf16 v = (c16 == 0) ? (__bf16)1.0f : (__bf16)0.0f;
    bf16x8 a;
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = v;
    return a;
}

// Reductions over the four 16-lane rows of a wave (lanes c16, c16 + 16,
// c16 + 32, c16 + 48), with the gfx950 lane-swap instructions instead of an
// LDS round trip.  v_permlane16_swap on two copies of v leaves rows (0, 0, 2, 2)
// in one copy and (1, 1, 3, 3) in the other; v_permlane32_swap leaves the low
// and the high half.  Combining the two copies therefore gives every lane the
// pairwise result (x ^ 16, then x ^ 32), bitwise the same in both partners
// because max and + are commutative.
__device__ __forceinline__ float xor_max(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const uint32_t w = __float_as_uint(v);
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ __forceinline__ float xor_sum(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const uint32_t w = __float_as_uint(v);
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Workgroup -> (batch*head, tile).  Workgroups are dispatched round-robin over
// the 8 XCDs (each with its own L2), and within an XCD to whichever slots free
// up first.  When B*H is a multiple of 8, XCD x owns heads [x*BH/8, (x+1)*BH/8)
// so one head's tiles share an L2.  Those heads are taken in groups of hg,
// just enough heads for kGroupTiles workgroups (about twice the workgroups an
// XCD holds at once), one group after the other: the tiles in flight then
// stream the data of one or two heads, not of every head of the XCD (which
// would not fit in its L2 at long sequences).  Within a group the order is
// rank-major: every head's heaviest tile, then every head's next heaviest,
// ... , which makes the hardware's in-order dispatch a longest-first greedy
// schedule for any number of resident workgroups.  heavy_high selects which
// end is heavy: the query-major causal kernels' last tiles do the most work,
// the key-major kernels' first tiles do.
//
// resident: the workgroups that a compute unit holds (0: the order as it stands).
// An XCD places its i-th workgroup on unit i mod 32 while it has free slots (i mod
// 256 over the chip where heads are not split over the XCDs), so a grid of no more
// rounds than that is placed before any workgroup finishes, and no later dispatch
// evens the units out.  Its heavy-first list is dealt out like a snake draft: every
// other round, counted from the last one, runs backwards over the units.  The last
// round, which may be partial, then gives its few workgroups to the units that the
// round before gave its lightest ones, and every unit has about the same total work.
// beyond: in larger grids too, the first rounds; the forward and the FP32 baseline
// at d = 64, whose 3 to 5 resident rounds are most of a grid.  In larger grids of the
// others the longest-first order balances by itself (2 per unit and a grid of twice
// that: 5 % slower with the snake), and the backward passes at d = 128 hold one.
//
// Heaviest first alone and with this, us: at d = 128 the forward of 4 heads of 4608,
// 6144, 7680 and 8192 tokens 69.9, 94.4, 119.4 and 131 and 67.4, 91.0, 118.8 and 115,
// 5 heads of 4160 71.0 and 63.8; at d = 64 query pass and key pass of 8 heads of
// 2304, 3072, 3584 and 4096 tokens 26.9 + 31.0, 35.6 + 41.5, 41.5 + 49.1 and 47.5 +
// 56.2 and 25.0 + 29.4, 31.8 + 37.9, 36.7 + 44.1 and 42.7 + 51.0, the forward of 5
// heads of 4160 48.8 and 39.1.
constexpr int kGroupTiles = 128;
__device__ __forceinline__ void map_block(int bid, int BH, int T, bool heavy_high, int* bh,
                                          int* tile, int resident = 0, bool beyond = false) {
    int heads = BH, base = 0, li = bid, shift = 8;  // a round of all 256 units
    if ((BH & 7) == 0) {
        heads = BH >> 3;
        base = (bid & 7) * heads;
        li = bid >> 3;
        shift = 5;  // of an XCD's 32
    }
    if (resident > 0) {
        const int last = (heads * T - 1) >> shift, q = li >> shift;
        const bool back = last < resident ? ((last - q) & 1) != 0
                                          : beyond && (q & 1) && q < resident;
        if (back) li ^= (1 << shift) - 1;  // the same round, backwards
    }
    const int hg = min(heads, max(1, (kGroupTiles + T - 1) / T));
    const int group = li / (hg * T);
    const int first = group * hg;
    const int gs = min(hg, heads - first);  // the last group may be smaller
    const int within = li - group * hg * T;
    const int rank = within / gs;
    *bh = base + first + (within - rank * gs);
    *tile = heavy_high ? (T - 1 - rank) : rank;
}

// Workgroup -> (problem, tile) for packed sequences of unequal lengths, where
// map_block's contiguous blocks of problems would give a whole long sequence to
// one or two XCDs.  Query heads are split over the XCDs instead when Hq is a
// multiple of 8 (XCD x takes heads [x Hq/8, (x+1) Hq/8) of every sequence, so
// the XCDs carry equal work whatever the lengths and heads that share K and V
// mostly share an L2); otherwise the heads rotate from one tile to the next,
// which spreads every sequence over the XCDs.  Tiles are taken by the steps they
// have left (a sequence with Ts tiles has one with each of Ts, Ts - 1, ..., 1
// steps), most first across sequences: heavy_high: the last tile is the heaviest
// (query-major, causal); otherwise the first one is (key-major, causal) or all
// weigh the same.  The sequences are taken in groups of about kPackedTiles
// workgroups per XCD: a group this size ends with a tail of a few per cent, and
// bounds the number of heads whose K and V stream at the same time.
//
// With kPackedCompact sequences or fewer, lane s holds the tile count of sequence
// s and a binary search over the steps left finds the k-th tile of the group's
// order, so the grid needs about one workgroup per tile (packed_grid; those left
// over, at most one per sequence and head, exit).  With more, every sequence has
// as many places as the longest one, and workgroups whose sequence has no such
// tile exit: 1000 exits cost a pass about 4 us.  Returns false where there is no
// tile.
//
// Measured, forward + query pass + key pass: 12 sequences of 243 to 2431 tokens,
// 16 query heads on 4, d = 128: 1453 us with map_block, 574 us with a place for
// every tile of the longest sequence (groups of 128 workgroups 27 % slower, one
// group 12 %), 552 us with this; the same on 4 heads 177 and 155; 16 sequences of
// 500 to 7904 tokens, 32 heads on 8: 24.5, 8.08 and 7.83 ms; seven runs of 8192
// and one of 8000, 32 heads: 25.0, 24.0 and 24.3 ms (37.9 in one group, where
// every head's K and V stream at once and miss in L2).
constexpr int kPackedTiles = 512;

// Sum over the 64 lanes, in every lane: rotations within the rows of 16 lanes,
// then the row and half swaps of xor_sum.
__device__ __forceinline__ int wave_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true);  // row_ror:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, true);  // row_ror:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, true);  // row_ror:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, true);  // row_ror:1
    const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    v = (int)(a[0] + a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return __builtin_amdgcn_readfirstlane((int)(b[0] + b[1]));
}

__device__ __forceinline__ bool map_packed(int bid, int BH, int Hq, int Nmax, const int* cu,
                                           int total, bool heavy_high, int* bh, int* tile) {
    const int nseq = BH / Hq;
    const int T = (Nmax + kTile - 1) / kTile;
    const bool by_head = (Hq & 7) == 0;
    const int per = by_head ? Hq >> 3 : Hq;  // heads of a place in one list
    const int li = by_head ? bid >> 3 : bid;
    const int tiles = by_head ? kPackedTiles : 8 * kPackedTiles;
    const int gseq = (tiles + T * per - 1) / (T * per);  // sequences of a group
    int k = li / per;                                    // place in the list of tiles
    int h = li - k * per;
    h = by_head ? (bid & 7) * per + h : (h + k) % per;
    if (nseq > kPackedCompact) {
        // places [group][steps left][sequence]
        const int group = k / (gseq * T);
        const int first = group * gseq;
        const int gs = min(gseq, nseq - first);
        const int within = k - first * T;
        const int r = within / gs;
        const int s = first + (within - r * gs);
        const int x = min(max(cu[s], 0), total);
        const int n = min(min(max(cu[s + 1], x), total) - x, Nmax);
        const int Ts = (n + kTile - 1) / kTile;
        *bh = s * Hq + h;
        *tile = heavy_high ? T - 1 - r : Ts - T + r;
        return T - r <= Ts;
    }
    const int lane = threadIdx.x & 63;
    int Ts = 0;
    if (lane < nseq) {
        const int x = min(max(cu[lane], 0), total);
        const int n = min(min(max(cu[lane + 1], x), total) - x, Nmax);
        Ts = (n + kTile - 1) / kTile;
    }
    int t = 0, first = 0;
    for (; first < nseq; first += gseq) {
        t = lane >= first && lane < first + gseq ? Ts : 0;
        const int sum = wave_sum(t);
        if (k < sum) break;
        k -= sum;
    }
    if (first >= nseq) return false;
    // the most steps left, `lo`, that more than k tiles have or exceed
    int lo = 1, hi = T;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (wave_sum(max(t - mid + 1, 0)) > k) lo = mid;
        else hi = mid - 1;
    }
    k -= wave_sum(max(t - lo, 0));
    const uint64_t with = __builtin_amdgcn_ballot_w64(t >= lo);
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(with >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)with, 0));
    const uint64_t mine = __builtin_amdgcn_ballot_w64(t >= lo && rank == k);
    const int s = __builtin_ctzll(mine);
    *bh = s * Hq + h;
    *tile = heavy_high ? lo - 1 : __builtin_amdgcn_readlane(Ts, s) - lo;
    return true;
}

// Asks for the offsets' pointers with the first kernel arguments.  Left alone, the
// compiler may load them only where seq_rows reads them, one more trip to memory in
// front of everything else (0.3 to 0.4 us of a pass).  Uneven packs need them first
// anyway (and the query pass of 12 sequences, d = 128, was 2 % slower with this).
__device__ __forceinline__ void offsets_early(const int* cu, const int* cu_k) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : : "s"(cu), "s"(cu_k));
#else
    (void)cu; (void)cu_k;
#endif
}

// Rows of one attention problem (a query head of one sequence) and its query
// and key counts.  Dense batches ([B, H, N, d], cu == nullptr): query head
// bh = b * Hq + h starts at row bh * N of Q and reads key/value head bh / G;
// nq = nk = N.  Packed sequences (query-side tensors [H, total, d], key-side
// [H, total_k, d]): bh = s * Hq + h is head h over queries [cu[s], cu[s + 1])
// and keys [cu_k[s], cu_k[s + 1]); the offsets are clamped to the tensors and
// the counts to the longest runs, so malformed offsets cannot address rows
// outside the tensors.  With causal masking query i sees key j iff
// j <= i + (nk - nq): the diagonal is aligned at the last query and key.
struct SeqRows {
    size_t q0;   // first row of the query-head tensors (Q, O, dO, dQ; LSE, row statistics)
    size_t kv0;  // first row of the key/value-head tensors (K, V, dK, dV)
    size_t p0;   // first row of this query head's key-side FP32 partials (grouped heads)
    int nq;      // queries of this problem
    int nk;      // keys of this problem
};
__device__ __forceinline__ SeqRows seq_rows(const int* cu, const int* cu_k, int bh, int Nq_max,
                                            int Nk_max, int G, int Hq, int total, int total_k) {
    if (cu == nullptr)
        return {(size_t)bh * Nq_max, (size_t)(bh / G) * Nq_max, (size_t)bh * Nq_max, Nq_max,
                Nq_max};
    const int s = bh / Hq, h = bh - s * Hq;
    const int a = min(max(cu[s], 0), total);
    const int b = min(max(cu[s + 1], a), total);
    const int ak = min(max(cu_k[s], 0), total_k);
    const int bk = min(max(cu_k[s + 1], ak), total_k);
    return {(size_t)h * total + a, (size_t)(h / G) * total_k + ak, (size_t)h * total_k + ak,
            min(b - a, Nq_max), min(bk - ak, Nk_max)};
}

// Floor division by a positive divisor, also for negative numerators.
__device__ __forceinline__ int floor_div(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

// Key tiles of a 64-query tile: keys [0, 64 * nkv) hold every key a query of
// the tile can see, and tiles [nplain, nkv) need masks (at most two: the
// causal diagonal crosses at most two key tiles, and the key tail).
struct KeyRange {
    int nkv, nplain;
};
__device__ __forceinline__ KeyRange key_range(int qtile, int Nk, int off, int causal) {
    const int kv_end = causal ? min(max((qtile + 1) * kTile + off, 0), Nk) : Nk;
    const int nkv = (kv_end + kTile - 1) / kTile;
    // fully visible tiles: every key <= the first query's last visible key, and
    // no key beyond Nk
    const int nfull = causal ? floor_div(qtile * kTile + off + 1, kTile) : Nk / kTile;
    return {nkv, max(0, min(min(nfull, Nk / kTile), nkv))};
}

// Target waves per SIMD of each MFMA kernel (build-time tuning constants).
#ifndef GPA_FWD_OCC
#define GPA_FWD_OCC 2
#endif
#ifndef GPA_FWD16_OCC
#define GPA_FWD16_OCC 4
#endif
#ifndef GPA_DQ_OCC64
#define GPA_DQ_OCC64 2
#endif
#ifndef GPA_DKDV_OCC64
#define GPA_DKDV_OCC64 2
#endif

}  // namespace gpa
