// FlashAttention forward for gfx950 with a selectable K/V scan order (cyclic or sawtooth).
//
// One workgroup = 4 wavefronts = one 128-row query tile (paper Sec. 2.2, Alg. 1); wavefront w owns
// query rows 32w..32w+31 of the tile and keeps them in registers for the whole inner loop.  K and V
// are streamed in 64-row tiles through two LDS buffers each, filled by direct global->LDS loads.
//
// Three kernels do this.  They share the transposed form of both contractions
//     S^T (kv x q) = K_j   (kv x d) . Q_i^T (d x q)
//     O^T (d  x q) = V_j^T (d x kv) . P^T   (kv x q)
// because the accumulator layout of S^T is then, register for register, the B-operand layout of the second
// product, so P never leaves registers.  V^T in the matching A-operand layout comes from ds_read_b64_tr_b16, which
// hands lane i of a 16-lane group the column i of a 4 x 16 block whose four row addresses are supplied by lanes
// 4e + c (row e, 8-byte column chunk c) of that group.  The workgroups of one XCD walk the same head together and
// re-align between heads (domain_sync).
//
// attn_fwd_kernel (pipelined_range, general_range), for workgroups that have a compute unit to themselves: both
// contractions on v_mfma_f32_32x32x16.  A lane holds, for its query column lane%32, the kv rows
// 8*(r/4) + 4*(lane/32) + r%4 of a 32-row block in register r; the contraction index of each 16-wide step of the second
// product is read as  slot (lane/32, e) <-> kv = 16*step + 8*(e/4) + 4*(lane/32) + e%4.  Softmax statistics live per
// lane: lanes l and l+32 share a query row and hold disjoint key subsets, so the running maximum is merged across the
// pair every tile while the running sum stays a per-lane partial (it is linear) and is merged once in the epilogue.  A
// query tile's scan is a software-pipelined run of full, unmasked K/V tiles (pipelined_range) plus, at one end, a short
// run of masked tiles (general_range).  With 64-row tiles it walks the two halves of a scan at once (HALVES), short scans
// with everything in one pipeline (scan_halves).
//
// attn_fwd_shared_kernel (scan_tiles), 128-row tiles where workgroups share the compute units: both contractions on
// v_mfma_f32_16x16x32, layouts as described there.  Four lanes share a query row, row sums are a product with ones,
// the running maximum is compared on raw scores, and masked tiles stay in the pipeline.
//
// attn_fwd_kernel with 256-row tiles, head dimension 128 (NH = 2 in its template, scan_tiles_wide): the same with 64 query rows per
// wavefront and one workgroup per CU, so that every K / V^T fragment read from LDS feeds four MFMAs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <type_traits>
#include <utility>

#include "running_max.h"
#include "sawattn.h"
#include "schedule.h"

// Scratch memory of attn_fwd_static (the entry point that may not allocate): binary16 copies of K and V.
// In host code this name is only a handle for hipGetSymbolAddress, never an address.
static __device__ __align__(256) unsigned char scratch[SAWATTN_STATIC_SCRATCH_BYTES];

namespace sawattn {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef unsigned u8 __attribute__((ext_vector_type(8)));
typedef _Float16 h16 __attribute__((ext_vector_type(16)));
typedef unsigned u16v __attribute__((ext_vector_type(16)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));

#define LDS_PTR(T) __attribute__((address_space(3))) T*

struct Params {
    const void* Q;
    const void* K;
    const void* V;
    void* O;
    int32_t* trace;        // optional: [grid][max_local][4]
    int32_t* trace_count;  // optional: [grid]
    int N;
    int o_dtype;
    int sawtooth;
    int negate_q;          // scale < 0: use -Q and |scale|
    int q_bf16;            // wide variant on converted inputs: Q is still bfloat16 (K and V are binary16 copies)
    int stream_o;          // O leaves through LDS as whole lines, non-temporal (variant.qo_streaming)
    int stream_q;          // Q arrives through LDS as whole lines, non-temporal
    int max_local;
    int ticket_set;        // which set of arrival counters this launch uses (domain_sync)
    float c;               // |scale| * log2(e): scores are handled in the log2 domain
    Schedule sched;
};

// LDS tile layout.  A tile is 64 rows of D 16-bit elements, rows packed back to back (no padding, so
// that one wavefront-wide direct global->LDS load, which writes 64 x 16 contiguous bytes, fills whole
// rows).  Inside a row the 16-byte chunks are permuted: chunk cc of row r sits at chunk position
// cc ^ swz(r).  swz is chosen so that both read patterns are free of bank conflicts:
//   * K operand: 16 lanes read the same chunk of 16 consecutive rows          -> swz distinct over them
//   * V operand (ds_read_b64_tr_b16): 32 lanes read 4 consecutive rows x 64 B -> the rows land in
//     four different 64-byte bank groups.
template <int D>
struct Geo {
    static constexpr int kRowBytes = D * 2;
    static constexpr int kChunksPerRow = D / 8;                       // 16-byte chunks per row
    static constexpr int kTile = kTileKV * kRowBytes;                 // one K or V tile in LDS
    static constexpr int kRowsPerWaveLoad = 1024 / kRowBytes;         // rows one 64-lane x 16 B load covers
    static constexpr int kLoadsPerWave = kTile / 1024 / (kThreads / 64);
    static constexpr int kLdsBytes = 4 * kTile;                       // K0 K1 V0 V1
    __device__ static __forceinline__ int swz(int row) {
        if constexpr (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
        else return ((row & 2) << 1) | ((row >> 2) & 3);              // u = row>>1: (u&1)<<2 | (u>>1)&3
    }
};

template <bool BF16>
__device__ __forceinline__ f16v mfma_16bit(u4 a, u4 b, f16v c) {
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// Eight bfloat16 -> eight binary16 (round to nearest even; exact for normal binary16 magnitudes).
__device__ __forceinline__ u4 bf16x8_to_f16x8(u4 w) {
    u4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f2 x;
        x[0] = __builtin_bit_cast(float, w[i] << 16);
        x[1] = __builtin_bit_cast(float, w[i] & 0xffff0000u);
        r[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(x, h2));
    }
    return r;
}

// Compile-time loop: f(std::integral_constant<int, I>) for I in [0, N).
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl<N>(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

// Lane-constant addresses, computed once per kernel.
//
// Tile fill: wavefront w, load i covers LDS bytes [(i*4 + w) * 1024, +1024) of a tile: lane l
// writes chunk position l % CPR of row (i*4+w)*rows_per_load + l / CPR and therefore fetches source
// chunk (l % CPR) ^ swz(row) of that row.
// K operand (S^T = K Q^T): lane reads chunk 2*ks + g of rows ln and 32 + ln (same swz for both).
// V operand (ds_read_b64_tr_b16): source lane 4e + c of a 16-lane group addresses row e, 8-byte
// column chunk c of the 4 x 16 block whose columns the lanes of the group receive; the rows are
// kv = 16*ks + 8*h + 4*g + e, so that the contraction slots line up with the registers of P^T.
template <int D>
struct LaneMap {
    using G = Geo<D>;
    unsigned fill_src[G::kLoadsPerWave];   // row * row_bytes + byte offset of the source chunk
    unsigned fill_dst;                     // wave * 1024 (+ i * 4096): LDS byte offset inside the tile
    unsigned k_rd[D / 16];                 // byte offset inside a K tile, MFMA step ks, rows ln (+32 rows: +32*row_bytes)
    unsigned v_rd[D / 32][2];              // byte offset inside a V tile for [db][h], kv step 0 (+ks: +16*row_bytes*ks)
    __device__ __forceinline__ LaneMap(int wave, int lane) {
        const int g = lane >> 5, ln = lane & 31;
#pragma unroll
        for (int i = 0; i < G::kLoadsPerWave; ++i) {
            const int r = (i * 4 + wave) * G::kRowsPerWaveLoad + lane / G::kChunksPerRow;
            fill_src[i] = r * G::kRowBytes + ((lane % G::kChunksPerRow) ^ G::swz(r)) * 16;
        }
        fill_dst = wave * 1024;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) k_rd[ks] = ln * G::kRowBytes + ((2 * ks + g) ^ G::swz(ln)) * 16;
        const int vrow = 4 * g + ((lane & 15) >> 2);
        const int chunk = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
        const int half = (lane & 1) * 8;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = vrow + 8 * h;     // swz(r + 16*ks) == swz(r)
                v_rd[db][h] = r * G::kRowBytes + ((4 * db + chunk) ^ G::swz(r)) * 16 + half;
            }
    }
};

// One 64-lane x 16-byte direct global -> LDS load: lane l's 16 bytes from base + voff land at LDS
// byte address lds_addr + 16*l.  Issued as inline assembly so that the compiler does not treat every
// later LDS read as depending on it (it would wait for the whole next tile before reading the
// current one); the landing is awaited explicitly with wait_tile_landed() before the barrier that
// publishes the tile.
__device__ __forceinline__ void load_to_lds_16B(const char* base, unsigned voff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
}
// The same marked non-temporal: data read once (a Q tile) that should not take the place of K/V tiles in the L2.
__device__ __forceinline__ void load_to_lds_16B_nt(const char* base, unsigned voff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :: "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
}
// The same with the LDS address given as a scalar base plus a compile-time offset (one scalar add into M0).
template <int LDS_IMM>
__device__ __forceinline__ void load_to_lds_16B_at(const char* base, unsigned voff, unsigned lds_base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(voff), "s"(base), "n"(LDS_IMM) : "memory", "m0", "scc");
}
// The same in two steps, for several loads into neighbouring places: where the first of them goes, and a load.  The offset AT of the instruction
// counts on both sides: 16 bytes from base + voff + AT land at lds_addr + AT + 16*l.  Nothing else in the kernels writes M0.
__device__ __forceinline__ void aim_lds(unsigned lds_addr) { asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" :: "s"(lds_addr) : "memory", "m0"); }
template <int AT>
__device__ __forceinline__ void load_aimed_16B(const char* base, unsigned voff) {
    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" :: "v"(voff), "s"(base), "n"(AT) : "memory");
}
__device__ __forceinline__ void wait_tile_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Per-lane byte offsets (relative to the head's base) of this lane's chunks of tile j.  A ragged
// last tile re-reads row N-1 for the rows beyond N: always valid memory and finite data; such
// keys are masked before use.
template <int D>
__device__ __forceinline__ void tile_offsets(int j, int N, const LaneMap<D>& lm, unsigned (&off)[Geo<D>::kLoadsPerWave]) {
    using G = Geo<D>;
    const int kv0 = j * kTileKV;
    if (kv0 + kTileKV <= N) {
#pragma unroll
        for (int i = 0; i < G::kLoadsPerWave; ++i) off[i] = lm.fill_src[i];
    } else {
#pragma unroll
        for (int i = 0; i < G::kLoadsPerWave; ++i) {
            const unsigned row = lm.fill_src[i] / G::kRowBytes, chunk = lm.fill_src[i] % G::kRowBytes;
            unsigned r = kv0 + row;
            r = r < (unsigned)N ? r : (unsigned)N - 1;
            off[i] = (r - kv0) * G::kRowBytes + chunk;   // (r >= kv0: tile j exists, so its first row is below N)
        }
    }
}

// Direct global -> LDS copy of tile j of a head into the tile at LDS byte address dst.
template <int D>
__device__ __forceinline__ void tile_to_lds(const char* head, int j, const unsigned (&off)[Geo<D>::kLoadsPerWave],
                                            const LaneMap<D>& lm, unsigned dst) {
    using G = Geo<D>;
    const char* base = head + (size_t)j * kTileKV * G::kRowBytes;
#pragma unroll
    for (int i = 0; i < G::kLoadsPerWave; ++i) load_to_lds_16B(base, off[i], dst + lm.fill_dst + i * 4096);
}

// Register path for V in bfloat16 (converted to binary16 before it reaches LDS).
template <int D>
__device__ __forceinline__ void tile_to_regs(const char* head, int j, const unsigned (&off)[Geo<D>::kLoadsPerWave],
                                             u4 (&reg)[Geo<D>::kLoadsPerWave]) {
    using G = Geo<D>;
    const char* base = head + (size_t)j * kTileKV * G::kRowBytes;
#pragma unroll
    for (int i = 0; i < G::kLoadsPerWave; ++i) reg[i] = *reinterpret_cast<const u4*>(base + off[i]);
}
template <int D>
__device__ __forceinline__ void regs_to_lds_f16(const u4 (&reg)[Geo<D>::kLoadsPerWave], const LaneMap<D>& lm, int lane,
                                                LDS_PTR(char) dst) {
    using G = Geo<D>;
#pragma unroll
    for (int i = 0; i < G::kLoadsPerWave; ++i)
        *(LDS_PTR(u4))(dst + lm.fill_dst + i * 4096 + lane * 16) = bf16x8_to_f16x8(reg[i]);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Exchange between the lanes l and l^32, the two lanes that share a query row.  v_permlane32_swap
// swaps the upper 32 lanes of its first operand with the lower 32 lanes of its second; starting
// from two copies of x this leaves (lower half of x everywhere, upper half of x everywhere).
__device__ __forceinline__ void lane_pair(float x, float& lower, float& upper) {
    unsigned a = __builtin_bit_cast(unsigned, x), b = a;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    lower = __builtin_bit_cast(float, a);
    upper = __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float pair_max(float x) {
    float lo, hi;
    lane_pair(x, lo, hi);
    return fmaxf(lo, hi);
}
__device__ __forceinline__ float pair_sum(float x) {
    float lo, hi;
    lane_pair(x, lo, hi);
    return lo + hi;
}

// Row sums of the rounded probabilities on the matrix cores: a sparse product with ones, 64 keys x 16 columns in one v_smfmac_f32_16x16x64, which
// takes the 16 cycles of a 16x16x32.  Of each four neighbouring halves of the second operand a row of the first takes two; even rows
// take the first two, odd rows the last two, so a column's sum is that of an even and an odd row.  Accumulated in binary32 like the products.
struct SparseOnes {
    u4 one;       // the values of this lane's row of the first operand, row lane % 16
    int pick;     // which halves they meet, two bits each
};
__device__ __forceinline__ SparseOnes sparse_ones(int lane, unsigned one) {
    SparseOnes s;
    s.one = u4{one, one, one, one};
    asm volatile("" : "+v"(s.one));      // (or the compiler makes them anew in every iteration)
    s.pick = lane & 1 ? (int)0xeeeeeeee : 0x44444444;
    asm volatile("" : "+v"(s.pick));
    return s;
}
constexpr unsigned kOnes = 0x3c003c00u;      // binary16 1.0, twice
__device__ __forceinline__ f4 sparse_sum(const SparseOnes& ones, const u8& p, f4 acc) {
    return __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, ones.one), __builtin_bit_cast(h16, p), acc, ones.pick, 0, 0);
}
// The same with 32 columns, second operands in the layout of 32x32x16 and the sum of a column in acc[0] + acc[1] of both lanes that hold it: two per
// tile in place of two mixed-precision additions per pair, which took a tenth of pipelined_range's issue slots (4 x 4096, d = 64 26.5 -> 25.4 us,
// 1 x 16384, d = 64, causal 88.0 -> 83.8, 2 x 4096, d = 128 35.8 -> 35.0), or of four plain products (8 x 2048, d = 64, causal 14.9 -> 14.6).  (Half the
// time would do with 16 columns and zeros against the others' values, but 0 times an infinity or no number is no number: query rows would mix.)
__device__ __forceinline__ f16v sparse_sum_32(const SparseOnes& ones, const u8& p, f16v acc) {
    return __builtin_amdgcn_smfmac_f32_32x32x32_f16(__builtin_bit_cast(h8, ones.one), __builtin_bit_cast(h16, p), acc, ones.pick, 0, 0);
}
// Probabilities of 64 keys x 16 N query rows as second operands: part kh, qt = keys 32kh..32kh+31 of the rows 16qt.. .  Sparse sums want the two parts of
// some rows in eight registers in a row; for plain sums they lie apart, which is easier to find registers for.
template <bool SPARSE, int N>
struct Probabilities {
    u8 v[N];
    __device__ __forceinline__ void set(int kh, int qt, int word, unsigned x) { v[qt][4 * kh + word] = x; }
    __device__ __forceinline__ u4 part(int kh, int qt) const { return kh ? __builtin_shufflevector(v[qt], v[qt], 4, 5, 6, 7) : __builtin_shufflevector(v[qt], v[qt], 0, 1, 2, 3); }
    __device__ __forceinline__ void pin() {      // nothing that writes them moves behind this, nothing that reads them ahead of it
#pragma unroll
        for (int qt = 0; qt < N; qt += 2) asm volatile("" : "+v"(v[qt]), "+v"(v[qt + 1]));
    }
};
template <int N>
struct Probabilities<false, N> {
    u4 v[2][N];
    __device__ __forceinline__ void set(int kh, int qt, int word, unsigned x) { v[kh][qt][word] = x; }
    __device__ __forceinline__ u4 part(int kh, int qt) const { return v[kh][qt]; }
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int qt = 0; qt < N; qt += 2) asm volatile("" : "+v"(v[0][qt]), "+v"(v[0][qt + 1]), "+v"(v[1][qt]), "+v"(v[1][qt + 1]));
    }
};
__device__ __forceinline__ u4 half_of(const u8& p, int hi) {
    return hi ? __builtin_shufflevector(p, p, 4, 5, 6, 7) : __builtin_shufflevector(p, p, 0, 1, 2, 3);
}

// Adds the two binary16 values of `ph` to two float partial sums (one mixed-precision FMA each: exact, and cheaper in
// the instruction stream than the two-element dot product).  `one` is binary16 1.0 held in a register the compiler
// cannot see through (opaque_one()): the widened products then become v_fma_mix_f32.  Written in C and not as inline
// assembly because the compiler separates dependent assembly statements that have nothing in between by a no-op each.
__device__ __forceinline__ _Float16 opaque_one() {
    _Float16 one = (_Float16)1.0f;
    asm volatile("" : "+v"(one));
    return one;
}
__device__ __forceinline__ void add_pair(float& sum_lo, float& sum_hi, h2 ph, _Float16 one) {
    sum_lo = __builtin_fmaf((float)ph[0], (float)one, sum_lo);
    sum_hi = __builtin_fmaf((float)ph[1], (float)one, sum_hi);
}

// A wavefront's running row sums in pipelined_range.  of_lane(): a lane's part of its row's sum, which the lanes that share the row add up to.
// Sparse products take 21 registers and two places among the MFMAs of a tile, additions three registers and 32 places of the vector unit's.  Products
// on 64-row tiles (see sparse_sum_32), but for d = 128, bfloat16 in the kernel of full even scans, whose start took 0.25 us more (2 x 128 8.0 -> 8.2, 5 x 256
// 9.4 -> 9.7 us) and whose tiles only 0 to 1 % less; on 128-row tiles where they gain and fit: d = 128, binary16, causal, from additions -0.3 % in the mean of
// 51 launches (-1.6 to +1.4 %; 1 x 20000 240.7 -> 237.7 us).  Additions elsewhere: d = 128 without a mask, where the matrix pipe is the busier one, products take up to 1.6 % more (1 x 32768
// 534 -> 543 us), and with bfloat16 they spill; d = 64 has 168 registers, and 40 to 60 bytes of scratch per lane cost short scans 1 to 11 % (128 x 256
// 7.6 -> 8.5 us, 64 x 512 9.9 -> 10.6).  (With 256 registers products take up to 5 % less there, 16 x 2000 25.9 -> 25.0 us, but two workgroups
// to a compute unit in place of three slow down launches on three streams: 16 x 2000 18.7 -> 20.0 us each, bfloat16 19.6 -> 21.4.)
template <bool SPARSE>
struct RowSums {
    SparseOnes ones;
    f16v sum;
    __device__ __forceinline__ explicit RowSums(int lane) : ones(sparse_ones(lane, (lane & 3) < 2 ? kOnes : 0u)) {
        sum = f16v{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void add(const u8& p) { sum = sparse_sum_32(ones, p, sum); }
    __device__ __forceinline__ void scale(float alpha) { sum *= alpha; }
    __device__ __forceinline__ float of_lane() const { return 0.5f * (sum[0] + sum[1]); }      // (both lanes of a pair hold the row's sum)
};
template <>
struct RowSums<false> {
    _Float16 one = opaque_one();
    float lo = 0.f, hi = 0.f;
    __device__ __forceinline__ explicit RowSums(int) {}
    __device__ __forceinline__ void add(h2 p) { add_pair(lo, hi, p, one); }
    __device__ __forceinline__ void scale(float alpha) { lo *= alpha; hi *= alpha; }
    __device__ __forceinline__ float of_lane() const { return lo + hi; }
};

// Per-wavefront state of one query tile that the K/V loop carries along.
template <int D>
struct TileState {
    u4 qf[D / 16];      // Q^T as B operand: lane holds Q[qrow][16*ks + 8*g .. +7]
    f16v o[D / 32];     // O^T accumulator
    float M;            // reference maximum of score*c (log2 domain), same in both lanes of a pair
    float L;            // this lane's partial running sum
};

// This lane's LDS read addresses for the K/V buffer pair in use; flipped to the other pair after
// every iteration.
template <int D>
struct ReadAddr {
    unsigned k[D / 16];       // K operand, MFMA step ks, row ln (+32 rows: +32*row_bytes)
    unsigned v[D / 32][2];    // V operand [db][h], kv step 0 (+ks: +16*row_bytes*ks)
    __device__ __forceinline__ void flip(int delta) {
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) k[ks] += delta;
#pragma unroll
        for (int db = 0; db < D / 32; ++db) { v[db][0] += delta; v[db][1] += delta; }
    }
};

// One K/V tile for one wavefront out of the LDS buffers `ra` points at: S^T = K Q^T, softmax
// update, O^T += V^T P^T.
template <int D, bool BF16, bool CAUSAL, bool MASKED>
__device__ __forceinline__ void compute_tile(TileState<D>& st, const ReadAddr<D>& ra, float c, int kv0, int qrow, int lane,
                                             int N) {
    using G = Geo<D>;
    constexpr int KS = D / 16, DB = D / 32;
    const int g = lane >> 5;
    // ---- S^T = K_j Q_i^T : two 32(kv) x 32(q) blocks; operands fetched two steps ahead
    f16v s[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[0][r] = 0.f; s[1][r] = 0.f; }
    {
        u4 a[KS][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            a[ks][0] = *(LDS_PTR(u4))(size_t)(ra.k[ks]);
            a[ks][1] = *(LDS_PTR(u4))(size_t)(ra.k[ks] + 32 * G::kRowBytes);
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 2 < KS) {
                a[ks + 2][0] = *(LDS_PTR(u4))(size_t)(ra.k[ks + 2]);
                a[ks + 2][1] = *(LDS_PTR(u4))(size_t)(ra.k[ks + 2] + 32 * G::kRowBytes);
            }
            s[0] = mfma_16bit<BF16>(a[ks][0], st.qf[ks], s[0]);
            s[1] = mfma_16bit<BF16>(a[ks][1], st.qf[ks], s[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // ---- mask: keys at or beyond N, and keys after the query under the causal mask, get the score -inf, which
    //      c > 0 turns into the probability 0.  Register r of block b is key 32b + 8(r/4) + 4g + r%4 of the tile:
    //      visible up to the offset `ahead` (one comparison and one select per score).
    if constexpr (MASKED) {
        const int last_key = CAUSAL ? (qrow < N - 1 ? qrow : N - 1) : N - 1;
        const int ahead = last_key - kv0 - 4 * g;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (32 * b + 8 * (r >> 2) + (r & 3) > ahead) s[b][r] = -INFINITY;
    }
    // ---- online softmax in the log2 domain
    float mx = s[0][0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[0][r]);
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[1][r]);
    mx = pair_max(mx);
    const float tmax = mx * c;
    if (__builtin_amdgcn_ballot_w64(tmax > st.M + kRescaleSlack) != 0) {
        const float Mnew = fmaxf(st.M, tmax);
        const float alpha = (Mnew == -INFINITY) ? 1.0f : fast_exp2(st.M - Mnew);
        st.M = Mnew;
        st.L *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
    }
    const float Mref = (MASKED && st.M == -INFINITY) ? 0.f : st.M;
    u4 pf[4];
    const h2 ones = {(_Float16)1.0f, (_Float16)1.0f};
    float L = st.L;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 8 * h + 2 * i;
                const float x0 = fast_exp2(__builtin_fmaf(s[b][r], c, -Mref));
                const float x1 = fast_exp2(__builtin_fmaf(s[b][r + 1], c, -Mref));
                const h2 ph = __builtin_convertvector(f2{x0, x1}, h2);
                // running sum of the rounded probabilities, the values the second product uses
                L = __builtin_amdgcn_fdot2(ph, ones, L, false);
                w[i] = __builtin_bit_cast(unsigned, ph);
            }
            pf[2 * b + h] = w;
        }
    st.L = L;
    // ---- O^T += V_j^T P^T : 4 kv steps x DB row blocks; V^T operands fetched AHEAD steps ahead
    {
        constexpr int NSTEP = 4 * DB, AHEAD = 2;
        auto read_a = [&](int idx) -> s8 {
            const int ks = idx / DB, db = idx % DB;
            const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)(ra.v[db][0] + ks * 16 * G::kRowBytes));
            const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)(ra.v[db][1] + ks * 16 * G::kRowBytes));
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        };
        s8 av[NSTEP];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int idx = 0; idx < AHEAD; ++idx) av[idx] = read_a(idx);
#pragma unroll
        for (int idx = 0; idx < NSTEP; ++idx) {
            if (idx + AHEAD < NSTEP) av[idx + AHEAD] = read_a(idx + AHEAD);
            const int ks = idx / DB, db = idx % DB;
            st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, av[idx]), __builtin_bit_cast(h8, pf[ks]),
                                                              st.o[db], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// A run of `count` K/V tiles j_first, j_first + step, ... processed one tile at a time (all with or
// all without the mask code).  Self-contained: fetches its first tile itself and leaves with every
// wavefront past the barrier that follows its last tile.  Iteration `it` uses LDS buffer pair it & 1
// and, while computing, fetches the tile of iteration it+1 into the other pair.
template <int D, bool BF16, bool CAUSAL, bool MASKED>
__device__ __forceinline__ void general_range(TileState<D>& st, const LaneMap<D>& lm, const char* Kh, const char* Vh, int N,
                                              float c, int j_first, int step, int count, int qw0, int qrow, int lane,
                                              LDS_PTR(char) lds, bool idle = false) {
    // idle: this wavefront fetches and keeps the barriers like the others but computes nothing (its rows are another
    // wavefront's in this run)
    using G = Geo<D>;
    if (count <= 0) return;
    const unsigned lds0 = (unsigned)(size_t)lds;
    u4 vreg[G::kLoadsPerWave];   // only used for bfloat16 inputs
    // LDS: K buffers at 0 and kTile, V buffers at 2*kTile and 3*kTile.  Start on pair 0.
    ReadAddr<D> ra;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) ra.k[ks] = lds0 + lm.k_rd[ks];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) { ra.v[db][0] = lds0 + 2 * G::kTile + lm.v_rd[db][0]; ra.v[db][1] = lds0 + 2 * G::kTile + lm.v_rd[db][1]; }
    {
        unsigned off[G::kLoadsPerWave];
        tile_offsets<D>(j_first, N, lm, off);
        tile_to_lds<D>(Kh, j_first, off, lm, lds0);
        if constexpr (BF16) {
            tile_to_regs<D>(Vh, j_first, off, vreg);
            regs_to_lds_f16<D>(vreg, lm, lane, lds + 2 * G::kTile);
        } else {
            tile_to_lds<D>(Vh, j_first, off, lm, lds0 + 2 * G::kTile);
        }
        wait_tile_landed();
        __syncthreads();
    }
#pragma unroll 1
    for (int it = 0; it < count; ++it) {
        const int cur = it & 1;
        const int j = j_first + it * step;
        const bool more = it + 1 < count;
        if (more) {
            unsigned off[G::kLoadsPerWave];
            tile_offsets<D>(j + step, N, lm, off);
            tile_to_lds<D>(Kh, j + step, off, lm, lds0 + (cur ^ 1) * G::kTile);
            if constexpr (BF16) tile_to_regs<D>(Vh, j + step, off, vreg);
            else tile_to_lds<D>(Vh, j + step, off, lm, lds0 + (2 + (cur ^ 1)) * G::kTile);
        }
        const int kv0 = j * kTileKV;
        const bool active = !idle && qw0 < N && (!CAUSAL || kv0 <= qw0 + 31);
        if (active) compute_tile<D, BF16, CAUSAL, MASKED>(st, ra, c, kv0, qrow, lane, N);
        ra.flip(cur ? -G::kTile : G::kTile);
        if (more) {
            if constexpr (BF16) regs_to_lds_f16<D>(vreg, lm, lane, lds + (2 + (cur ^ 1)) * G::kTile);
            wait_tile_landed();
        }
        __syncthreads();
    }
}

// A run of `count` full, unmasked K/V tiles j_first, j_first + step, ..., software pipelined across
// tiles.  While the MFMAs of S(i+1)^T = K(i+1) Q^T run, the exponentials of tile i are issued
// between them; while the MFMAs of O^T += V(i)^T P(i)^T run, the row maximum of S(i+1), the
// lazy-rescale check and the (score*c - M) of tile i+1 are issued between them.  Two register sets
// alternate roles without copies: `A` accumulates the scores of the tile one ahead, `x` holds the
// shifted scores of the current tile until they have become probabilities.  K is therefore fetched
// two tiles ahead and V one tile ahead, still into two LDS buffers each.  For bfloat16 inputs V
// travels global -> registers -> binary16 -> LDS, the conversion spread over the second product.
// Self-contained like general_range().
//
// HALVES: the workgroup walks two runs of `count` tiles at once -- run r = tiles j_first + (r*count + i)*step,
// i = 0..count-1 -- for small problems, where the chip has more compute units than there are query tiles and
// the length of one wavefront's walk is what the launch takes.  All four wavefronts fetch the tiles of both
// runs (a second set of K/V buffers behind the first; for bfloat16 inputs a second set of V registers);
// this wavefront computes on run `run`.
//
// SPARSE: row sums as sparse products instead of additions, see RowSums.
template <int D, bool BF16, bool HALVES = false, bool SPARSE = HALVES>
__device__ __forceinline__ void pipelined_range(TileState<D>& st, const LaneMap<D>& lm, const char* Kh, const char* Vh,
                                                float c, int j_first, int step, int count, int lane, LDS_PTR(char) lds,
                                                int run = 0) {
    using G = Geo<D>;
    constexpr int RUNS = HALVES ? 2 : 1;
    constexpr unsigned kSet = 4 * G::kTile;   // one set of buffers: K0 K1 V0 V1
    constexpr int KS = D / 16, DB = D / 32;
    constexpr int NA = 2 * KS;            // MFMAs of one S^T tile
    constexpr int NB = 4 * DB;            // MFMAs of one O^T update
    constexpr int NL = G::kLoadsPerWave;
    constexpr int EU = 16 / NA;           // exp units (2 exp + convert + sum of one pair) per MFMA of phase A
    if (count <= 0) return;
    const unsigned lds0 = (unsigned)(size_t)lds;
    const f16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    RowSums<SPARSE> sums(lane);      // of the rounded probabilities, the values the second product uses
    f16v A[2];          // S^T of the tile one ahead: block b = keys 32b..32b+31 of the tile
    float x[32];        // score*c - M of the current tile, index 16*b + r
    Probabilities<SPARSE, 2> pf;      // its probabilities as B operands, 16 keys each: part(ks & 1, ks / 2)
    u4 vreg[(HALVES ? 2 : 1) * NL];   // bfloat16 V chunks in flight (BF16 only), run r in vreg[r * NL ...]

    // LDS read addresses: K of the tile one ahead, V of the current tile
    unsigned rk[KS], rv[DB][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rk[ks] = lds0 + run * kSet + lm.k_rd[ks];
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        rv[db][0] = lds0 + run * kSet + 2 * G::kTile + lm.v_rd[db][0];
        rv[db][1] = lds0 + run * kSet + 2 * G::kTile + lm.v_rd[db][1];
    }

    // tile i of run r
    auto tile_base = [&](const char* head, int i, int r = 0) {
        return head + (size_t)(j_first + (r * count + i) * step) * kTileKV * G::kRowBytes;
    };
    auto fetch_burst = [&](const char* head, int i, unsigned dst) {
#pragma unroll
        for (int r = 0; r < RUNS; ++r) {
            const char* base = tile_base(head, i, r);
#pragma unroll
            for (int l = 0; l < NL; ++l) load_to_lds_16B(base, lm.fill_src[l], dst + r * kSet + lm.fill_dst + l * 4096);
        }
    };
    auto k_read = [&](int m) -> u4 { return *(LDS_PTR(u4))(size_t)(rk[m / 2] + (m & 1) * 32 * G::kRowBytes); };
    auto v_read = [&](int idx) -> s8 {
        const int ks = idx / DB, db = idx % DB;
        const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)(rv[db][0] + ks * 16 * G::kRowBytes));
        const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)(rv[db][1] + ks * 16 * G::kRowBytes));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto rescale = [&](float tmax) {
        const float Mnew = fmaxf(st.M, tmax);
        const float alpha = (Mnew == -INFINITY) ? 1.0f : fast_exp2(st.M - Mnew);
        st.M = Mnew;
        st.L *= alpha;
        sums.scale(alpha);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[db][r] *= alpha;
    };
    float tmax_ahead = 0.f;   // row maximum (times c) of the tile in A, from the latest iteration
    // exp unit u (0..15): the two exponentials of pair u, and the convert of pair u-1
    float e0[16], e1[16];
    auto exp_unit = [&](int u) {
        if (u < 16) {
            e0[u] = fast_exp2(x[2 * u]);
            e1[u] = fast_exp2(x[2 * u + 1]);
        }
        if (u >= 1 && u <= 16) {
            const int v = u - 1;
            const h2 ph = __builtin_convertvector(f2{e0[v], e1[v]}, h2);
            if constexpr (!SPARSE) sums.add(ph);
            pf.set(v / 4 & 1, v / 8, v % 4, __builtin_bit_cast(unsigned, ph));
        }
    };

    // ---------------------------------------------------------------- prologue: tile 0
    fetch_burst(Kh, 0, lds0);
    if constexpr (BF16) {
#pragma unroll
        for (int r = 0; r < RUNS; ++r) {
            const char* base = tile_base(Vh, 0, r);
#pragma unroll
            for (int l = 0; l < NL; ++l) vreg[r * NL + l] = *reinterpret_cast<const u4*>(base + lm.fill_src[l]);
        }
#pragma unroll
        for (int r = 0; r < RUNS; ++r)
#pragma unroll
            for (int l = 0; l < NL; ++l)
                *(LDS_PTR(u4))(lds + r * kSet + 2 * G::kTile + lm.fill_dst + l * 4096 + lane * 16) = bf16x8_to_f16x8(vreg[r * NL + l]);
    } else {
        fetch_burst(Vh, 0, lds0 + 2 * G::kTile);
    }
    wait_tile_landed();
    __syncthreads();
    if (count > 1) fetch_burst(Kh, 1, lds0 + G::kTile);
    {
        u4 a[NA];
        a[0] = k_read(0);
        a[1] = k_read(1);
#pragma unroll
        for (int m = 0; m < NA; ++m) {
            if (m + 2 < NA) a[m + 2] = k_read(m + 2);
            A[m & 1] = mfma_16bit<BF16>(a[m], st.qf[m / 2], m < 2 ? zero : A[m & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        float mx = fmaxf(A[0][0], A[0][1]);
#pragma unroll
        for (int r = 2; r < 32; r += 2) mx = fmaxf(fmaxf(mx, A[r >> 4][r & 15]), A[r >> 4][(r & 15) + 1]);
        const float tmax = pair_max(mx) * c;
        if (__builtin_amdgcn_ballot_w64(!(tmax <= st.M + kRescaleSlack)) != 0) rescale(tmax);
#pragma unroll
        for (int r = 0; r < 32; ++r) x[r] = __builtin_fmaf(A[r >> 4][r & 15], c, -st.M);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rk[ks] += G::kTile;   // K of tile 1 is in buffer 1
    if (count > 1) {
        wait_tile_landed();
        __syncthreads();
    }

    // ---------------------------------------------------------------- steady state: iteration i
    // reads K(i+1) from K buffer (i+1)&1 and V(i) from V buffer i&1; fetches K(i+2) into K buffer
    // i&1 and V(i+1) into V buffer (i+1)&1.  Returns whether the reference maximum has to be raised
    // before tile i+1 can be used.
    auto iteration = [&](int i, auto fetch_k_tag) -> bool {
        constexpr bool FETCH_K = decltype(fetch_k_tag)::value;
        const int cur = i & 1;
        const char* kbase = tile_base(Kh, i + 2);
        const char* vbase = tile_base(Vh, i + 1);
        const char* kbase1 = tile_base(Kh, i + 2, RUNS - 1);   // the same tiles of the second run
        const char* vbase1 = tile_base(Vh, i + 1, RUNS - 1);
        const unsigned kdst = lds0 + cur * G::kTile + lm.fill_dst;
        const unsigned vdst = lds0 + (2 + (cur ^ 1)) * G::kTile + lm.fill_dst;
        // ---- phase A
        {
            u4 a[NA];
            a[0] = k_read(0);
            a[1] = k_read(1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < NA; ++m) {
                if (m + 2 < NA) a[m + 2] = k_read(m + 2);
                A[m & 1] = mfma_16bit<BF16>(a[m], st.qf[m / 2], m < 2 ? zero : A[m & 1]);
#pragma unroll
                for (int q = 0; q < EU; ++q) exp_unit(m * EU + q);
                // the fetches of an iteration, spread over its first product: K, then V (with two runs: K of
                // both, then V of both, one load per MFMA)
                constexpr int TL = 2 * RUNS * NL;
                if ((m * TL) / NA != ((m + 1) * TL) / NA) {
                    const int li = (m * TL) / NA;
                    const int what = li / NL, l = li % NL;     // what: K run 0, (K run 1,) V run 0, (V run 1)
                    if (what < RUNS) {
                        if (FETCH_K) load_to_lds_16B(what ? kbase1 : kbase, lm.fill_src[l], kdst + what * kSet + l * 4096);
                    } else if constexpr (BF16) {
                        vreg[(what - RUNS) * NL + l] = *reinterpret_cast<const u4*>((what - RUNS ? vbase1 : vbase) + lm.fill_src[l]);
                    } else {
                        load_to_lds_16B(what - RUNS ? vbase1 : vbase, lm.fill_src[l], vdst + (what - RUNS) * kSet + l * 4096);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            exp_unit(16);
        }
        // ---- phase B, first half: row maximum of A and the rescale check
        s8 av[NB];
        av[0] = v_read(0);
        av[1] = v_read(1);
        __builtin_amdgcn_sched_barrier(0);
        float mx = 0.f;
        constexpr int H = NB / 2;          // MFMAs before the check
        constexpr int MS = 2;              // first slot that may read A (MFMA result latency)
        constexpr int MPS = (16 + (H - MS) - 1) / (H - MS);   // max3 ops per slot
#pragma unroll
        for (int idx = 0; idx < H; ++idx) {
            av[idx + 2] = v_read(idx + 2);
            st.o[idx % DB] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, av[idx]), __builtin_bit_cast(h8, pf.part(idx / DB & 1, idx / DB / 2)),
                                                                    st.o[idx % DB], 0, 0, 0);
            if constexpr (SPARSE) { if (idx % (H / 2) == H / 2 - 1) sums.add(pf.v[idx / (H / 2)]); }
            if (idx >= MS) {
#pragma unroll
                for (int q = 0; q < MPS; ++q) {
                    const int op = (idx - MS) * MPS + q;   // op-th max3: elements 2*op, 2*op+1
                    if (op < 16) {
                        const float u0 = A[(2 * op) >> 4][(2 * op) & 15], u1 = A[(2 * op) >> 4][((2 * op) & 15) + 1];
                        mx = op == 0 ? fmaxf(u0, u1) : fmaxf(fmaxf(mx, u0), u1);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        tmax_ahead = pair_max(mx) * c;
        const bool need = __builtin_amdgcn_ballot_w64(!(tmax_ahead <= st.M + kRescaleSlack)) != 0;
        // ---- phase B, second half, with the shifted scores of tile i+1 in between (and, for
        //      bfloat16, the conversion of the fetched V chunks).  If the reference maximum has to
        //      be raised (need), the shifted scores are recomputed after the loop exit.
        constexpr int FPS = 32 / (NB - H);   // fmas per slot
        constexpr int CW = RUNS * NL * 4;                        // 32-bit words of bfloat16 V to convert
        constexpr int CPS = (CW + (NB - H) - 1) / (NB - H);      // ... per slot
#pragma unroll
        for (int idx = H; idx < NB; ++idx) {
            if (idx + 2 < NB) av[idx + 2] = v_read(idx + 2);
            st.o[idx % DB] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, av[idx]), __builtin_bit_cast(h8, pf.part(idx / DB & 1, idx / DB / 2)),
                                                                    st.o[idx % DB], 0, 0, 0);
#pragma unroll
            for (int q = 0; q < FPS; ++q) {
                const int r = (idx - H) * FPS + q;
                x[r] = __builtin_fmaf(A[r >> 4][r & 15], c, -st.M);
            }
            if constexpr (BF16) {
#pragma unroll
                for (int q = 0; q < CPS; ++q) {
                    const int w = (idx - H) * CPS + q;    // w-th 32-bit word of the fetched chunks
                    if (w < CW) {
                        f2 y;
                        y[0] = __builtin_bit_cast(float, vreg[w / 4][w % 4] << 16);
                        y[1] = __builtin_bit_cast(float, vreg[w / 4][w % 4] & 0xffff0000u);
                        vreg[w / 4][w % 4] = __builtin_bit_cast(unsigned, __builtin_convertvector(y, h2));
                        if (w % 4 == 3)   // chunk w/4 = load (w/4) % NL of run (w/4) / NL
                            *(LDS_PTR(u4))(size_t)(vdst + ((w / 4) / NL) * kSet + ((w / 4) % NL) * 4096 + lane * 16) = vreg[w / 4];
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- switch buffers, publish the fetched tiles
        const int dk = cur ? G::kTile : -G::kTile;   // K(i+2) is in buffer i&1
        const int dv = cur ? -G::kTile : G::kTile;   // V(i+1) is in buffer (i+1)&1
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) rk[ks] += dk;
#pragma unroll
        for (int db = 0; db < DB; ++db) { rv[db][0] += dv; rv[db][1] += dv; }
        wait_tile_landed();
        __syncthreads();
        return need;
    };
    // Raise the reference maximum for the tile held in A and redo its shifted scores; only reached
    // when the loop below stopped because an iteration asked for it.
    auto raise_reference = [&]() {
        rescale(tmax_ahead);
#pragma unroll
        for (int r = 0; r < 32; ++r) x[r] = __builtin_fmaf(A[r >> 4][r & 15], c, -st.M);
    };
    int i = 0;
    while (i + 2 < count) {
        bool need = false;
#pragma unroll 1
        for (; i + 2 < count; ++i) {
            need = iteration(i, std::true_type{});
            if (need) { ++i; break; }
        }
        if (need) raise_reference();
    }
    if (i + 1 < count) {
        const bool need = iteration(i, std::false_type{});
        ++i;
        if (need) raise_reference();
    }

    // ---------------------------------------------------------------- last tile: probabilities, then O^T += V^T P^T
#pragma unroll
    for (int u = 0; u <= 16; ++u) exp_unit(u);
    {
        s8 av[NB];
        av[0] = v_read(0);
        av[1] = v_read(1);
#pragma unroll
        for (int idx = 0; idx < NB; ++idx) {
            if (idx + 2 < NB) av[idx + 2] = v_read(idx + 2);
            st.o[idx % DB] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, av[idx]), __builtin_bit_cast(h8, pf.part(idx / DB & 1, idx / DB / 2)),
                                                                    st.o[idx % DB], 0, 0, 0);
            if constexpr (SPARSE) { if (idx % (NB / 2) == NB / 2 - 1) sums.add(pf.v[idx / (NB / 2)]); }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    st.L += sums.of_lane();
    __syncthreads();   // all reads of the last tile are done before anything refills the buffers
}

// ------------------------------------------------------------------------------------------------
// The scan of attn_fwd_shared_kernel: 128-row query tiles, 32 rows per wavefront, compute units shared by workgroups (the
// kernel for 128-row tiles that have a compute unit to themselves is attn_fwd_kernel, above).  Both contractions run on
// v_mfma_f32_16x16x32, in the transposed form: S^T in blocks of 16 keys x 16 query rows, O^T in blocks of 16 columns of
// O x 16 query rows.  Lane l holds, for query row l % 16 of a block, keys (columns) 4*(l/16) + r of it in register r.
// Two blocks of 16 keys of S^T are, register for register, one B operand of the second product once its contraction
// index is read as
//     slot (l/16, 4t + r) <-> key 16t + 4*(l/16) + r,
// and V^T in the matching A layout is two ds_read_b64_tr_b16.  Every K and V^T fragment read from LDS feeds two MFMAs,
// one per block of 16 query rows.
// Why this shape and not 32x32x16: with live operands the chip is at its power limit, and a 16x16x32 reads and writes
// half as many accumulators per multiply-add.  MFMA-only loops on N(0, 1/4) operands: 1912 against 1671 TFLOP/s.
template <int D, int QT = 2>
struct NarrowState {
    u4 qf[D / 32][QT];    // Q^T as B operand: lane holds Q[row 16*qt + l%16][32*ks + 8*(l/16) .. +7] in qf[ks][qt]
    f4 o[D / 16][QT];     // O^T accumulators: o[db][qt][r] is column 16*db + 4*(l/16) + r of row 16*qt + l%16
    float M[QT];          // [qt]: reference maximum of score*c (log2 domain), same in the four lanes of a query row
    f4 L[QT];             // [qt]: running sum of the query row, a product with ones: in every element (QT = 4: in element 0 of lanes
                          // 0..15, zeros elsewhere)
};

// Lane-constant addresses.  A tile is filled as described at Geo, with a permutation of its own: chunk cc of row r sits
// at chunk position cc ^ swz(r).  V operand: 32 lanes read two neighbouring chunks of 8 rows, so swz / 2 is distinct
// over rows 0..7 and 8..15.  K operand: a ds_read_b128 is served 16 lanes at a time, 0-3, 12-15, 20-27 together and
// 4-11, 16-19, 28-31 together (measured; the same 32 on), which are rows 0-3 and 12-15 of one chunk with rows 4-11 of
// its neighbour and the other way round, so rows r and r + 8 may share a position's upper bits exactly if their last
// bits agree.  (A map that is only distinct over the 16 rows of one chunk: 14 % of the cycles lost to bank conflicts.)
template <int D>
struct NarrowMap {
    using G = Geo<D>;
    __device__ static __forceinline__ int swz(int row) {
        return D == 128 ? (row & 7) << 1 : ((row >> 1) & 3) << 1;
    }
    unsigned fill_src;        // source offset of load 0 inside a tile (load l: + 4096 l, the permutation repeats every 16 rows)
    unsigned fill_dst;        // wave * 1024 (load l: + 4096 l): LDS byte offset inside the tile
    unsigned k_rd[D / 32];    // byte offset inside a K tile, MFMA step ks, keys l%16 (+16 kb: + 16 kb row_bytes)
    unsigned v_rd[D / 16];    // byte offset inside a V tile of column block db, keys 4*(l/16) .. (+16: + 16 row_bytes)
    __device__ __forceinline__ NarrowMap(int wave, int lane) {
        const int r0 = wave * G::kRowsPerWaveLoad + lane / G::kChunksPerRow;
        fill_src = r0 * G::kRowBytes + ((lane % G::kChunksPerRow) ^ swz(r0)) * 16;
        fill_dst = wave * 1024;
        const int g = lane >> 4, ln = lane & 15;
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) k_rd[ks] = ln * G::kRowBytes + ((4 * ks + g) ^ swz(ln)) * 16;
        const int vrow = 4 * g + (ln >> 2);
#pragma unroll
        for (int db = 0; db < D / 16; ++db)
            v_rd[db] = vrow * G::kRowBytes + ((2 * db + ((ln & 3) >> 1)) ^ swz(vrow)) * 16 + (ln & 1) * 8;
    }
};

// The values are computed before this point.
__device__ __forceinline__ void keep_here(float (&x)[32]) {
#pragma unroll
    for (int i = 0; i < 32; i += 16)
        asm volatile("" : "+v"(x[i]), "+v"(x[i + 1]), "+v"(x[i + 2]), "+v"(x[i + 3]), "+v"(x[i + 4]), "+v"(x[i + 5]),
                     "+v"(x[i + 6]), "+v"(x[i + 7]), "+v"(x[i + 8]), "+v"(x[i + 9]), "+v"(x[i + 10]), "+v"(x[i + 11]),
                     "+v"(x[i + 12]), "+v"(x[i + 13]), "+v"(x[i + 14]), "+v"(x[i + 15]));
}

template <bool BF16>
__device__ __forceinline__ f4 mfma_16x16(u4 a, u4 b, f4 c) {
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// Maximum and sum over the four lanes l, l+16, l+32, l+48 that share a query row.  v_permlane16_swap swaps the odd
// 16-lane rows of its first operand with the even ones of its second (see lane_pair).
__device__ __forceinline__ void lane_rows(float x, float& even, float& odd) {
    unsigned a = __builtin_bit_cast(unsigned, x), b = a;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
    even = __builtin_bit_cast(float, a);
    odd = __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float quad_max(float x) {
    float e, o;
    lane_rows(x, e, o);
    return pair_max(fmaxf(e, o));
}
__device__ __forceinline__ float quad_sum(float x) {
    float e, o;
    lane_rows(x, e, o);
    return pair_sum(e + o);
}

// Resource descriptor of a K/V tile: `bytes` of it exist.  Rows past the end of the sequence, and whole tiles past the
// end of a scan (bytes = 0), read as zeros and cost no memory traffic.
__device__ __forceinline__ u4 tile_descriptor(const char* tile, unsigned bytes) {
    u4 r;
    r[0] = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)tile);
    r[1] = __builtin_amdgcn_readfirstlane((unsigned)((unsigned long long)tile >> 32) & 0xffffu);
    r[2] = __builtin_amdgcn_readfirstlane(bytes);
    r[3] = 0x00020000u;
    return r;
}
// One load of this wavefront's share of a tile, straight into LDS (see load_to_lds_16B for the inline assembly).  The
// whole offset inside the tile is in `voff`, the vector offset: that is the part that the range check compares with the
// descriptor's size.  A scalar offset is not: the check takes it off the size, which may be smaller here (0 behind a
// scan, a single row in a ragged tile), or leaves it out.
__device__ __forceinline__ void tile_load_to_lds(u4 descriptor, unsigned voff, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds_addr), "v"(voff), "s"(descriptor) : "memory", "m0");
}
__device__ __forceinline__ u4 tile_load(u4 d, unsigned voff) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((unsigned long long)d[0] | (unsigned long long)d[1] << 32), 0, (int)d[2], (int)d[3]);
    return __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
}
// All but the last VM vector-memory loads of this wavefront have landed, its LDS accesses are done, and so it is for
// every wavefront of the workgroup.
template <int VM>
__device__ __forceinline__ void landed_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(VM) : "memory");
}

// The scan of one query tile over its `nkv` K/V tiles j0, j0 + step, ..., software pipelined across tiles.  While the MFMAs of S(i+1)^T = K(i+1) Q^T run, the exponentials of tile i
// are issued between them; while the MFMAs of O^T += V(i)^T P(i)^T run, the row maximum of S(i+1), the lazy-rescale
// check and the (score*c - M) of tile i+1 are issued between them.  Two register sets alternate roles without copies:
// `A` accumulates the scores of the tile one ahead, `x` holds the shifted scores of the current tile until they have
// become probabilities.
//
// The one barrier of an iteration stands between the two products.  By then nobody reads K(i+1) or V(i-1) any more,
// so K(i+3) and V(i+1) are fetched into their places right behind it and have a whole iteration to land, although
// there are only two buffers of each.
// PHASES: the wavefronts that are in their second product, with its MFMAs and few vector instructions, go before
// those in their first, with all the exponentials, so that the two share the SIMD's units (see default_phase_priority).
// (For bfloat16 inputs V travels global -> registers -> binary16 -> LDS: V(i+2) is loaded in the middle of the second
// product of iteration i and converted in the first half of the second product of iteration i+1.)
//
// Tiles that need a mask (they reach past the first row of this wavefront under the causal mask, or past the end of
// the sequence) take the same way: their scores are set to -inf once they are complete, one comparison and one select
// each, and the reference maximum starts from a finite value, so that nothing later meets -inf - (-inf).
template <int D, bool BF16, bool CAUSAL, bool PHASES>
__device__ __forceinline__ void scan_tiles(NarrowState<D>& st, const NarrowMap<D>& lm, const char* Kh, const char* Vh, int N,
                                           float c, int j0, int step, int nkv, int qw0, int qrow, int lane,
                                           LDS_PTR(char) lds) {
    using G = Geo<D>;
    constexpr int KS = D / 32, DB = D / 16;
    constexpr int NA = 4 * KS;            // K fragments of a tile (two MFMAs each)
    constexpr int NB = 2 * DB;            // V^T fragments of a tile (two MFMAs each)
    constexpr int NL = G::kLoadsPerWave;
    constexpr int TA = 2 * NA, TB = 2 * NB;   // MFMAs of the first and of the second product
    constexpr int LA = 2;                 // fragments read ahead of their use
    // At d = 128 fragments are read two at a time and used in the order second, first, so that the one wait for the later read covers
    // both: half as many waits in the instruction stream.  (Read one by one, three ahead: 12 heads x 5000, bfloat16: 155.7 against 152.7
    // us with the fetches below, 32 x 8192, causal: 487 against 477 us.  At d = 64 it costs registers: 0 to +3 %.)
    constexpr bool PAIRS = D == 128;
    const unsigned lds0 = (unsigned)(size_t)lds;
    const int g = lane >> 4;
    // Row sums: sparse products (their 16 columns are the query rows), in the first two elements of L; the first operand is zero in the other rows,
    // which switches less.  From plain products, in the mean of 15 to 73 launches: d = 64 without a mask -0.5 % (bfloat16 -1.2 %), causal -1.0 % (-0.5 %); d =
    // 128 -1.0 % (0), causal -0.1 % (0); single launches -3 to +6 %, where workgroups come to end together or apart (22 x 7168, d = 64, bfloat16,
    // causal 172 -> 178 us, 77 x 493, d = 128, bfloat16 37.7 -> 40.3).  8 x 32768, d = 64, causal 1030 -> 1013 us, 1 x 131072 4196 -> 4154, 12 x 5000, bfloat16
    // 146.4 -> 144.2, 16 x 8192, bfloat16, causal 248.1 -> 249.2, 128 x 512 21.1 both.
    const SparseOnes ones = sparse_ones(lane, (lane & 3) < 2 ? kOnes : 0u);
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 A[4][2];         // S^T of the tile one ahead: block (kb, qt) = keys 16kb.. x query rows 16qt..
    float x[32];        // score*c - M of the current tile, index 16*qt + 4*kb + r
    Probabilities<true, 2> pf;
    u4 vreg[NL];        // bfloat16 V chunks in flight (BF16 only)
    float lim[2] = {-INFINITY, -INFINITY};    // [qt]: the raw score above which the reference maximum has to be raised

    // LDS read addresses: K of the tile one ahead, V of the current tile
    unsigned rk[KS], rv[DB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rk[ks] = lds0 + lm.k_rd[ks];
#pragma unroll
    for (int db = 0; db < DB; ++db) rv[db] = lds0 + 2 * G::kTile + lm.v_rd[db];

    // The fetches walk the scan position by position.  dk, dv: descriptors of the next K and V tile; rows: rows of the
    // scan from the next K tile on (the sequence may end inside the last tile, which comes first in a backward scan and
    // last in a forward one).  V follows K two positions behind (one, if it goes through registers), so its sizes are
    // K's of before.
    const int ragged = kTileKV * ((N + kTileKV - 1) / kTileKV) - N;      // rows the last tile of the sequence lacks
    const int lack = nkv * kTileKV > N ? ragged : 0;                     // ... if the scan includes that tile
    const long long stride = (long long)step * G::kTile;
    // (readfirstlane: everything here is uniform, and has to stay in scalar registers)
    auto size_of = [](int rows) {
        return (unsigned)__builtin_amdgcn_readfirstlane((rows < 0 ? 0 : rows < kTileKV ? rows : kTileKV) * G::kRowBytes);
    };
    auto advance = [&](u4& d) {
        const unsigned long long at = ((unsigned long long)d[1] << 32 | d[0]) + (unsigned long long)stride;
        d[0] = __builtin_amdgcn_readfirstlane((unsigned)at);
        d[1] = __builtin_amdgcn_readfirstlane((unsigned)(at >> 32));
    };
    const int first_rows = step < 0 || nkv == 1 ? kTileKV - lack : kTileKV;
    u4 dk = tile_descriptor(Kh + (long long)j0 * G::kTile, size_of(first_rows));
    u4 dv = tile_descriptor(Vh + (long long)j0 * G::kTile, size_of(first_rows));
    int rows = nkv * kTileKV - lack - first_rows;
    unsigned bytes1 = 0, bytes2 = 0;         // sizes of the K tiles one and two before the one in dk
    auto next_k = [&]() {
        bytes2 = bytes1;
        bytes1 = dk[2];
        advance(dk);
        dk[2] = size_of(rows);
        rows -= kTileKV;
    };
    auto next_v = [&]() {
        advance(dv);
        dv[2] = BF16 ? bytes1 : bytes2;
    };
    auto fetch_burst = [&](u4 d, unsigned dst) {
#pragma unroll
        for (int l = 0; l < NL; ++l) tile_load_to_lds(d, lm.fill_src + l * 4096, dst + lm.fill_dst + l * 4096);
    };
    auto v_to_regs = [&]() {
#pragma unroll
        for (int l = 0; l < NL; ++l) vreg[l] = tile_load(dv, lm.fill_src + l * 4096);
    };
    // w-th 32-bit word of the fetched chunks from bfloat16 to binary16; every fourth completes 16 bytes for LDS
    auto convert_word = [&](int w, unsigned dst) {
        f2 y;
        const unsigned word = vreg[w / 4][w % 4];
        y[0] = __builtin_bit_cast(float, word << 16);
        y[1] = __builtin_bit_cast(float, word & 0xffff0000u);
        vreg[w / 4][w % 4] = __builtin_bit_cast(unsigned, __builtin_convertvector(y, h2));
        if (w % 4 == 3) *(LDS_PTR(u4))(size_t)(dst + (w / 4) * 4096 + lane * 16) = vreg[w / 4];
    };
    constexpr int CW = NL * 4;     // 32-bit words of bfloat16 V this wavefront converts per tile
    // fragment m of K: keys 16*(m / KS).., columns 32*(m % KS)..; fragment m of V^T: keys 32*(m / DB).., columns 16*(m % DB)..
    auto k_read = [&](int m) -> u4 { return *(LDS_PTR(u4))(size_t)(rk[m % KS] + (m / KS) * 16 * G::kRowBytes); };
    auto v_read = [&](int m) -> u4 {
        const unsigned at = rv[m % DB] + (m / DB) * 32 * G::kRowBytes;
        const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)at);
        const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)(at + 16 * G::kRowBytes));
        return __builtin_bit_cast(u4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto s_mfma = [&](int m, int qt, u4 a, bool first) {
        A[m / KS][qt] = mfma_16x16<BF16>(a, st.qf[m % KS][qt], first ? zero : A[m / KS][qt]);
    };
    auto o_mfma = [&](int m, int qt, u4 a) { st.o[m % DB][qt] = mfma_16x16<false>(a, pf.part(m / DB, qt), st.o[m % DB][qt]); };
    // The scores in A: -inf where the key is not visible.  Register r of block kb is key
    // 16kb + 4g + r of the tile: visible up to the offset `ahead`.
    const int all_see = CAUSAL ? (qw0 < N - 1 ? qw0 : N - 1) : N - 1;      // last key visible to every row of the wavefront
    int kv0 = j0 * kTileKV;          // first key of the tile in A
    const int kv_step = step * kTileKV;
    auto mask = [&]() {
        if (kv0 + kTileKV - 1 > all_see) {
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
                const int last_key = CAUSAL ? (qrow + 16 * qt < N - 1 ? qrow + 16 * qt : N - 1) : N - 1;
                int ahead = last_key - kv0 - 4 * g;
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        asm volatile("" : "+v"(ahead));     // (separate comparisons: no lane masks kept and combined)
                        A[kb][qt][r] = 16 * kb + r > ahead ? -INFINITY : A[kb][qt][r];
                    }
            }
        }
    };
    auto shift_score = [&](int k) { x[k] = __builtin_fmaf(A[(k >> 2) & 3][k >> 4][k & 3], c, -st.M[k >> 4]); };
    // Raises the reference maxima for the tile in A, whose largest raw scores in this lane are mx (at least lim, see
    // score_limit), and takes its shifted scores again from the scores themselves: a difference of shifted scores would
    // carry the rounding at the distance from the old reference.  A row that has met no key yet (L = 0, lim = -inf) takes
    // any maximum, and starts from O = 0 whatever the values behind its masked keys were (0 times an infinite one is no number).
    float mx[2];
    auto max_op = [&](int qt, int op) {     // op-th of the 8 updates of mx[qt]: two scores each
        const f4& a = A[op / 2][qt];
        mx[qt] = fmaxf(fmaxf(mx[qt], a[2 * (op & 1)]), a[2 * (op & 1) + 1]);
    };
    auto raise_reference = [&]() {
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            const float t = quad_max(mx[qt]);           // the lanes of a query row move together
            const bool up = t > lim[qt];
            const float Mnew = up ? t * c : st.M[qt];
            const bool fresh = st.L[qt][0] + st.L[qt][1] == 0.f;
            const float alpha = up && !fresh ? fast_exp2(st.M[qt] - Mnew) : 1.0f;
            st.M[qt] = Mnew;
            st.L[qt] *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 4; ++r) st.o[db][qt][r] = fresh ? 0.f : st.o[db][qt][r] * alpha;
            if (up) lim[qt] = score_limit(t, Mnew, c);
#pragma unroll
            for (int k = 16 * qt; k < 16 * qt + 16; ++k) shift_score(k);
        }
    };
    // Pair u = 0..15 of probabilities is word u % 4 of B operand (kh, qt) = (u / 8, u / 4 % 2): keys
    // 16 (2 kh + u % 4 / 2) + 4g + 2 (u % 2), + 1.  Its steps: the two exponentials and the convert.
    float e[16][2];
    auto exp_op = [&](int u, int h) { e[u][h] = fast_exp2(x[16 * (u / 4 % 2) + 4 * (2 * (u / 8) + u % 4 / 2) + 2 * (u % 2) + h]); };
    auto convert_op = [&](int u) {
        pf.set(u / 8, u / 4 % 2, u % 4, __builtin_bit_cast(unsigned, __builtin_convertvector(f2{e[u][0], e[u][1]}, h2)));
    };
    // Row sums of the rounded probabilities, the values the second product uses.
    auto sum_mfma = [&](int qt) { st.L[qt] = sparse_sum(ones, pf.v[qt], st.L[qt]); };      // (all probabilities are there from the start of the second product)
    // What runs under the first product, in order: step k of pair u, the convert one pair behind its exponentials.
    constexpr int OA = 48;
    auto op_a = [&](int n) {
        const int u = n / 3, k = n % 3;
        if (k < 2) exp_op(u, k);
        else if (u > 0) convert_op(u - 1);
    };

    // ---------------------------------------------------------------- prologue: S(0), K(1..2) and V(0) on their way
    fetch_burst(dk, lds0);
    next_k();
    fetch_burst(dk, lds0 + G::kTile);
    if constexpr (BF16) v_to_regs();
    else fetch_burst(dv, lds0 + 2 * G::kTile);
    landed_barrier<NL>();
    {
        u4 a[NA];
#pragma unroll
        for (int m = 0; m < LA; ++m) a[m] = k_read(m);
#pragma unroll
        for (int m = 0; m < NA; ++m) {
            if (m + LA < NA) a[m + LA] = k_read(m + LA);
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) s_mfma(m, qt, a[m], m % KS == 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (BF16) {
#pragma unroll
        for (int w = 0; w < CW; ++w) convert_word(w, lds0 + 2 * G::kTile + lm.fill_dst);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // K(0) has been read
    next_k();
    fetch_burst(dk, lds0);
    if constexpr (BF16) {
        next_v();
        v_to_regs();
    }
    mask();
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        mx[qt] = lim[qt];
#pragma unroll
        for (int op = 0; op < 8; ++op) max_op(qt, op);
    }
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        const float t = quad_max(mx[qt]);
        st.M[qt] = t == -INFINITY ? 0.f : t * c;
        if (t != -INFINITY) lim[qt] = score_limit(t, st.M[qt], c);
    }
#pragma unroll
    for (int k = 0; k < 32; ++k) shift_score(k);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rk[ks] += G::kTile;   // K of tile 1 is in buffer 1
    u4 ak[LA];          // the first K fragments of the tile one ahead, read before the iteration starts
#pragma unroll
    for (int m = 0; m < LA; ++m) ak[m] = k_read(m);

    unsigned kdst = lds0 + G::kTile + lm.fill_dst, vdst = lds0 + 3 * G::kTile + lm.fill_dst;      // buffers (i+1)&1
    int flip = -G::kTile;                                                                         // ... to buffers i&1
    // The first K fragments of the next iteration are read at the end of one, ahead of the loop's branch.  For bfloat16 at d = 64
    // there are no registers for them beside the scores in A, which a raise still reads: there they follow the raise.
    // (Everywhere behind it: 12 heads x 5000, d = 128, bfloat16: 156.1 -> 157.2 us, 1 x 131072, d = 64: 4855 -> 4944 us.)
    constexpr bool READ_EARLY = D == 128 || !BF16;
    auto read_ahead = [&]() {
#pragma unroll
        for (int m = 0; m < LA; ++m) ak[m] = k_read(m);
    };
    // ---------------------------------------------------------------- steady state: iteration i
    // reads K(i+1) from K buffer (i+1)&1 and V(i) from V buffer i&1; fetches K(i+3) and V(i+1) into the buffers (i+1)&1.
    // Returns whether the reference maximum has to be raised before tile i+1 can be used.
    auto iteration = [&](int i) -> bool {
        if constexpr (PHASES) __builtin_amdgcn_s_setprio(1);
        next_k();     // K(i+3)
        next_v();     // V(i+1), with V through registers V(i+2)
        // ---- phase A
        {
            u4 a[NA];
#pragma unroll
            for (int m = 0; m < LA; ++m) a[m] = ak[m];
#pragma unroll
            for (int q = 0; q < NA; ++q) {
                const int m = PAIRS ? q ^ 1 : q;
                if (!PAIRS && q + LA < NA) a[q + LA] = k_read(q + LA);
                if (PAIRS && q % 2 == 0 && q + LA < NA) { a[q + LA] = k_read(q + LA); a[q + LA + 1] = k_read(q + LA + 1); }
#pragma unroll
                for (int qt = 0; qt < 2; ++qt) {
                    const int t = 2 * q + qt;
                    s_mfma(m, qt, a[m], q % KS == 0);
#pragma unroll
                    for (int n = t * OA / TA; n < (t + 1) * OA / TA; ++n) op_a(n);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            convert_op(15);
        }
        // ---- everything fetched in the iteration before has landed; nobody reads K(i+1) and V(i-1) any more
        //      (the probabilities pass through the statement, or the compiler moves the exponentials behind it)
        pf.pin();
        landed_barrier<0>();
        if constexpr (PHASES) __builtin_amdgcn_s_setprio(2);
        kv0 += kv_step;
        mask();
        // ---- phase B.  Under its MFMAs, in order: the row maxima of A, the row sums of tile i, the shifted scores of tile
        //      i+1 -- if the reference maximum has to be raised (need), they are taken again behind the iteration.  The direct
        //      loads of an iteration come along too, one behind every fourth MFMA (spread over all of it: 0 to +1 %; at d = 64 under
        //      the mask that is 0.4 % better), V first because it is needed first.
        //      With V through registers the conversion comes along with the maxima, then the next V loads.  (The V registers
        //      have landed: the compiler is told so here, or it would wait for them where it uses them, and with them for the
        //      direct loads issued in between, which it does not know of.)
        if constexpr (BF16) {
#pragma unroll
            for (int l = 0; l < NL; ++l) asm volatile("" : "+v"(vreg[l]));
        }
        u4 av[NB];
#pragma unroll
        for (int m = 0; m < LA; ++m) av[m] = v_read(m);
        __builtin_amdgcn_sched_barrier(0);
        mx[0] = lim[0];
        mx[1] = lim[1];
        bool need = false;
        constexpr int OC = BF16 ? 3 * CW : 0;            // conversions count as three
        constexpr int OM = 16 + OC, OB = OM + 32;        // maxima (and conversions), all
        constexpr int T0 = (OM * TB + OB - 1) / OB;      // first MFMA after the conversions
        constexpr int NV = BF16 ? 0 : NL;
        constexpr int TL = NV + NL;               // direct loads
        auto op_b = [&](int n) {
            if (n < OM) {
                const int j = n * 16 / OM, done = (n + 1) * 16 / OM;      // maxima begun before and with this step
                if (j != done) max_op(j & 1, j >> 1);
                if constexpr (BF16) {
                    const int w = n * CW / OM;
                    if (w != (n + 1) * CW / OM) convert_word(w, vdst);
                }
            } else {
                shift_score(n - OM);
            }
        };
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const int q = t / 2, m = PAIRS ? q ^ 1 : q;
            if (!PAIRS && t % 2 == 0 && q + LA < NB) av[q + LA] = v_read(q + LA);
            if (PAIRS && t % 4 == 0 && q + LA < NB) { av[q + LA] = v_read(q + LA); av[q + LA + 1] = v_read(q + LA + 1); }
            if (BF16 && t == T0) v_to_regs();
            o_mfma(m, t & 1, av[m]);
            // Row sums: behind the first MFMA of each half at d = 64 without a mask (4 x 14836 259.1 us, behind the 4th of the first two quarters 269.9, with
            // plain products 260.6; 18 x 3260 63.9, 65.5, 64.4; in the mean of 87 bfloat16 launches -1.3 and -1.0 % from plain products), elsewhere early in
            // the first two quarters (under the mask at d = 64 the compiler spills with later ones).
            constexpr int S0 = D == 128 ? 5 : CAUSAL ? TB / 4 - 1 : 1, S1 = D == 128 ? TB / 4 + 5 : CAUSAL ? TB / 2 - 1 : TB / 2 + 1;
            if (t == S0 || t == S1) sum_mfma(t == S1);
            constexpr bool EARLY = D == 128 || !CAUSAL;
            for (int li = EARLY ? t / 4 : t * TL / TB; li < TL && (EARLY ? t % 4 == 1 && li == t / 4 : li < (t + 1) * TL / TB); ++li) {
                if (li < NV) tile_load_to_lds(dv, lm.fill_src + li * 4096, vdst + li * 4096);
                else tile_load_to_lds(dk, lm.fill_src + (li - NV) * 4096, kdst + (li - NV) * 4096);
            }
#pragma unroll
            for (int n = t * OB / TB; n < (t + 1) * OB / TB; ++n) {
                op_b(n);
                // (mx starts from lim: it exceeds lim exactly when a score does)
                if (n == OM + 8) need = __builtin_amdgcn_ballot_w64(!(mx[0] <= lim[0]) || !(mx[1] <= lim[1])) != 0;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        keep_here(x);       // (or the compiler moves what no instruction up to here reads behind the loop's branch)
        // ---- switch buffers: K(i+2) is in buffer i&1, V(i+1) in buffer (i+1)&1
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) rk[ks] += flip;
#pragma unroll
        for (int db = 0; db < DB; ++db) rv[db] -= flip;
        kdst += flip;
        vdst += flip;
        flip = -flip;
        if constexpr (READ_EARLY) read_ahead();
        return need;
    };
    int i = 0;
#pragma unroll 1
    for (; i + 1 < nkv; ++i) {
        if (iteration(i)) raise_reference();
        if constexpr (!READ_EARLY) read_ahead();
    }

    // ---------------------------------------------------------------- last tile: probabilities, then O^T += V^T P^T
    if constexpr (PHASES) __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int n = 0; n < OA; ++n) op_a(n);
    convert_op(15);
    landed_barrier<0>();      // also the fetches past the end of the scan, which write zeros into buffers nobody reads
    if (!CAUSAL || kv0 <= qw0 + 31) {      // (not if every row of the wavefront lies before the tile's first key)
        u4 av[NB];
#pragma unroll
        for (int m = 0; m < LA; ++m) av[m] = v_read(m);
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const int m = t / 2;
            if ((t & 1) == 0 && m + LA < NB) av[m + LA] = v_read(m + LA);
            o_mfma(m, t & 1, av[m]);
            if (t == TB / 4 - 1 || t == TB / 2 - 1) sum_mfma(t == TB / 2 - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();   // all reads of the last tile are done before anything refills the buffers
}

// ------------------------------------------------------------------------------------------------
// 256-row tiles (head dimension 128): a wavefront owns 64 query rows, as four blocks of 16, and a workgroup has the compute
// unit to itself.  Products, layouts, masks, row sums and the running maximum are those of scan_tiles; every K and V^T
// fragment read from LDS feeds four MFMAs instead of two, which halves the operand traffic from LDS and the L2 -> LDS
// traffic per multiply-add.
//
// What bounds it: with live operands the power limit, and the issue of its one wavefront per SIMD, which holds with zeros too.  A launch takes 3170
// cycles per tile at 1.93 GHz (zeros: 3100 at 2.36) for 132 MFMAs of 16 cycles (128 for the products, 4 for the row sums), 64 exponentials, 149 other
// vector, 48 LDS and 33 scalar instructions and 8 loads; bfloat16 3450 at 2.06 GHz (3380 at 2.39) for 136 MFMAs, 8 of them for the row sums, 201 other
// vector and 52 LDS instructions (profiles/wide_kernel_cycles.txt).  Both count: less clock goes with less voltage, so a tile in 7 % fewer cycles takes 3.5 % less time at the power limit.  What
// that rests on: work spread evenly over the MFMAs (WidePlan); loads that share M0, and bases that move by a tile, in place of some 40 scalar
// instructions a tile; nothing behind the loop's branch.  32 heads x 16384, before and after: binary16 3375 -> 3257 us
// (zeros: 2941 -> 2739), bfloat16, causal 1796 -> 1755 us.  And neighbouring MFMAs share an operand wherever they can: columns of K go
// in the outer loop, query blocks there and back (MFMA-only loops: 1898 -> 1935 TFLOP/s; here -0.5 to -1.5 % with live operands).
// 16x16x32 and not 32x32x16 because it reads and writes half as many accumulators per multiply-add: from 32x32x16 to this shape, 32 heads x
// 16384, binary16 3592 -> 3403 us, bfloat16 3785 -> 3445 us.
//
// What is spread how: exponentials and converts of tile i under the MFMAs of S(i+1)^T and the first of O^T += V(i)^T P(i)^T, maxima and shifted
// scores of tile i+1 under the rest of those.  K(i+4) and V(i+2) are fetched in the first product of iteration i, one load behind every eighth MFMA,
// into four buffers each, and have until the barrier of iteration i+1.  By then V(i+1) is needed, whose first fragments are read ahead of the
// barrier of iteration i+1 like K's first ones ahead of the loop's branch (first V fragments behind the barrier: +2 %).  Fragments are
// read two at a time, one pair ahead, and used in the order second, first: one wait covers both.
//
// MFMAs are inline assembly with the register file of every operand fixed: with more than 256 registers per wavefront the accumulation
// registers have to hold what only the matrix pipe touches (O^T, Q^T, the row sums) and nothing the vector ALU reads, or every use
// costs a copy.  The compiler does not see them as MFMAs and inserts no wait states; wide_settle_*() stands wherever vector
// instructions read what the last few MFMAs may still be writing (4 passes + 3 wait states), wide_guard() where MFMAs read
// accumulators that vector instructions have just written.  In the loop the distance is kept by the order: the first maximum comes
// behind the exponentials of the second product, 23 MFMAs (bfloat16: 33) after the last one that wrote a score.  static_asserts beside the
// plan and a test that walks the built code hold that.
constexpr int kWideBuffers = 4;
constexpr int kWideLdsBytes = 2 * kWideBuffers * Geo<128>::kTile;

template <bool BF16>
__device__ __forceinline__ void wide_s_first(f4& acc, const u4& k, const u4& q) {
    if constexpr (BF16) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(k), "a"(q));
    else asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=&v"(acc) : "v"(k), "a"(q));
}
template <bool BF16>
__device__ __forceinline__ void wide_s(f4& acc, const u4& k, const u4& q) {
    if constexpr (BF16) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(k), "a"(q));
    else asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(k), "a"(q));
}
__device__ __forceinline__ void wide_o(f4& acc, const u4& v, const u4& p) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(v), "v"(p));
}
__device__ __forceinline__ void wide_sum(f4& acc, const u4& ones, const u4& p) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "a"(ones), "v"(p));
}
__device__ __forceinline__ void wide_sparse_sum(f4& acc, const SparseOnes& ones, const u8& p) {
    asm volatile("v_smfmac_f32_16x16x64_f16 %0, %1, %2, %3" : "+a"(acc) : "a"(ones.one), "v"(p), "v"(ones.pick));
}
// The accumulators pass through these statements, so that no use of them can be scheduled ahead of the wait (or, wide_guard, behind it).
__device__ __forceinline__ void wide_settle_s(f4 (&A)[4][4]) {
    asm volatile("s_nop 15" ::: "memory");
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) asm volatile("" : "+v"(A[kb][0]), "+v"(A[kb][1]), "+v"(A[kb][2]), "+v"(A[kb][3]));
}
__device__ __forceinline__ void wide_hold_o(NarrowState<128, 4>& st) {
#pragma unroll
    for (int db = 0; db < 8; ++db) asm volatile("" : "+a"(st.o[db][0]), "+a"(st.o[db][1]), "+a"(st.o[db][2]), "+a"(st.o[db][3]));
    asm volatile("" : "+a"(st.L[0]), "+a"(st.L[1]), "+a"(st.L[2]), "+a"(st.L[3]));
}
__device__ __forceinline__ void wide_settle_o(NarrowState<128, 4>& st) {
    asm volatile("s_nop 15" ::: "memory");
    wide_hold_o(st);
}
// Probabilities that have just been converted, ahead of the MFMAs that read them (a vector instruction's result: 2 wait states).
template <bool SPARSE>
__device__ __forceinline__ void wide_settle_p(Probabilities<SPARSE, 4>& pf) {
    pf.pin();
    asm volatile("s_nop 3");
    pf.pin();
}
__device__ __forceinline__ void wide_guard_o(NarrowState<128, 4>& st) {
    wide_hold_o(st);
    asm volatile("s_nop 7" ::: "memory");
}

// Which of N operations stand behind which of W MFMAs: first[w] .. first[w + 1] - 1 behind MFMA w.  cost[n] is what operation n takes of the
// issue port, taken[w] what else stands behind MFMA w; the sum is spread as evenly as the order of the operations allows.
template <int W>
struct Windows {
    int first[W + 1];
};
template <int W, int N>
constexpr Windows<W> spread(const int (&cost)[N], const int (&taken)[W]) {
    int total = 0, spent = 0, n = 0;
    for (int k = 0; k < N; ++k) total += cost[k];
    for (int w = 0; w < W; ++w) total += taken[w];
    Windows<W> r{};
    for (int w = 0; w < W; ++w) {
        r.first[w] = n;
        spent += taken[w];
        while (n < N && (2 * spent + cost[n]) * W <= 2 * total * (w + 1)) spent += cost[n++];
    }
    r.first[W] = N;
    return r;
}

// What runs under the MFMAs of an iteration of scan_tiles_wide.  One wavefront per SIMD issues an MFMA in 8 cycles, a vector instruction in 4.5, an
// exponential in 8.5 and an LDS read in 5 to 6 (measured one wavefront at a time: an MFMA alone 16.6 cycles, with 1, 2, 3, 4 vector instructions
// behind it 16.9, 17.2, 22, 26, with 1, 2, 3 exponentials 17, 26, 34), and an MFMA that comes late is not made up for: work has to be even from
// one MFMA to the next.  In vector instructions an exponential counts as three here (two: 0 to +0.2 %, four: +1.5 %).  The last PAIRS
// pairs of exponentials run in the second product, whose first half does not need them: the first would overflow and the second have room
// (32 x 16384, binary16, all operands zero, where the power limit plays no part: none 2878 us, 4: 2738, 6: 2696, 7: 2689, 10: 2705;
// bfloat16, causal: 3: 1760, 4: 1780, 5: 1755, 6: 1770, 7: 1787).
template <bool BF16>
struct WidePlan {
    static constexpr int PAIRS = BF16 ? 5 : 7;
    static constexpr int OX = 3 * PAIRS, OA = 96 - OX;        // steps of the exponentials in the second product, in the first
    static constexpr int CW = BF16 ? 16 : 0;                  // words of V to convert
    static constexpr int exponential = 3;
    static constexpr Windows<64> first_product() {
        int cost[OA] = {}, taken[64] = {};
        for (int n = 0; n < OA; ++n) cost[n] = n % 3 < 2 ? exponential : 1;
        for (int t = 0; t < 64; ++t) {
            if (t % 8 == 0) taken[t] += t < 56 ? 2 : 4;                               // fragment reads: a pair of K, at the end of V^T
            if (!BF16 && t % 8 == 4) taken[t] += t == 4 || t == 36 ? 3 : 1;           // a direct load, the first of a tile with M0
            if (t >= 57 && t < 61) taken[t] += 1;                                     // K addresses
        }
        return spread<64>(cost, taken);
    }
    // OX steps of exponentials, CW conversions, 32 maxima, 4 comparisons, 64 shifted scores
    static constexpr int OM = OX + CW, OQ = OM + 32, OS = OQ + 4, OB = OS + 64;
    // MFMAs of the second product: the 64 of the product in order, row sums in between.  Sparse ones (see sparse_sum) want all of a row's probabilities and
    // stand in the second half; bfloat16 has no registers left for them (0 to +10 %) and sums every 32 keys.
    static constexpr bool SPARSE = !BF16;
    static constexpr int SUMS = SPARSE ? 4 : 8, W = 64 + SUMS, HALF = SPARSE ? 32 : 36;
    // The sum of this lane's row from its accumulators: sparse products leave it in two, plain ones in the first alone (with the second, a zero, added
    // there too the bfloat16 kernels needed three registers more than they have).
    static __device__ __forceinline__ float row_sum(const f4& L) { return quad_sum(SPARSE ? L[0] + L[1] : L[0]); }
    static constexpr bool sum_at(int w) { return SPARSE ? w >= HALF && w % 9 == 4 : w % 9 == 8; }
    static constexpr int product_at(int w) {
        int t = 0;
        for (int v = 0; v < w; ++v) t += !sum_at(v);
        return t;
    }
    // Sparse sums read all of a row's probabilities, sum k of the others those of 32 keys: the second 32 from k = 4 on.
    static constexpr bool sums_in_time() {
        for (int w = 0, k = 0; w < W; ++w)
            if (sum_at(w) && (SPARSE || k++ >= 4) && w < HALF) return false;
        return true;
    }
    static constexpr Windows<W> second_product() {
        int cost[OB] = {}, taken[W] = {};
        for (int n = 0; n < OB; ++n) cost[n] = n < OX ? (n % 3 < 2 ? exponential : 1) : n < OM ? 3 : 1;
        for (int w = 0; w < W; ++w) {
            if (!sum_at(w) && product_at(w) % 8 == 0) taken[w] += product_at(w) < 56 ? 4 : 2;      // fragment reads: a pair of V^T, at the end of K
            if (BF16 && w < 4) taken[w] += 1;                                         // direct loads
            if (w >= W - 12) taken[w] += w < W - 8 ? w % 2 == 0 : 1;                 // bases, V addresses
        }
        return spread<W>(cost, taken);
    }
};

template <bool BF16, bool CAUSAL>
__device__ __forceinline__ void scan_tiles_wide(NarrowState<128, 4>& st, const NarrowMap<128>& lm, const char* Kh, const char* Vh, int N, float c,
                                                int j0, int step, int nkv, int qw0, int wave, int lane, LDS_PTR(char) lds) {
    constexpr int D = 128, QT = 4;
    using G = Geo<D>;
    using P = WidePlan<BF16>;
    constexpr int KS = 4, DB = 8, NA = 16, NB = 16, NL = G::kLoadsPerWave, TA = 64, TB = 64;
    constexpr int LA = 2;                              // fragments read ahead of their use
    constexpr unsigned VB = kWideBuffers * G::kTile;   // V buffers follow the K buffers
    const unsigned lds0 = (unsigned)(size_t)lds;
    const int g = lane >> 4;
    // A operand of the row sums: binary16 ones in its first row or two, zeros in the others (all ones: +0.7 %, the zeros switch nothing)
    const unsigned one = (lane & 15) > (P::SPARSE ? 1 : 0) ? 0u : kOnes;
    SparseOnes ones = sparse_ones(lane, one);
    asm volatile("" : "+a"(ones.one));
    f4 A[4][QT];        // S^T of the tile one ahead: block (kb, qt) = keys 16kb.. x query rows 16qt..
    float x[16 * QT];   // score*c - M of the current tile, index 16*qt + 4*kb + r
    Probabilities<P::SPARSE, QT> pf;
    u4 vreg[NL];        // bfloat16 V chunks in flight (BF16 only)
    float lim[QT], mx[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) lim[qt] = -INFINITY;

    unsigned rk[KS], rv[DB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rk[ks] = lds0 + lm.k_rd[ks];
#pragma unroll
    for (int db = 0; db < DB; ++db) rv[db] = lds0 + VB + lm.v_rd[db];

    // Position p of the scan lives in K buffer p & 3 and V buffer p & 3.  A wavefront fetches 16 neighbouring rows of a tile with four loads of four
    // rows each, so that one M0 and the offsets of the instructions serve all four.  The permutation repeats every eight rows: of a whole tile, loads
    // 0 and 2, 1 and 3 have the same addresses but for those offsets.  The rows that the last tile of the sequence lacks repeat row N-1
    // (masked before use; bases lie kBias below the tile, so that no offset is negative).  Fetches beyond the scan re-fetch its last tile into a
    // buffer nobody reads.
    constexpr unsigned kBias = 4096;
    const unsigned fill_dst = wave * 4096;
    auto base_of = [&](const char* head, int p) {
        const unsigned long long at = (unsigned long long)(head + (size_t)(j0 + p * step) * G::kTile - kBias);
        return (unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(at >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((unsigned)at);
    };
    auto offset_of = [&](int l, int rows) {      // ... of load l in a tile of `rows` rows
        const int row = 16 * wave + 4 * l + g;
        return (unsigned)((row < rows ? row : rows - 1) * G::kRowBytes + ((lane & 15) ^ NarrowMap<D>::swz(4 * l + g)) * 16 + (int)kBias - 1024 * l);
    };
    typedef const __attribute__((address_space(1))) u4* Global16B;
    auto rows_of = [&](int p) { return N - (j0 + p * step) * kTileKV; };
    auto fetch = [&](const char* head, int p, unsigned buffer) {
        p = p < nkv ? p : nkv - 1;
        const unsigned long long base = base_of(head, p);
        aim_lds(buffer + fill_dst);
        static_for<NL>([&](auto l) { load_aimed_16B<1024 * decltype(l)::value>((const char*)base, offset_of(l, rows_of(p))); });
    };
    auto v_to_regs = [&](int p) {
        p = p < nkv ? p : nkv - 1;
        const unsigned long long base = base_of(Vh, p);
#pragma unroll
        for (int l = 0; l < NL; ++l) vreg[l] = *(Global16B)(base + offset_of(l, rows_of(p)) + 1024 * l);
    };
    // In the loop: bases that move by a tile (move_k, move_v) and the offsets of whole tiles.  From the last position ahead of `whole` on, the first
    // one that is not a whole tile further on, the bases stand still: the tile there is fetched again, and where the scan goes on with
    // a tile that is not whole, that one in its place afterwards (mend).
    const unsigned long long stride = (unsigned long long)((long long)step * G::kTile);
    const int whole = step > 0 && nkv * kTileKV > N ? nkv - 1 : nkv;
    const unsigned off[2] = {offset_of(0, kTileKV), offset_of(1, kTileKV)};
    unsigned long long base_k, base_v, move_k, move_v;
    // word w of the chunks in vreg; `dst` is where this lane's first one goes
    auto convert_word = [&](int w, unsigned dst) {
        f2 y;
        const unsigned word = vreg[w / 4][w % 4];
        y[0] = __builtin_bit_cast(float, word << 16);
        y[1] = __builtin_bit_cast(float, word & 0xffff0000u);
        vreg[w / 4][w % 4] = __builtin_bit_cast(unsigned, __builtin_convertvector(y, h2));
        if (w % 4 == 3) *(LDS_PTR(u4))(size_t)(dst + (w / 4) * 1024) = vreg[w / 4];
    };
    constexpr int CW = NL * 4;
    // fragment m of K: columns 32*(m / 4).., keys 16*(m % 4)..; fragment m of V^T: keys 32*(m / DB).., columns 16*(m % DB)..
    auto k_read = [&](int m) -> u4 { return *(LDS_PTR(u4))(size_t)(rk[m / 4] + (m % 4) * 16 * G::kRowBytes); };
    auto v_read = [&](int m) -> u4 {
        const unsigned at = rv[m % DB] + (m / DB) * 32 * G::kRowBytes;
        const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)at);
        const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)(at + 16 * G::kRowBytes));
        return __builtin_bit_cast(u4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto s_mfma = [&](int m, int qt, const u4& a) {
        if (m < 4) wide_s_first<BF16>(A[m % 4][qt], a, st.qf[m / 4][qt]);
        else wide_s<BF16>(A[m % 4][qt], a, st.qf[m / 4][qt]);
    };
    auto o_mfma = [&](int m, int qt, const u4& a) {
        wide_o(st.o[m % DB][qt], a, pf.part(m / DB, qt));
    };
    auto sum_mfma = [&](int k) {      // the k-th row sum of a tile
        if constexpr (P::SPARSE) wide_sparse_sum(st.L[k], ones, pf.v[k]);
        else wide_sum(st.L[k % QT], ones.one, pf.part(k / QT, k % QT));
    };
    // Masks, maxima, shifted scores and raises as in scan_tiles.
    const int all_see = CAUSAL ? (qw0 < N - 1 ? qw0 : N - 1) : N - 1;
    int kv0 = j0 * kTileKV;
    const int kv_step = step * kTileKV;
    auto mask = [&]() {
        if (__builtin_expect(kv0 + kTileKV - 1 > all_see, 0)) {
            wide_settle_s(A);
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
                const int row = qw0 + (lane & 15) + 16 * qt;
                const int last_key = CAUSAL ? (row < N - 1 ? row : N - 1) : N - 1;
                const int ahead = last_key - kv0 - 4 * g;
                float none = -INFINITY;
                asm volatile("" : "+v"(none));
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // (assembly: in place, or the compiler keeps A in two sets of registers and copies it in every iteration)
                        float s = A[kb][qt][r];
                        asm volatile("v_cmp_gt_i32_e32 vcc, %1, %2\n\ts_nop 1\n\tv_cndmask_b32_e32 %0, %0, %3, vcc"
                                     : "+v"(s) : "n"(16 * kb + r), "v"(ahead), "v"(none) : "vcc");
                        A[kb][qt][r] = s;
                    }
            }
        }
    };
    auto shift_score = [&](int k) { x[k] = __builtin_fmaf(A[(k >> 2) & 3][k >> 4][k & 3], c, -st.M[k >> 4]); };
    auto max_op = [&](int qt, int op) {
        const f4& a = A[op / 2][qt];
        mx[qt] = fmaxf(fmaxf(mx[qt], a[2 * (op & 1)]), a[2 * (op & 1) + 1]);
    };
    auto raise_reference = [&]() {
        wide_settle_s(A);
        wide_settle_o(st);
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            float t = mx[qt];
            asm volatile("" : "+v"(t));
            t = quad_max(t);
            const bool up = t > lim[qt];
            const float Mnew = up ? t * c : st.M[qt];
            const bool fresh = P::row_sum(st.L[qt]) == 0.f;
            const float alpha = up && !fresh ? fast_exp2(st.M[qt] - Mnew) : 1.0f;
            st.M[qt] = Mnew;
            st.L[qt] *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 4; ++r) st.o[db][qt][r] = fresh ? 0.f : st.o[db][qt][r] * alpha;
            if (up) lim[qt] = score_limit(t, Mnew, c);
#pragma unroll
            for (int k = 16 * qt; k < 16 * qt + 16; ++k) shift_score(k);
        }
        wide_guard_o(st);
    };
    // Pair u = 0..31 of probabilities is word u % 4 of B operand (kh, qt) = (u / 16, u / 4 % 4)
    float e[32][2];
    auto exp_op = [&](int u, int h) { e[u][h] = fast_exp2(x[16 * (u / 4 % 4) + 4 * (2 * (u / 16) + u % 4 / 2) + 2 * (u % 2) + h]); };
    auto convert_op = [&](int u) {
        pf.set(u / 16, u / 4 % 4, u % 4, __builtin_bit_cast(unsigned, __builtin_convertvector(f2{e[u][0], e[u][1]}, h2)));
    };
    // step n of a pair: its two exponentials, and the convert of the pair before
    auto op_a = [&](int n) {
        const int u = n / 3, k = n % 3;
        if (k < 2) exp_op(u, k);
        else if (u > 0) convert_op(u - 1);
    };
    wide_guard_o(st);

    // ---------------------------------------------------------------- prologue: K(0..3) and V(0..1) on their way, S(0)
    static_for<4>([&](auto p) {
        fetch(Kh, p, lds0 + p * G::kTile);
        if constexpr (!BF16 && (p == 1 || p == 2)) fetch(Vh, p - 1, lds0 + VB + (p - 1) * G::kTile);
    });
    if constexpr (BF16) {
        // V(0) and V(1) go through registers into their buffers, V(2) waits in vreg
#pragma unroll 1
        for (int p = 0; p < 2; ++p) {
            v_to_regs(p);
#pragma unroll
            for (int w = 0; w < CW; ++w) convert_word(w, lds0 + VB + p * G::kTile + fill_dst + lane * 16);
        }
        v_to_regs(2);
        landed_barrier<0>();
    } else {
        landed_barrier<12>();
    }
    {
        u4 a[NA];
#pragma unroll
        for (int m = 0; m < LA; ++m) a[m] = k_read(m);
        static_for<NA>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            if constexpr (m + LA < NA) a[m + LA] = k_read(m + LA);
            static_for<QT>([&](auto q) { s_mfma(m, decltype(q)::value, a[m]); });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // K(0) has been read: iteration 0 fetches K(4) into its place
    wide_settle_s(A);
    mask();
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        mx[qt] = lim[qt];
#pragma unroll
        for (int op = 0; op < 8; ++op) max_op(qt, op);
        const float t = quad_max(mx[qt]);
        st.M[qt] = t == -INFINITY ? 0.f : t * c;
        if (t != -INFINITY) lim[qt] = score_limit(t, st.M[qt], c);
#pragma unroll
        for (int k = 16 * qt; k < 16 * qt + 16; ++k) shift_score(k);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rk[ks] += G::kTile;
    u4 ak[LA];
#pragma unroll
    for (int m = 0; m < LA; ++m) ak[m] = k_read(m);

    // ---------------------------------------------------------------- steady state: iteration i
    // reads K(i+1) and V(i), fetches K(i+4) into the place of K(i), which was read before the barrier of iteration i-1, and V(i+2) into that
    // of V(i-2), read before it too.  Behind its barrier K(i+2) and V(i+1) have landed (all but the eight loads of its own).
    // bfloat16: V(i+2) goes from registers into its place in the second product, then V(i+3) is loaded; K(i+4) is fetched there too, as the
    // compiler waits for all loads where it uses those registers.
    // Returns whether the reference maximum has to be raised before tile i+1 can be used.
    unsigned ring = 0;        // byte offset of buffer i & 3
    auto k_place = [&]() { return (unsigned)__builtin_amdgcn_readfirstlane(lds0 + ring); };
    auto v_place = [&]() { return (unsigned)__builtin_amdgcn_readfirstlane(lds0 + VB + (ring ^ 2 * G::kTile)); };
    auto turn = [&]() { ring = (unsigned)__builtin_amdgcn_readfirstlane((ring + G::kTile) & 3 * G::kTile); };
    static constexpr auto plan_a = P::first_product();
    static constexpr auto plan_b = P::second_product();
    // What the order has to keep apart, as the compiler adds no wait states.  (Operation n stands behind MFMA w where first[w] <= n < first[w + 1].)
    static_assert(plan_b.first[8] <= P::OM, "no score is read within eight MFMAs after the one that wrote the last");
    static_assert(P::OA / 3 > 16, "the first half of the probabilities is complete ahead of the barrier");
    static_assert(plan_b.first[P::HALF - 1] > P::OX, "an MFMA and more between the last conversion, ahead of operation OX, and the first that reads it");
    static_assert(P::product_at(P::HALF) == 32 && P::sums_in_time(), "the second half of the probabilities is read from MFMA HALF on");
    // (assembly: left to itself the compiler collects these additions behind the loop's branch, where nothing hides them)
    auto move = [](unsigned& at, int by) { asm volatile("v_add_u32 %0, %1, %0" : "+v"(at) : "s"(by)); };
    auto iteration = [&]() -> unsigned long long {
        const int dka = ring == 2 * G::kTile ? -3 * (int)G::kTile : (int)G::kTile, dva = ring == 3 * G::kTile ? -3 * (int)G::kTile : (int)G::kTile;
        u4 av[NB];
        {
            u4 a[NA];
#pragma unroll
            for (int m = 0; m < LA; ++m) a[m] = ak[m];
            // Fragments are read two at a time and used in the order second, first: the one wait for the later read covers both.
            static_for<TA>([&](auto tc) {
                constexpr int t = decltype(tc)::value, q = t / QT, m = q ^ 1, qt = q & 1 ? QT - 1 - t % QT : t % QT;
                if constexpr (t % 8 == 0) {
                    if constexpr (q + LA < NA) { a[q + LA] = k_read(q + LA); a[q + LA + 1] = k_read(q + LA + 1); }
                    else { av[q + LA - NA] = v_read(q + LA - NA); av[q + LA - NA + 1] = v_read(q + LA - NA + 1); }
                }
                s_mfma(m, qt, a[m]);
                if constexpr (!BF16 && t % 8 == 4) {
                    constexpr int li = t / 8;
                    if constexpr (li == 0) aim_lds(v_place() + fill_dst);
                    if constexpr (li == 4) aim_lds(k_place() + fill_dst);
                    if constexpr (li < 4) load_aimed_16B<1024 * li>((const char*)base_v, off[li & 1]);
                    else load_aimed_16B<1024 * (li - 4)>((const char*)base_k, off[li & 1]);
                }
                if constexpr (t >= 57 && t < 61) move(rk[t - 57], dka);
                static_for<plan_a.first[t + 1] - plan_a.first[t]>([&](auto k) { op_a(plan_a.first[t] + decltype(k)::value); });
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        // (the probabilities pass through the statement, or the compiler moves the exponentials behind the barrier)
        pf.pin();
        if constexpr (BF16) landed_barrier<0>();
        else landed_barrier<8>();
        kv0 += kv_step;
        asm volatile("" : "+s"(kv0));
        mask();
        if constexpr (BF16) {      // (the V registers have landed: the compiler is told so here, see scan_tiles)
#pragma unroll
            for (int l = 0; l < NL; ++l) asm volatile("" : "+v"(vreg[l]));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) mx[qt] = lim[qt];
        unsigned long long need = 0;
        unsigned vdst = v_place();      // (bfloat16: this lane's place; one address, the rest in the instructions' offsets)
        if constexpr (BF16) asm volatile("v_lshl_add_u32 %0, %1, 4, %2" : "=v"(vdst) : "v"(lane), "s"(vdst + fill_dst));
        auto op_b = [&](auto nc) {
            constexpr int n = decltype(nc)::value;
            if constexpr (n < P::OX) op_a(P::OA + n);
            else if constexpr (n < P::OM) {
                if constexpr (n == P::OX) convert_op(31);
                convert_word(n - P::OX, vdst);
            } else if constexpr (n < P::OQ) {
                if constexpr (n == P::OM && !BF16) convert_op(31);
                max_op((n - P::OM) & 3, (n - P::OM) >> 2);
            } else if constexpr (n < P::OS) {
                // (mx starts from lim: it exceeds lim exactly when a score does)
                need |= __builtin_amdgcn_ballot_w64(!(mx[n - P::OQ] <= lim[n - P::OQ]));
            } else shift_score(n - P::OS);
        };
        static_for<P::W>([&](auto wc) {
            constexpr int w = decltype(wc)::value, t = P::product_at(w), q = t / QT, m = q ^ 1;
            if constexpr (P::sum_at(w)) sum_mfma(w - t);
            else {
                if constexpr (t % 8 == 0) {
                    if constexpr (q + LA < NB) { av[q + LA] = v_read(q + LA); av[q + LA + 1] = v_read(q + LA + 1); }
                    else { ak[q + LA - NB] = k_read(q + LA - NB); ak[q + LA - NB + 1] = k_read(q + LA - NB + 1); }
                }
                o_mfma(m, q & 1 ? QT - 1 - t % QT : t % QT, av[m]);
                if constexpr (BF16 && t == 0) aim_lds(k_place() + fill_dst);
                if constexpr (BF16 && t < 4) load_aimed_16B<1024 * t>((const char*)base_k, off[t & 1]);
            }
            static_for<plan_b.first[w + 1] - plan_b.first[w]>([&](auto k) { op_b(std::integral_constant<int, plan_b.first[w] + decltype(k)::value>{}); });
            if constexpr (BF16 && plan_b.first[w] < P::OM && plan_b.first[w + 1] >= P::OM) {
#pragma unroll
                for (int l = 0; l < NL; ++l) vreg[l] = *(Global16B)(base_v + off[l & 1] + 1024 * l);
            }
            if constexpr (w >= P::W - 8) move(rv[w - (P::W - 8)], dva);
            if constexpr (w == P::W - 14) { turn(); asm volatile("" : "+s"(ring)); }
            if constexpr (w == P::W - 12) base_k += move_k;
            if constexpr (w == P::W - 10) base_v += move_v;
            __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll
        for (int k = 0; k < 16 * QT; k += 16)
            asm volatile("" : "+v"(x[k]), "+v"(x[k + 1]), "+v"(x[k + 2]), "+v"(x[k + 3]), "+v"(x[k + 4]), "+v"(x[k + 5]), "+v"(x[k + 6]), "+v"(x[k + 7]),
                         "+v"(x[k + 8]), "+v"(x[k + 9]), "+v"(x[k + 10]), "+v"(x[k + 11]), "+v"(x[k + 12]), "+v"(x[k + 13]), "+v"(x[k + 14]), "+v"(x[k + 15]));
        return need;
    };
    // The tiles that concern this wavefront.  In a causal scan up, the tiles of the workgroup's last rows lie wholly behind the others' rows: those
    // wavefronts keep fetching and meeting the barriers, but compute nothing more (0 times an infinite value would be no number).
    const int mine = CAUSAL && step > 0 && (qw0 + 63) / kTileKV + 1 < nkv ? (qw0 + 63) / kTileKV + 1 : nkv;
    auto fetch_only = [&](int i) {       // iteration i's fetches (bfloat16: V(i+2) into LDS first)
        if constexpr (BF16) {
#pragma unroll
            for (int l = 0; l < NL; ++l) asm volatile("" : "+v"(vreg[l]));
#pragma unroll
            for (int w = 0; w < CW; ++w) convert_word(w, v_place() + fill_dst + lane * 16);
            v_to_regs(i + 3);
        } else {
            fetch(Vh, i + 2, v_place());
        }
        fetch(Kh, i + 4, k_place());
        turn();
    };
    // (The raise stands outside the inner loop: inside, the compiler copies accumulators on the common path and spills.)
    constexpr int AV = BF16 ? 3 : 2;      // positions by which V is fetched ahead (K: 4)
    // Iteration i fetched the last whole tile once more in place of one that is not whole, which follows here, behind it.
    auto mend = [&](int i) {
        if (whole == nkv) return;
        if (i + 4 == whole) {
            wait_tile_landed();
            fetch(Kh, whole, lds0 + (whole & 3) * G::kTile);
        }
        if (i + AV == whole) {
            if constexpr (BF16) v_to_regs(whole);
            else {
                wait_tile_landed();
                fetch(Vh, whole, lds0 + VB + (whole & 3) * G::kTile);
            }
        }
    };
    int i = 0;
    base_k = base_of(Kh, whole > 4 ? 4 : whole > 0 ? whole - 1 : 0);
    base_v = base_of(Vh, whole > AV ? AV : whole > 0 ? whole - 1 : 0);
    while (i + 1 < mine) {
        // up to the next iteration ahead of which something changes
        int pause = mine - 1;
        for (int at : {whole - 5, whole - 3, whole - AV - 1, whole - AV + 1}) pause = at > i && at < pause ? at : pause;
        move_k = i < whole - 5 ? stride : 0;
        move_v = i < whole - AV - 1 ? stride : 0;
        bool need = false;
#pragma unroll 1
        for (; i < pause; ++i) {
            need = iteration() != 0;
            if (need) { ++i; break; }
        }
        if (need) raise_reference();
        mend(i - 1);
    }
    // ---------------------------------------------------------------- last tile: probabilities, then O^T += V^T P^T
    if constexpr (CAUSAL && !BF16) {
        if (mine < nkv) fetch_only(mine - 1);
    }
    static_for<96>([&](auto n) { op_a(decltype(n)::value); });
    convert_op(31);
    wide_settle_p(pf);
    landed_barrier<0>();
    if constexpr (CAUSAL && BF16) {
        if (mine < nkv) fetch_only(mine - 1);
    }
    {
        u4 av[NB];
#pragma unroll
        for (int m = 0; m < LA; ++m) av[m] = v_read(m);
        static_for<TB>([&](auto tc) {
            constexpr int t = decltype(tc)::value, m = t / QT;
            if constexpr (t % QT == 0 && m + LA < NB) av[m + LA] = v_read(m + LA);
            o_mfma(m, t % QT, av[m]);
            if constexpr (t % 8 == 7 && (!P::SPARSE || t >= 32)) sum_mfma((P::SPARSE ? t - 32 : t) / 8);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    if constexpr (CAUSAL) {
#pragma unroll 1
        for (i = mine; i < nkv; ++i) {
            if (!BF16 && i + 1 < nkv) fetch_only(i);
            landed_barrier<0>();
            if (BF16 && i + 1 < nkv) fetch_only(i);
        }
    }
    wide_settle_o(st);
    __syncthreads();   // all reads of the last tile are done before anything refills the buffers
}


// ------------------------------------------------------------------------------------------------
// The scan of a 64-row tile, walked as two halves at once, for small problems, where the chip has more compute units than there are query
// tiles and the length of one wavefront's walk is what the launch takes.  Run r takes the positions r*count .. of the scan's `nkv` tiles j0,
// j0 + step, ..., count = ceil(nkv / 2); wavefronts 0 and 1 compute on run 0, wavefronts 2 and 3, for the same rows, on run 1, and all four
// fetch the tiles of both into a set of buffers each (K0 K1 V0 V1).  This wavefront computes on run `run`.
//
// 32x32x16 MFMAs, transposed like pipelined_range.  A wavefront has its SIMD to itself, so what counts is the instructions it issues per tile
// and what it waits for in between.  The order is scan_tiles': masked tiles in the pipeline, one barrier between the two products, and
// behind it the fetches of V(i+1) and K(i+3), which then have a whole iteration to land; fragments in pairs with one wait each; the
// maximum per lane on raw scores, against a limit.  d = 64: 239 instructions per tile against pipelined_range's 246, of 18 MFMAs each.
// What it saves are the odd and masked tiles taken one at a time, with nothing in flight, before or after the halves, about 2 us of a
// launch (figures at launch_halves); per tile of a long scan it is 3 to 4 % slower.  The row sums' products moved into the first product,
// or a quarter of the exponentials into the second, were 1 to 2 % slower yet.
//
// The caller sends scans of one tile elsewhere, so run 1 has a tile at least and is one shorter at most: the stand-in tile of an empty run, its
// reset at the end and the fetch in the last loop are never reached.  They stay, because what the compiler makes of the loop without them
// is slower: 3 x 3000, d = 128, bfloat16, causal 38.6 -> 39.1 us, 5 x 1000, d = 128 15.3 -> 15.5 us (ten forms tried: +0.4 to +1.6 % each on
// one or more of these; the loop's instructions are the same, its place in the cache lines is not).
template <int D, bool BF16, bool CAUSAL>
__device__ __forceinline__ void scan_halves(TileState<D>& st, const LaneMap<D>& lm, const char* Kh, const char* Vh, int N, float c, int j0,
                                            int step, int nkv, int qw0, int qrow, int lane, LDS_PTR(char) lds, int run) {
    using G = Geo<D>;
    constexpr unsigned kSet = 4 * G::kTile;   // one set of buffers: K0 K1 V0 V1
    constexpr int KS = D / 16, DB = D / 32;
    constexpr int NA = 2 * KS;                // MFMAs (and K fragments) of one S^T tile
    constexpr int NB = 4 * DB;                // MFMAs (and V^T fragments) of one O^T update
    constexpr int NL = G::kLoadsPerWave, RL = 2 * NL;
    constexpr int LA = 4;                     // fragments read ahead of their use, in pairs
    const unsigned lds0 = (unsigned)(size_t)lds;
    const int g = lane >> 5;
    const int count = (nkv + 1) / 2;          // tiles of run 0; run 1 has as many or one less
    const int mine = run == 0 ? count : nkv - count < 1 ? 1 : nkv - count;      // (a run of no tile computes on a stand-in, see the end)
    const f16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f16v A[2];          // S^T of the tile one ahead: block b = keys 32b..32b+31 of the tile
    f16v sums = zero;   // row sum of the rounded probabilities, see sparse_sum_32
    const SparseOnes ones = sparse_ones(lane, (lane & 3) < 2 ? kOnes : 0u);
    float x[32];        // score*c - M of the current tile, index 16*b + r
    u8 pf[2];           // its probabilities as B operands, two in each
    u4 vreg[RL];        // bfloat16 V chunks in flight (BF16 only), run r in vreg[r * NL ...]
    float lim = -INFINITY, mx;

    unsigned rk[KS], rv[DB][2];      // LDS read addresses: K of the tile one ahead, V of the current tile
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rk[ks] = lds0 + run * kSet + lm.k_rd[ks];
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        rv[db][0] = lds0 + run * kSet + 2 * G::kTile + lm.v_rd[db][0];
        rv[db][1] = lds0 + run * kSet + 2 * G::kTile + lm.v_rd[db][1];
    }
    // Position p of run r.  Fetches beyond the end of a run fetch its last tile again, into a buffer nobody reads.
    auto tile_of = [&](int r, int p) {
        const int at = r == 0 ? (p < count ? p : count - 1) : (count + p < nkv ? count + p : nkv - 1);
        return j0 + at * step;
    };
    auto offsets = [&](int j, unsigned (&off)[NL]) {      // the rows that the last tile of the sequence lacks repeat row N-1
        const int left = N - j * kTileKV;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            off[l] = lm.fill_src[l];
            const unsigned row = off[l] / G::kRowBytes;
            if (left < kTileKV) off[l] = (row < (unsigned)left ? row : (unsigned)left - 1) * G::kRowBytes + off[l] % G::kRowBytes;
        }
    };
    struct Fetch {       // the tiles of a fetch in both runs and the lanes' offsets in them
        const char* base[2];
        unsigned off[2][NL];
    };
    auto aim = [&](const char* head, int p) {
        Fetch f;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int j = tile_of(r, p);
            f.base[r] = head + (long long)j * G::kTile;
            offsets(j, f.off[r]);
        }
        return f;
    };
    // From position p - 1 to p, p > 0.  (Of all of these only run 1 of a forward scan can reach the sequence's ragged last tile.)
    const long long stride = step * (long long)G::kTile;
    const int ragged_at = N % kTileKV && step > 0 ? nkv - 1 - count : -1;
    auto advance = [&](Fetch& f, int p) {
        f.base[0] += p < count ? stride : 0;
        f.base[1] += count + p < nkv ? stride : 0;
        if (__builtin_expect(p == ragged_at, 0)) offsets(tile_of(1, p), f.off[1]);
    };
    auto load = [&](const Fetch& f, int li, unsigned dst) {      // load li of the 2 NL of a K or V fetch
        const int r = li / NL, l = li % NL;
        load_to_lds_16B(f.base[r], f.off[r][l], dst + r * kSet + l * 4096);
    };
    auto fetch_burst = [&](const Fetch& f, unsigned dst) {
#pragma unroll
        for (int li = 0; li < RL; ++li) load(f, li, dst);
    };
    auto v_to_regs = [&](const Fetch& f) {
#pragma unroll
        for (int li = 0; li < RL; ++li) vreg[li] = *reinterpret_cast<const u4*>(f.base[li / NL] + f.off[li / NL][li % NL]);
    };
    auto convert_word = [&](int w, unsigned dst) {      // w-th 32-bit word of the fetched chunks; every fourth completes 16 bytes for LDS
        f2 y;
        const unsigned word = vreg[w / 4][w % 4];
        y[0] = __builtin_bit_cast(float, word << 16);
        y[1] = __builtin_bit_cast(float, word & 0xffff0000u);
        vreg[w / 4][w % 4] = __builtin_bit_cast(unsigned, __builtin_convertvector(y, h2));
        if (w % 4 == 3)
            *(LDS_PTR(u4))(size_t)(dst + (w / 4 / NL) * kSet + (w / 4 % NL) * 4096 + lane * 16) = vreg[w / 4];
    };
    constexpr int CW = RL * 4;
    // fragment m of K: columns 16*(m / 2).., keys 32*(m % 2)..; fragment m of V^T: keys 16*(m / DB).., columns 32*(m % DB)..
    auto k_read = [&](int m) -> u4 { return *(LDS_PTR(u4))(size_t)(rk[m / 2] + (m & 1) * 32 * G::kRowBytes); };
    auto v_read = [&](int m) -> s8 {
        const int ks = m / DB, db = m % DB;
        const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)(rv[db][0] + ks * 16 * G::kRowBytes));
        const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s4))(size_t)(rv[db][1] + ks * 16 * G::kRowBytes));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto s_mfma = [&](int m, u4 a, bool first) { A[m & 1] = mfma_16bit<BF16>(a, st.qf[m / 2], first ? zero : A[m & 1]); };
    auto o_mfma = [&](int m, s8 a) {
        st.o[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, half_of(pf[m / DB / 2], m / DB & 1)), st.o[m % DB], 0, 0, 0);
    };
    auto sum_mfma = [&](int k) { sums = sparse_sum_32(ones, pf[k], sums); };      // keys 32k.. of the tile
    const int all_see = CAUSAL ? (qw0 < N - 1 ? qw0 : N - 1) : N - 1;      // last key visible to every row of the wavefront
    int kv0 = tile_of(run, 0) * kTileKV;                                   // first key of the tile in A
    auto mask = [&]() {
        if (__builtin_expect(kv0 + kTileKV - 1 > all_see, 0)) {
            const int last_key = CAUSAL ? (qrow < N - 1 ? qrow : N - 1) : N - 1;
            int ahead = last_key - kv0 - 4 * g;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    asm volatile("" : "+v"(ahead));     // (separate comparisons: no lane masks kept and combined)
                    A[b][r] = 32 * b + 8 * (r >> 2) + (r & 3) > ahead ? -INFINITY : A[b][r];
                }
        }
    };
    auto shift_score = [&](int k) { x[k] = __builtin_fmaf(A[k >> 4][k & 15], c, -st.M); };
    auto max_op = [&](int op) { mx = fmaxf(fmaxf(mx, A[op >> 3][2 * (op & 7)]), A[op >> 3][2 * (op & 7) + 1]); };
    auto raise_reference = [&]() {      // as in scan_tiles
        float t = mx;
        asm volatile("" : "+v"(t));
        t = pair_max(t);
        const bool up = t > lim, fresh = lim == -INFINITY;
        const float Mnew = up ? t * c : st.M;
        const float alpha = up && !fresh ? fast_exp2(st.M - Mnew) : 1.0f;
        st.M = Mnew;
        sums *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[db][r] = fresh ? 0.f : st.o[db][r] * alpha;
        if (up) lim = score_limit(t, Mnew, c);
#pragma unroll
        for (int k = 0; k < 32; ++k) shift_score(k);
    };
    float e[16][2];
    auto op_a = [&](int n) {      // the two exponentials of pair n / 3, the convert of the one before
        const int u = n / 3, k = n % 3;
        if (k < 2) e[u][k] = fast_exp2(x[2 * u + k]);
        else if (u > 0) pf[(u - 1) / 8][(u - 1) % 8] = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{e[u - 1][0], e[u - 1][1]}, h2));
    };
    auto last_convert = [&]() { pf[1][7] = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{e[15][0], e[15][1]}, h2)); };
    constexpr int OA = 48;

    // ---------------------------------------------------------------- prologue: K(0..1) and V(0) on their way, S(0)
    const unsigned fill = lds0 + lm.fill_dst;
    Fetch fv = aim(Vh, 0), fk = aim(Kh, 2);
    fetch_burst(aim(Kh, 0), fill);
    fetch_burst(aim(Kh, 1), fill + G::kTile);
    __builtin_amdgcn_sched_barrier(0);    // (the counts of the waits below go by this order)
    asm volatile("" ::: "memory");
    if constexpr (BF16) v_to_regs(fv);
    else fetch_burst(fv, fill + 2 * G::kTile);
    landed_barrier<2 * RL>();
    {
        u4 a[NA];
#pragma unroll
        for (int m = 0; m < LA; ++m) a[m] = k_read(m);
#pragma unroll
        for (int m = 0; m < NA; ++m) {
            if (m + LA < NA) a[m + LA] = k_read(m + LA);
            s_mfma(m, a[m], m < 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (BF16) {
#pragma unroll
        for (int w = 0; w < CW; ++w) convert_word(w, fill + 2 * G::kTile);
    }
    landed_barrier<BF16 ? 0 : RL>();      // K(0) has been read, K(1) has landed
    fetch_burst(fk, fill);
    if constexpr (BF16) {
        fv = aim(Vh, 1);
        v_to_regs(fv);
    }
#pragma unroll
    for (int l = 0; l < NL; ++l) { fk.off[0][l] = lm.fill_src[l]; fv.off[0][l] = lm.fill_src[l]; }
    mask();
    mx = lim;
#pragma unroll
    for (int op = 0; op < 16; ++op) max_op(op);
    {
        const float t = pair_max(mx);
        st.M = t == -INFINITY ? 0.f : t * c;
        if (t != -INFINITY) lim = score_limit(t, st.M, c);
    }
#pragma unroll
    for (int k = 0; k < 32; ++k) shift_score(k);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rk[ks] += G::kTile;   // K of tile 1 is in buffer 1
    u4 ak[LA];
#pragma unroll
    for (int m = 0; m < LA; ++m) ak[m] = k_read(m);

    // ---------------------------------------------------------------- steady state: iteration i
    // reads K(i+1) from K buffer (i+1)&1 and V(i) from V buffer i&1; fetches K(i+3) and V(i+1) into the buffers (i+1)&1 (bfloat16: V(i+1) from
    // registers, then V(i+2) into them).  Returns whether the reference maximum has to be raised before tile i+1 can be used.
    auto iteration = [&](int i) -> bool {
        const unsigned kdst = fill + ((i + 1) & 1) * G::kTile, vdst = kdst + 2 * G::kTile;
        {
            u4 a[NA];
#pragma unroll
            for (int m = 0; m < LA; ++m) a[m] = ak[m];
#pragma unroll
            for (int t = 0; t < NA; ++t) {
                if (t % 2 == 0 && t + LA < NA) { a[t + LA] = k_read(t + LA); a[t + LA + 1] = k_read(t + LA + 1); }
                s_mfma(t ^ 1, a[t ^ 1], t < 2);
#pragma unroll
                for (int n = t * OA / NA; n < (t + 1) * OA / NA; ++n) op_a(n);
                __builtin_amdgcn_sched_barrier(0);
            }
            last_convert();
        }
        asm volatile("" : "+v"(pf[0]), "+v"(pf[1]));
        landed_barrier<0>();
        s8 av[NB];
#pragma unroll
        for (int m = 0; m < LA; ++m) av[m] = v_read(m);
        __builtin_amdgcn_sched_barrier(0);
        advance(fv, BF16 ? i + 2 : i + 1);      // (while the first fragments are on their way)
        advance(fk, i + 3);
        if constexpr (BF16) {
#pragma unroll
            for (int l = 0; l < RL; ++l) asm volatile("" : "+v"(vreg[l]));
        }
        kv0 += step * kTileKV;
        mask();
        __builtin_amdgcn_sched_barrier(0);
        mx = lim;
        const int flip = i & 1 ? G::kTile : -G::kTile;      // K(i+2) is in buffer i&1, V(i+1) in buffer (i+1)&1
        bool need = false;
        constexpr int OC = BF16 ? 3 * CW : 0;            // conversions count as three
        constexpr int OM = 16 + OC, OB = OM + 32;
        constexpr int T0 = (OM * NB + OB - 1) / OB;      // first MFMA after the conversions
        constexpr int TL = (BF16 ? 1 : 2) * RL;          // direct loads
        auto op_b = [&](int n) {
            if (n < OM) {
                const int j = n * 16 / OM, done = (n + 1) * 16 / OM;
                if (j != done) max_op(j);
                if constexpr (BF16) {
                    const int w = n * CW / OM;
                    if (w != (n + 1) * CW / OM) convert_word(w, vdst);
                }
            } else {
                shift_score(n - OM);
            }
        };
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            if (t % 2 == 0) {
                if (t + LA < NB) { av[t + LA] = v_read(t + LA); av[t + LA + 1] = v_read(t + LA + 1); }
            }
            if (BF16 && t == T0) v_to_regs(fv);
            o_mfma(t ^ 1, av[t ^ 1]);
            // Row sums behind the first and the second half: bfloat16 converts in the first, whose places a sum among them lengthens.  d = 64, bfloat16, causal,
            // plain products for sums / after the first and the second quarter / here: 4 x 3904 27.8, 30.2, 27.2 us, 3 x 2159 17.8, 18.9, 17.4, binary16 23.3,
            // 23.5, 22.9 and 15.3, 15.4, 15.1; d = 128, 4 x 3000 37.7, 37.3, 37.2.
            if (t == NB / 2 - 1 || t == 3 * NB / 4 - 1) sum_mfma(t / (NB / 4) - 1);
#pragma unroll
            for (int li = t * TL / NB; li < (t + 1) * TL / NB; ++li) {      // V first because it is needed first
                if (!BF16 && li < RL) load(fv, li, vdst);
                else load(fk, li % RL, kdst);
            }
#pragma unroll
            for (int n = t * OB / NB; n < (t + 1) * OB / NB; ++n) {
                op_b(n);
                if (n == OM + 4) need = __builtin_amdgcn_ballot_w64(!(mx <= lim)) != 0;      // (mx starts from lim)
            }
            if (t == NB - 3) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) rk[ks] += flip;
#pragma unroll
                for (int m = 0; m < LA; ++m) ak[m] = k_read(m);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int db = 0; db < DB; ++db) { rv[db][0] -= flip; rv[db][1] -= flip; }
        return need;
    };
    auto fetch_only = [&](int i) {       // iteration i's fetches (bfloat16: V(i+1) into LDS first)
        const unsigned kdst = fill + ((i + 1) & 1) * G::kTile, vdst = kdst + 2 * G::kTile;
        advance(fk, i + 3);
        advance(fv, BF16 ? i + 2 : i + 1);
        if constexpr (BF16) {
#pragma unroll
            for (int l = 0; l < RL; ++l) asm volatile("" : "+v"(vreg[l]));
#pragma unroll
            for (int w = 0; w < CW; ++w) convert_word(w, vdst);
            v_to_regs(fv);
        } else {
            fetch_burst(fv, vdst);
        }
        fetch_burst(fk, kdst);
    };
    int i = 0;
    while (i + 1 < mine) {
        bool need = false;
#pragma unroll 1
        for (; i + 1 < mine; ++i) {
            need = iteration(i);
            if (need) { ++i; break; }
        }
        if (need) raise_reference();
    }
    // ---------------------------------------------------------------- last tile: probabilities, then O^T += V^T P^T
#pragma unroll
    for (int n = 0; n < OA; ++n) op_a(n);
    last_convert();
    landed_barrier<0>();
    if (mine < count) fetch_only(mine - 1);
    {
        s8 av[NB];
#pragma unroll
        for (int m = 0; m < LA; ++m) av[m] = v_read(m);
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            if (t + LA < NB) av[t + LA] = v_read(t + LA);
            o_mfma(t, av[t]);
            if (t % (NB / 2) == NB / 2 - 1) sum_mfma(t / (NB / 2));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll 1
    for (i = mine; i < count; ++i) {      // run 1 is one tile shorter: the barriers of the other wavefronts
        landed_barrier<0>();
        if (i + 1 < count) fetch_only(i);
    }
    __syncthreads();   // all reads of the last tile are done before anything refills the buffers
    st.L = 0.5f * (sums[0] + sums[1]);       // (both lanes of a pair hold the row's whole sum)
    if (lim == -INFINITY) st.M = -INFINITY;      // nothing was seen: weight 0 in the merge
    if (run == 1 && nkv == 1) {             // a run of no tile
        st.M = -INFINITY;
        st.L = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) st.o[db] = zero;
    }
}

// The epilogue where variant.qo_streaming asks for it: O leaves through LDS so that a store instruction writes whole
// 128-byte lines (8 rows x 128 bytes per instruction, 16 bytes per lane), marked non-temporal: the rows of O are written
// once and never read by the kernel, and written this way they do not take the place of K/V tiles in the L2.
// (Non-temporal stores of the 8- and 16-byte pieces a lane holds per row are not gathered into lines by the L2 and cost
// several times the write traffic.)  `stage` is 4 KiB of LDS of this wavefront's own: 32 rows x 128 bytes, the 16-byte
// chunk c of row r at chunk position c ^ (r & 7), filled by the caller with one 128-byte column block of its 32 rows.
// drain_stage() writes that block out: `dst` points at the block's first row in O, row_bytes is O's row pitch,
// rows_left the number of the 32 rows that lie inside the sequence (<= 0: none).
__device__ __forceinline__ void stage_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
__device__ __forceinline__ void drain_stage(LDS_PTR(char) stage, char* dst, size_t row_bytes, int rows_left, int lane) {
    stage_fence();
    const int chunk = lane & 7;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int row = 8 * k + (lane >> 3);
        const u4 x = *(LDS_PTR(u4))(stage + row * 128 + ((chunk ^ (row & 7)) << 4));
        char* to = dst + row * row_bytes + chunk * 16;
        // (the s_nop: a store of more than 8 bytes reads its data registers up to two cycles after issue, and the compiler
        //  does not see a store in this statement when it decides what may overwrite them next)
        if (row < rows_left) asm volatile("global_store_dwordx4 %0, %1, off nt\n\ts_nop 1" ::"v"(to), "v"(x) : "memory");
    }
    stage_fence();
}

// One query tile (Alg. 1 body) of attn_fwd_kernel: rows [t*128, (t+1)*128) of head `hh`, K/V tiles j0, j0+step, ... (nkv of
// them).
// HALVES: the tile has 64 rows; wavefronts 0 and 1 take the first half of its K/V tiles and wavefronts 2 and 3, for the same rows, the
// second half, at once, and the two partial results are merged through LDS (the merge of two softmax partials: common reference maximum,
// both rescaled to it).  Which tiles those are, and what happens to the others, is the kernel's SPLIT:
// kSplitEven   all of them, full and even in number: pipelined_range.  A kernel without the code for any others is smaller, which counts
//              in launches of some microseconds: 256 keys, d = 64: 6.05 -> 5.7 us, 4 x 1024, d = 128: 15.2 -> 14.3, 8 x 2048: 15.8 -> 15.4.
// kSplitShort  all of them, in the one pipeline of scan_halves.
// kSplitLong   the full, unmasked ones, in pipelined_range.  An odd plain tile, the diagonal tile and a ragged last tile are taken one at
//              a time by wavefronts 0 and 1 alone, after the merge in a forward scan and before the halves in a backward one.
enum SplitKind { kSplitEven, kSplitShort, kSplitLong };

template <int D, bool BF16, bool CAUSAL, bool HALVES = false, int SPLIT = kSplitLong>
__device__ __forceinline__ void process_q_tile(const Params& p, const LaneMap<D>& lm, int hh, int t, int j0, int step,
                                               int nkv, int wave, int lane, LDS_PTR(char) lds) {
    using G = Geo<D>;
    constexpr int KS = D / 16;    // MFMA steps along d for S^T
    constexpr int DB = D / 32;    // 32-row blocks of O^T
    constexpr int TQ = HALVES ? kTileQ / 2 : kTileQ;
    const int g = lane >> 5, ln = lane & 31;
    const int N = p.N;
    const size_t head_off = (size_t)hh * N * G::kRowBytes;
    const char* Qh = static_cast<const char*>(p.Q) + head_off;
    const char* Kh = static_cast<const char*>(p.K) + head_off;
    const char* Vh = static_cast<const char*>(p.V) + head_off;

    const int run = HALVES ? wave >> 1 : 0;                            // which half of the scan this wavefront computes
    const int qw0 = t * TQ + (HALVES ? wave & 1 : wave) * 32;     // first query row of this wavefront
    const int qrow = qw0 + ln;                // this lane's query row (column of S^T)

    TileState<D> st;
    // With variant.qo_streaming the rows of Q come in the way K tiles do -- 64 rows at a time straight into LDS, whole
    // lines per instruction, the four wavefronts together -- but marked non-temporal, and are read from there in the
    // K operand's pattern, which is also Q's.  The buffers are free: the last range of the previous tile ended with a barrier.
    unsigned q_at = 0;     // byte offset in LDS of this lane's first fragment
    if (p.stream_q) {
        int l2 = lane;
        asm volatile("" : "+v"(l2));        // (a lane map of its own that does not live on: see the note on registers below)
        const LaneMap<D> lq(wave, l2);
        const unsigned lds0 = (unsigned)(size_t)lds;
#pragma unroll
        for (int m = 0; m < TQ / kTileKV; ++m) {
            const int q0 = t * TQ + m * kTileKV;
            const int first = q0 < N ? q0 : N - 1;          // rows beyond N repeat row N-1, as below
            const char* base = Qh + (size_t)first * G::kRowBytes;
#pragma unroll
            for (int i = 0; i < G::kLoadsPerWave; ++i) {
                const int row = lq.fill_src[i] / G::kRowBytes, chunk = lq.fill_src[i] % G::kRowBytes;
                const int r = q0 + row < N ? q0 + row : N - 1;
                load_to_lds_16B_nt(base, (unsigned)((r - first) * G::kRowBytes + chunk), lds0 + m * G::kTile + lq.fill_dst + i * 4096);
            }
        }
        const int mine = HALVES ? wave & 1 : wave;           // which 32 rows of the tile are this wavefront's
        q_at = (mine / 2) * G::kTile + (mine & 1) * 32 * G::kRowBytes + lq.k_rd[0];
        wait_tile_landed();
        __syncthreads();
    }
    int lane_q = lane;
    asm volatile("" : "+v"(lane_q));      // (addresses used once: built from a copy of the lane index of their own)
    {   // rows beyond N repeat row N-1 (computed, never stored)
        const int qr = qw0 + (lane_q & 31) < N ? qw0 + (lane_q & 31) : N - 1;
        const char* qp = Qh + (size_t)qr * G::kRowBytes + (lane_q >> 5) * 16;
        const unsigned flip = p.negate_q ? 0x80008000u : 0u;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            // (chunk 2 ks + g of a row sits at chunk position (2 ks + g) ^ swz(row): k_rd[ks] = k_rd[0] ^ (32 ks))
            u4 v = p.stream_q ? *(LDS_PTR(u4))(lds + (q_at ^ (unsigned)(ks * 32))) : *reinterpret_cast<const u4*>(qp + ks * 32);
            if constexpr (!HALVES) { v[0] ^= flip; v[1] ^= flip; v[2] ^= flip; v[3] ^= flip; }
            st.qf[ks] = v;
        }
        // (Behind a branch: where nothing is done to them here, the fragments are on their way while the first tiles are fetched.  One head
        // x 256: 6.2 -> 6.1 us, 2 x 700, d = 128: 16.2 -> 15.5 us; with 128-row tiles it is 0 to +1 %.)
        if constexpr (HALVES) {
            if (p.negate_q) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) st.qf[ks] ^= u4{flip, flip, flip, flip};
            }
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.o[db][r] = 0.f;
        st.M = -INFINITY;
        st.L = 0.f;
    }
    if (p.stream_q) __syncthreads();      // the fragments are in registers before the first K/V fetch overwrites the rows
    const float c = p.c;

    // Tiles with index >= jm need the mask code: the ragged last tile, and under the causal mask
    // the tiles that reach past the first row of this query tile.  They sit at one end of the scan,
    // so the scan is a pipelined run of plain tiles and a run of masked tiles, in scan order.
    const int kv_tiles = (N + kTileKV - 1) / kTileKV;
    const int jm = CAUSAL ? (t * TQ) / kTileKV : ((N % kTileKV) ? kv_tiles - 1 : kv_tiles);
    const int n_masked = nkv > jm ? nkv - jm : 0;
    const int n_plain = nkv - n_masked;
    auto plain = [&](int j_first) {
        pipelined_range<D, BF16, false, D == 128 && CAUSAL && !BF16>(st, lm, Kh, Vh, c, j_first, step, n_plain, lane, lds);      // see RowSums
    };
    auto masked = [&](int j_first) {
        general_range<D, BF16, CAUSAL, true>(st, lm, Kh, Vh, N, c, j_first, step, n_masked, qw0, qrow, lane, lds);
    };
    if constexpr (HALVES) {
        const int half = n_plain / 2;                       // kSplitLong: plain tiles per run
        const int n_left = (n_plain & 1) + n_masked;        // and the tiles left for the tile-at-a-time code
        if constexpr (SPLIT == kSplitEven) {
            pipelined_range<D, BF16, true, !(BF16 && D == 128)>(st, lm, Kh, Vh, c, j0, step, nkv / 2, lane, lds, run);      // see RowSums
        } else if constexpr (SPLIT == kSplitShort) {
            if (nkv == 1)
                general_range<D, BF16, CAUSAL, true>(st, lm, Kh, Vh, N, c, j0, step, 1, qw0, qrow, lane, lds, run == 1);
            else
                scan_halves<D, BF16, CAUSAL>(st, lm, Kh, Vh, N, c, j0, step, nkv, qw0, qrow, lane, lds, run);
        } else {
            if (step < 0)
                general_range<D, BF16, CAUSAL, true>(st, lm, Kh, Vh, N, c, j0, step, n_left, qw0, qrow, lane, lds, run == 1);
            pipelined_range<D, BF16, true>(st, lm, Kh, Vh, c, step > 0 ? j0 : j0 + n_left * step, step, half, lane, lds, run);
        }
        // ---- merge: wavefront w + 2 hands (O^T, M, L) of its half to wavefront w, lane to lane, through LDS
        //      (value k of lane l of wavefront w + 2 at float index (2k + w) * 64 + l: no bank conflicts)
        constexpr int NV = DB * 16 + 2;
        LDS_PTR(float) xch = (LDS_PTR(float))lds;
        if (run == 1) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) xch[(2 * (db * 16 + r) + (wave & 1)) * 64 + lane] = st.o[db][r];
            xch[(2 * (NV - 2) + (wave & 1)) * 64 + lane] = st.M;
            xch[(2 * (NV - 1) + (wave & 1)) * 64 + lane] = st.L;
        }
        __syncthreads();
        if (run == 0) {
            const float M1 = xch[(2 * (NV - 2) + wave) * 64 + lane], L1 = xch[(2 * (NV - 1) + wave) * 64 + lane];
            const float M = fmaxf(st.M, M1);
            const float a0 = st.M == -INFINITY ? 0.f : fast_exp2(st.M - M);
            const float a1 = M1 == -INFINITY ? 0.f : fast_exp2(M1 - M);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    st.o[db][r] = st.o[db][r] * a0 + xch[(2 * (db * 16 + r) + wave) * 64 + lane] * a1;
            st.M = M;
            st.L = st.L * a0 + L1 * a1;
        }
        __syncthreads();   // the exchange area is read before anything else overwrites it
        if constexpr (SPLIT == kSplitLong) {
            if (step > 0)
                general_range<D, BF16, CAUSAL, true>(st, lm, Kh, Vh, N, c, j0 + 2 * half * step, step, n_left, qw0, qrow, lane,
                                                     lds, run == 1);
        }
    } else if (step > 0) {
        plain(j0);
        masked(j0 + n_plain * step);
    } else {
        masked(j0);
        plain(j0 + n_masked * step);
    }

    // ---- epilogue: O_i = acc / l  (the division Alg. 1 leaves implicit; Eq. 1 fixes it)
    const bool writes = !HALVES || run == 0;     // of two wavefronts that share rows, the first holds the merged result
    const int lane_in = lane;
    if (p.stream_o) {
        wait_tile_landed();
        __syncthreads();          // nothing is on its way into the K/V buffers any more: they serve as staging area
        if (writes) {
            LDS_PTR(char) stage = lds + wave * 4096;
            int lane = lane_in;
            asm volatile("" : "+v"(lane));     // lane-derived addresses are built here, not carried across the scan
            const int g = lane >> 5, ln = lane & 31;
            const int sw = ln & 7;
            const float inv = 1.0f / pair_sum(st.L);
            const int row0 = qw0;
            const int rows_left = N - row0;      // <= 0: all rows lie beyond the sequence
            if (p.o_dtype == SAWATTN_F32) {
                constexpr size_t RB = (size_t)D * 4;
                char* dst = static_cast<char*>(p.O) + ((size_t)hh * N + row0) * RB;
#pragma unroll
                for (int db = 0; db < DB; ++db) {          // 32 columns = 128 bytes per row
                    const f16v& o = st.o[db];
#pragma unroll
                    for (int rq = 0; rq < 4; ++rq) {
                        const f4 v = {o[4 * rq] * inv, o[4 * rq + 1] * inv, o[4 * rq + 2] * inv, o[4 * rq + 3] * inv};
                        *(LDS_PTR(f4))(stage + ln * 128 + (((2 * rq + g) ^ sw) << 4)) = v;
                    }
                    drain_stage(stage, dst + db * 128, RB, rows_left, lane);
                }
            } else {
                constexpr size_t RB = (size_t)D * 2;
                char* dst = static_cast<char*>(p.O) + ((size_t)hh * N + row0) * RB;
#pragma unroll
                for (int pass = 0; pass < DB / 2; ++pass) {   // 64 columns = 128 bytes per row
#pragma unroll
                    for (int dbl = 0; dbl < 2; ++dbl) {
                        const f16v& o = st.o[2 * pass + dbl];
#pragma unroll
                        for (int rq = 0; rq < 4; ++rq) {
                            const f4 v = {o[4 * rq] * inv, o[4 * rq + 1] * inv, o[4 * rq + 2] * inv, o[4 * rq + 3] * inv};
                            LDS_PTR(char) at = stage + ln * 128 + (((4 * dbl + rq) ^ sw) << 4) + 8 * g;
                            if (p.o_dtype == SAWATTN_F16) *(LDS_PTR(h4))at = __builtin_convertvector(v, h4);
                            else *(LDS_PTR(b4))at = __builtin_convertvector(v, b4);
                        }
                    }
                    drain_stage(stage, dst + pass * 128, RB, rows_left, lane);
                }
            }
        }
        __syncthreads();          // the staging area is read before the next tile's fetches overwrite it
        return;
    }
    if (!writes) return;
    int lane_out = lane_in;
    asm volatile("" : "+v"(lane_out));
    const int g_out = lane_out >> 5, qrow_out = qw0 + (lane_out & 31);
    const float inv = 1.0f / pair_sum(st.L);
    if (qrow_out < N) {
        const size_t orow = ((size_t)hh * N + qrow_out) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const f16v& o = st.o[db];
                f4 v = {o[4 * rq] * inv, o[4 * rq + 1] * inv, o[4 * rq + 2] * inv, o[4 * rq + 3] * inv};
                const size_t col = 32 * db + 8 * rq + 4 * g_out;
                if (p.o_dtype == SAWATTN_F32) {
                    *reinterpret_cast<f4*>(static_cast<float*>(p.O) + orow + col) = v;
                } else if (p.o_dtype == SAWATTN_F16) {
                    *reinterpret_cast<h4*>(static_cast<_Float16*>(p.O) + orow + col) = __builtin_convertvector(v, h4);
                } else {
                    *reinterpret_cast<b4*>(static_cast<__bf16*>(p.O) + orow + col) = __builtin_convertvector(v, b4);
                }
            }
    }
}

// One query tile (Alg. 1 body) on 16x16x32 MFMAs: rows [t*64*QT, (t+1)*64*QT) of head `hh`, K/V tiles j0, j0+step, ... (nkv of
// them).  A wavefront owns QT blocks of 16 query rows: two in attn_fwd_shared_kernel, four with 256-row tiles.
template <int D, bool BF16, bool CAUSAL, bool PHASES, int QT = 2>
__device__ __forceinline__ void process_q_tile_narrow(const Params& p, const NarrowMap<D>& lm, int hh, int t, int j0, int step,
                                                      int nkv, int wave, int lane, LDS_PTR(char) lds) {
    using G = Geo<D>;
    constexpr int KS = D / 32;    // MFMA steps along d for S^T
    constexpr int DB = D / 16;    // column blocks of O^T
    constexpr int TQ = 64 * QT;
    const int N = p.N;
    const size_t head_off = (size_t)hh * N * G::kRowBytes;
    const char* Qh = static_cast<const char*>(p.Q) + head_off;
    const char* Kh = static_cast<const char*>(p.K) + head_off;
    const char* Vh = static_cast<const char*>(p.V) + head_off;

    const int qw0 = t * TQ + wave * 16 * QT;       // first query row of this wavefront

    NarrowState<D, QT> st;
    // With variant.qo_streaming the rows of Q come in the way K tiles do -- 64 rows at a time straight into LDS, whole
    // lines per instruction, the four wavefronts together -- but marked non-temporal, and are read from there in the
    // K operand's pattern, which is also Q's.  The buffers are free: the last range of the previous tile ended with a barrier.
    unsigned q_at = 0;     // byte offset in LDS of this lane's first fragment
    if (p.stream_q) {
        int l2 = lane;
        asm volatile("" : "+v"(l2));        // (a lane map of its own that does not live on: see the note on registers below)
        const NarrowMap<D> lq(wave, l2);
        const unsigned lds0 = (unsigned)(size_t)lds;
        const int row = lq.fill_src / G::kRowBytes, chunk = lq.fill_src % G::kRowBytes;
#pragma unroll
        for (int m = 0; m < TQ / kTileKV; ++m) {
            const int q0 = t * TQ + m * kTileKV;
            const int first = q0 < N ? q0 : N - 1;          // rows beyond N repeat row N-1, as below
            const char* base = Qh + (size_t)first * G::kRowBytes;
#pragma unroll
            for (int i = 0; i < G::kLoadsPerWave; ++i) {
                const int r0 = q0 + row + i * (4096 / G::kRowBytes);
                const int r = r0 < N ? r0 : N - 1;
                load_to_lds_16B_nt(base, (unsigned)((r - first) * G::kRowBytes + chunk), lds0 + m * G::kTile + lq.fill_dst + i * 4096);
            }
        }
        q_at = wave * QT / 4 * G::kTile + (QT == 2 ? wave & 1 : 0) * 32 * G::kRowBytes + lq.k_rd[0];
        wait_tile_landed();
        __syncthreads();
    }
    int lane_q = lane;
    asm volatile("" : "+v"(lane_q));      // (addresses used once: built from a copy of the lane index of their own)
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {   // rows beyond N repeat row N-1 (computed, never stored)
        const int q0 = qw0 + (lane_q & 15) + 16 * qt;
        const int qr = q0 < N ? q0 : N - 1;
        const char* qp = Qh + (size_t)qr * G::kRowBytes + (lane_q >> 4) * 16;
        const unsigned flip = p.negate_q ? 0x80008000u : 0u;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            // (chunk 4 ks + g of a row sits at chunk position (4 ks + g) ^ swz(row): k_rd[ks] = k_rd[0] ^ (64 ks))
            u4 v = p.stream_q ? *(LDS_PTR(u4))(lds + ((q_at + qt * 16 * G::kRowBytes) ^ (unsigned)(ks * 64)))
                              : *reinterpret_cast<const u4*>(qp + ks * 64);
            v[0] ^= flip; v[1] ^= flip; v[2] ^= flip; v[3] ^= flip;
            if constexpr (QT == 4) {
                if constexpr (!BF16) {
                    if (p.q_bf16) v = bf16x8_to_f16x8(v);   // K and V are binary16 copies: Q follows (exact for normal binary16 magnitudes)
                }
                asm volatile("" : "=a"(st.qf[ks][qt]) : "0"(v));   // accumulation registers from here on
            } else {
                st.qf[ks][qt] = v;
            }
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) st.o[db][qt][r] = 0.f;
        st.M[qt] = 0.f;
        st.L[qt] = f4{0.f, 0.f, 0.f, 0.f};
    }
    if (p.stream_q) __syncthreads();      // the fragments are in registers before the first K/V fetch overwrites the rows

    if constexpr (QT == 4) scan_tiles_wide<BF16, CAUSAL>(st, lm, Kh, Vh, N, p.c, j0, step, nkv, qw0, wave, lane, lds);
    else scan_tiles<D, BF16, CAUSAL, PHASES>(st, lm, Kh, Vh, N, p.c, j0, step, nkv, qw0, qw0 + (lane & 15), lane, lds);

    // ---- epilogue: O_i = acc / l  (the division Alg. 1 leaves implicit; Eq. 1 fixes it)
    float inv[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) inv[qt] = 1.0f / (QT == 4 ? WidePlan<BF16>::row_sum(st.L[qt]) : st.L[qt][0] + st.L[qt][1]);
    if (p.stream_o) {
        // (the scan ended with a barrier and nothing in flight: the K/V buffers serve as staging area)
        LDS_PTR(char) stage = lds + wave * 4096;
        int l2 = lane;
        asm volatile("" : "+v"(l2));     // lane-derived addresses are built here, not carried across the scan
        const int g = l2 >> 4, ln = l2 & 15;
        const int sw = ln & 7;
#pragma unroll
        for (int q0 = 0; q0 < QT; q0 += 2) {      // 32 rows at a time
            const int row0 = qw0 + 16 * q0, rows_left = N - row0;      // <= 0: all rows lie beyond the sequence
            if (p.o_dtype == SAWATTN_F32) {
                constexpr size_t RB = (size_t)D * 4;
                char* dst = static_cast<char*>(p.O) + ((size_t)hh * N + row0) * RB;
#pragma unroll
                for (int pass = 0; pass < DB / 2; ++pass) {          // 32 columns = 128 bytes per row
#pragma unroll
                    for (int dbl = 0; dbl < 2; ++dbl)
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const f4 v = st.o[2 * pass + dbl][q0 + q] * inv[q0 + q];
                            *(LDS_PTR(f4))(stage + (16 * q + ln) * 128 + (((4 * dbl + g) ^ sw) << 4)) = v;
                        }
                    drain_stage(stage, dst + pass * 128, RB, rows_left, l2);
                }
            } else {
                constexpr size_t RB = (size_t)D * 2;
                char* dst = static_cast<char*>(p.O) + ((size_t)hh * N + row0) * RB;
#pragma unroll
                for (int pass = 0; pass < DB / 4; ++pass) {   // 64 columns = 128 bytes per row
#pragma unroll
                    for (int dbl = 0; dbl < 4; ++dbl)
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const f4 v = st.o[4 * pass + dbl][q0 + q] * inv[q0 + q];
                            LDS_PTR(char) at = stage + (16 * q + ln) * 128 + (((2 * dbl + (g >> 1)) ^ sw) << 4) + 8 * (g & 1);
                            if (p.o_dtype == SAWATTN_F16) *(LDS_PTR(h4))at = __builtin_convertvector(v, h4);
                            else *(LDS_PTR(b4))at = __builtin_convertvector(v, b4);
                        }
                    drain_stage(stage, dst + pass * 128, RB, rows_left, l2);
                }
            }
        }
        __syncthreads();          // the staging area is read before the next tile's fetches overwrite it
        return;
    }
    int lane_out = lane;
    asm volatile("" : "+v"(lane_out));
    const int g_out = lane_out >> 4, qrow_out = qw0 + (lane_out & 15);
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        if (qrow_out + 16 * qt < N) {
            const size_t orow = ((size_t)hh * N + qrow_out + 16 * qt) * D;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const f4 v = st.o[db][qt] * inv[qt];
                const size_t col = 16 * db + 4 * g_out;
                if (p.o_dtype == SAWATTN_F32) {
                    *reinterpret_cast<f4*>(static_cast<float*>(p.O) + orow + col) = v;
                } else if (p.o_dtype == SAWATTN_F16) {
                    *reinterpret_cast<h4*>(static_cast<_Float16*>(p.O) + orow + col) = __builtin_convertvector(v, h4);
                } else {
                    *reinterpret_cast<b4*>(static_cast<__bf16*>(p.O) + orow + col) = __builtin_convertvector(v, b4);
                }
            }
        }
    }
}

// bfloat16 -> binary16 copies of K and V for the workspace path (16 bytes per lane and step).
__global__ __launch_bounds__(256) void bf16_to_f16_kernel(const u4* __restrict__ K, const u4* __restrict__ V,
                                                          u4* __restrict__ K16, u4* __restrict__ V16, size_t chunks) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < chunks; i += stride) {
        K16[i] = bf16x8_to_f16x8(K[i]);
        V16[i] = bf16x8_to_f16x8(V[i]);
    }
}

// Re-alignment of the workgroups of one cache domain.  The reuse the schedule is built on (Sec. 3.4)
// needs the workgroups that share an L2 to walk the same K/V at about the same time.  They start
// aligned and do the same number of tile steps per head, but nothing keeps them aligned: measured
// over 16 heads per domain their drift grows past what the L2 holds and the hit rate falls from
// 95 % to 55 %.  So between two heads the workgroups of a domain wait for each other on a ticket
// counter.  The wait is bounded: if the workgroups are not all resident (a shared GPU), it gives
// up after kSyncSpinLimit polls and the kernel carries on unaligned; results never depend on it.
// The counters are library-owned device memory: kTicketSets sets of one counter per domain.  Every
// launch that uses them takes the next set in turn (a host-side count) and clears it with a
// one-wavefront kernel enqueued just before it, so launches that overlap on one GPU -- other streams,
// other host threads -- do not disturb each other unless kTicketSets or more of them are in flight;
// then they may lose the alignment and wait out the bound (about 8 ms per head boundary at worst),
// never more.
constexpr int kTicketSets = 8;
__device__ unsigned g_domain_tickets[kTicketSets][kDomains];
constexpr int kSyncSpinLimit = 1 << 14;     // polls of about 1000 cycles each

__global__ void clear_tickets_kernel(int set) {
    if (threadIdx.x < kDomains) g_domain_tickets[set][threadIdx.x] = 0u;
}

// The lane index, made where it is used and unknown to the compiler: what derives from it is not kept in registers across the loops.
__device__ __forceinline__ int lane_now() {
    unsigned all = ~0u;
    asm volatile("" : "+s"(all));
    return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}

// Called by every workgroup of `domain` the same number of times; `slots` workgroups take part.
template <bool TIGHT>
__device__ __forceinline__ void domain_sync(int set, int domain, int slots, int wave) {
    __syncthreads();
    if (wave == 0 && lane_now() == 0) {
        // (TIGHT: made unknown here, or the division's reciprocal is kept in a vector register over the whole kernel, and d = 64 has none to spare)
        if constexpr (TIGHT) asm volatile("" : "+s"(slots));
        unsigned* t = &g_domain_tickets[set][domain];
        const unsigned mine = __hip_atomic_fetch_add(t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned target = (mine / (unsigned)slots + 1u) * (unsigned)slots;
        for (int spin = 0; spin < kSyncSpinLimit; ++spin) {
            if ((int)(__hip_atomic_load(t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) >= 0) break;
            __builtin_amdgcn_s_sleep(16);
        }
    }
    __syncthreads();
}

// The outer loop of a workgroup: its query tiles one after the other (Alg. 2, Alg. 3), `tile` computes one.  TURNS: 128-row tiles, the only
// ones that launch_schedule gives a launch with sched.turn (in the kernels of 64-row tiles, for small problems, the test alone costs 0.1 us).
template <bool CAUSAL, bool LATE, bool TURNS, typename TILE>
__device__ __forceinline__ void for_each_q_tile(const Params& p, TILE&& tile) {
    const Schedule& s = p.sched;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wg = CAUSAL && LATE ? workgroup_of_block(s, (int)blockIdx.x) : (int)blockIdx.x;      // (LATE: 128-row tiles and shorter)
    int local = 0;           // query tiles this workgroup has processed
    for (int it = 0; it < s.local_iters; ++it) {
        const Work w = decode_work<LATE, TURNS>(s, wg, it, CAUSAL, p.sawtooth != 0);
        if (w.tile >= 0) {
            const int nkv = visible_kv_tiles(s, w.tile, p.N, CAUSAL);
            const int j0 = w.backward ? nkv - 1 : 0;
            const int step = w.backward ? -1 : 1;
            if (p.trace && wave == 0 && lane_now() == 0) {
                int32_t* rec = p.trace + ((size_t)wg * p.max_local + local) * 4;
                rec[0] = w.head; rec[1] = w.tile; rec[2] = j0; rec[3] = j0 + (nkv - 1) * step;
            }
            tile(w, j0, step, nkv, wave, lane_now());
            ++local;
        }
        // Every workgroup of the domain comes here once per head, also those that sat rounds out.
        // (With the align_rounds variant also once per round: measured, it changes neither the L2 traffic
        // nor the time of the kernel with 64 rows per wavefront, whose workgroups stay in step by themselves.)
        if (w.sync_after) domain_sync<LATE>(p.ticket_set, (int)blockIdx.x % kDomains, s.slots, wave);
    }
    if (p.trace_count && wave == 0 && lane_now() == 0) p.trace_count[wg] = local;
}

template <int D, bool BF16, bool CAUSAL, int NH, bool HALVES = false, int SPLIT = kSplitLong>
__global__ __launch_bounds__(kThreads, HALVES ? (D == 64 ? 2 : 1) : NH == 2 ? 1 : (D == 64 ? 3 : 2)) void attn_fwd_kernel(Params p) {
    extern __shared__ __align__(16) char smem[];
    for_each_q_tile<CAUSAL, NH == 1, NH == 1 && !HALVES>(p, [&](const Work& w, int j0, int step, int nkv, int wave, int lane) {
        if constexpr (NH == 2) {
            const NarrowMap<D> lm(wave, lane);
            process_q_tile_narrow<D, BF16, CAUSAL, false, 4>(p, lm, w.head, w.tile, j0, step, nkv, wave, lane, (LDS_PTR(char))smem);
        } else {
            const LaneMap<D> lm(wave, lane);
            process_q_tile<D, BF16, CAUSAL, HALVES, SPLIT>(p, lm, w.head, w.tile, j0, step, nkv, wave, lane, (LDS_PTR(char))smem);
        }
    });
}

// 128-row tiles where workgroups share the compute units (see default_shared_kernel, default_phase_priority).
template <int D, bool BF16, bool CAUSAL, bool PHASES>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_fwd_shared_kernel(Params p) {
    extern __shared__ __align__(16) char smem[];
    for_each_q_tile<CAUSAL, true, true>(p, [&](const Work& w, int j0, int step, int nkv, int wave, int lane) {
        const NarrowMap<D> lm(wave, lane);
        process_q_tile_narrow<D, BF16, CAUSAL, PHASES>(p, lm, w.head, w.tile, j0, step, nkv, wave, lane, (LDS_PTR(char))smem);
    });
}


// ------------------------------------------------------------------------------------------- host

thread_local char g_err[256] = "";

int fail(int code, const char* msg) {
    std::snprintf(g_err, sizeof g_err, "%s", msg);
    return code;
}

int check_shape(int B, int H, int N, int d) {
    if (B <= 0 || H <= 0 || N <= 0 || d <= 0) return fail(SAWATTN_ERR_INVALID_ARG, "B, H, N and d must be positive");
    if (d != 64 && d != 128) return fail(SAWATTN_ERR_UNSUPPORTED, "head dimension must be 64 or 128");
    const long long heads = (long long)B * H;
    if (heads >= (1LL << 31) / kDomains) return fail(SAWATTN_ERR_INVALID_ARG, "B*H too large");
    const long long q_tiles = (N + (long long)kTileQ - 1) / kTileQ;
    if (heads * q_tiles >= (1LL << 31)) return fail(SAWATTN_ERR_INVALID_ARG, "B*H*ceil(N/128) must be below 2^31");
    if ((double)heads * (double)N * (double)d >= 1099511627776.0) return fail(SAWATTN_ERR_INVALID_ARG, "B*H*N*d must be below 2^40");
    return SAWATTN_OK;
}

void fill_info(const Schedule& s, int d, sawattn_launch_info* out) {
    out->tile_q = s.tile_q;
    out->tile_kv = kTileKV;
    out->block_threads = kThreads;
    out->grid = s.grid;
    out->lds_bytes = s.tile_q > kTileQ ? kWideLdsBytes
                                       : (s.tile_q < kTileQ ? 2 : 1) * (d == 128 ? Geo<128>::kLdsBytes : Geo<64>::kLdsBytes);
    out->domains = kDomains;
    out->slots = s.slots;
    out->parts_per_head = s.parts;
    out->q_tiles_per_head = s.q_tiles;
    out->max_local_tiles = s.local_iters;
    out->launch = s.launch == kLaunchGrid ? SAWATTN_LAUNCH_GRID : SAWATTN_LAUNCH_PERSISTENT;
    out->tiles_per_workgroup = s.tiles_per_wg;
    out->qo_streaming = s.qo_streaming;
}

std::atomic<unsigned> g_ticket_turn{0};

// (KERNEL a template argument: the state below is kept per kernel)
template <void (*KERNEL)(Params)>
int launch_kernel(Params& p, int grid, int lds_bytes, hipStream_t stream) {
    auto kern = KERNEL;
    // The LDS size a kernel may ask for is a per-device attribute of the function: set once per device (bit = device).
    static std::atomic<unsigned long long> configured{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return fail(SAWATTN_ERR_RUNTIME, "hipGetDevice failed (or more than 64 devices)");
    }
    if (!(configured.load(std::memory_order_acquire) >> dev & 1ull)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                lds_bytes) != hipSuccess) {
            (void)hipGetLastError();
            return fail(SAWATTN_ERR_RUNTIME, "hipFuncSetAttribute(MaxDynamicSharedMemorySize) failed");
        }
        configured.fetch_or(1ull << dev, std::memory_order_release);
    }
    p.ticket_set = 0;
    if (p.sched.sync_heads || p.sched.sync_rounds) {
        p.ticket_set = (int)(g_ticket_turn.fetch_add(1u, std::memory_order_relaxed) % (unsigned)kTicketSets);
        hipLaunchKernelGGL(clear_tickets_kernel, dim3(1), dim3(64), 0, stream, p.ticket_set);
    }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds_bytes, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        char msg[200];
        std::snprintf(msg, sizeof msg, "kernel launch failed: %s", hipGetErrorString(e));
        return fail(SAWATTN_ERR_RUNTIME, msg);
    }
    return SAWATTN_OK;
}

template <int D, bool BF16, bool CAUSAL, int NH, bool HALVES = false, int SPLIT = kSplitLong>
int launch(Params& p, int grid, hipStream_t stream) {
    return launch_kernel<attn_fwd_kernel<D, BF16, CAUSAL, NH, HALVES, SPLIT>>(
        p, grid, NH == 2 ? kWideLdsBytes : (HALVES ? 2 : 1) * Geo<D>::kLdsBytes, stream);
}

// 128-row tiles: the kernel for shared compute units or the one for workgroups that have theirs to themselves.
template <int D, bool BF16, bool CAUSAL>
int launch_128(Params& p, int grid, hipStream_t stream) {
    if (!default_shared_kernel(p.sched, D, CAUSAL, BF16)) return launch<D, BF16, CAUSAL, 1>(p, grid, stream);
    if constexpr (CAUSAL) {      // (without a mask always with precedence: the other kernel is not built)
        if (!default_phase_priority(p.sched, D, CAUSAL))
            return launch_kernel<attn_fwd_shared_kernel<D, BF16, CAUSAL, false>>(p, grid, Geo<D>::kLdsBytes, stream);
    }
    return launch_kernel<attn_fwd_shared_kernel<D, BF16, CAUSAL, true>>(p, grid, Geo<D>::kLdsBytes, stream);
}

// 64-row tiles: which of the kernels.  Without a mask a sequence of an even number of full tiles needs nothing but the pipeline (see
// SplitKind).  Otherwise short scans go through scan_halves and long ones, where the pipeline's cheaper tiles outweigh the odd and masked ones
// taken singly, stay with it.  Measured, pipeline -> scan_halves: 16 x 1000, d = 64: 12.1 -> 10.5 us; 8 x 2048 causal, bf16: 19.1 -> 17.2;
// 24 x 2600 causal: 35.5 -> 34.3; 2 x 100, d = 128, causal: 9.4 -> 8.1; 5 x 1000, d = 128: 20.0 -> 18.3; 3000 causal, d = 128: 30.8 -> 28.6;
// but 3 x 5000, d = 128, causal: 47.9 -> 49.6, 3 x 10000: 113.7 -> 115.0, 30000: 289.7 -> 297.1, and between 4096 and 16384 keys it goes either way
// (2 x 8000, d = 128, causal: 68.9 -> 65.8).  One tile is all masked code, in the kernel that starts sooner, long / short: 8 x 64, d
// = 64 5.6, 5.3 us, bfloat16, causal 5.4, 5.3; d = 128 8.1, 7.7 and 7.9, 7.5.
template <int D, bool BF16>
int launch_halves(Params& p, bool causal, int grid, hipStream_t stream) {
    const bool brief = p.N <= 64 * kTileKV;
    if (causal) {
        if (brief) return launch<D, BF16, true, 1, true, kSplitShort>(p, grid, stream);
        return launch<D, BF16, true, 1, true, kSplitLong>(p, grid, stream);
    }
    if (p.N % (2 * kTileKV) == 0) return launch<D, BF16, false, 1, true, kSplitEven>(p, grid, stream);
    if (brief) return launch<D, BF16, false, 1, true, kSplitShort>(p, grid, stream);
    return launch<D, BF16, false, 1, true, kSplitLong>(p, grid, stream);
}

// Validates a variant description (NULL = the default schedule) and builds its schedule.
int schedule_for(int B, int H, int N, int d, bool causal, bool bf16, const sawattn_variant* v, Schedule* out) {
    int launch = -1 /* open */, decode = kDecodeDomain, max_slots = 0, tiles_per_wg = 0, rows = 0, halves = 0;
    bool align_rounds = false;
    if (v) {
        if (v->kv_halves < 0 || v->kv_halves > 2)
            return fail(SAWATTN_ERR_INVALID_ARG, "variant.kv_halves must be 0 (default), 1 or 2");
        halves = v->kv_halves;
        if (halves == 2) {
            if (v->rows_per_wavefront == 64)
                return fail(SAWATTN_ERR_UNSUPPORTED, "variant.kv_halves = 2 goes with 32 rows per wavefront");
        }
        if (v->launch != SAWATTN_LAUNCH_PERSISTENT && v->launch != SAWATTN_LAUNCH_GRID && v->launch != SAWATTN_LAUNCH_AUTO)
            return fail(SAWATTN_ERR_INVALID_ARG,
                        "variant.launch must be SAWATTN_LAUNCH_PERSISTENT, SAWATTN_LAUNCH_GRID or SAWATTN_LAUNCH_AUTO");
        if (v->decode != SAWATTN_DECODE_DOMAIN && v->decode != SAWATTN_DECODE_LINEAR)
            return fail(SAWATTN_ERR_INVALID_ARG, "variant.decode must be SAWATTN_DECODE_DOMAIN or SAWATTN_DECODE_LINEAR");
        if (v->rows_per_wavefront != 0 && v->rows_per_wavefront != 32 && v->rows_per_wavefront != 64)
            return fail(SAWATTN_ERR_INVALID_ARG, "variant.rows_per_wavefront must be 0 (default), 32 or 64");
        if (v->rows_per_wavefront == 64 && d != 128)
            return fail(SAWATTN_ERR_UNSUPPORTED, "variant.rows_per_wavefront = 64 needs head dimension 128");
        rows = v->rows_per_wavefront;
        if (halves == 0) halves = rows == 64 ? 1 : default_kv_halves(B * H, N, d, causal, bf16);
        if (halves == 2) rows = 32;
        if (rows == 0) rows = v->slots_per_domain > resident_slots(d, 2 * kTileQ) ? 32 : default_rows_per_wavefront(B * H, N, d, causal, bf16);
        if (v->slots_per_domain < 0 ||
            v->slots_per_domain > resident_slots(d, rows == 64 ? 2 * kTileQ : (halves == 2 ? kTileQ / 2 : kTileQ)))
            return fail(SAWATTN_ERR_INVALID_ARG,
                        "variant.slots_per_domain must be 0 (default) or 1..64 (1..96 for d = 64, 1..32 with 64 rows per "
                        "wavefront; with kv_halves = 2: 1..64 for d = 64, 1..32 for d = 128)");
        if (v->tiles_per_workgroup < 0 || v->tiles_per_workgroup > 2)
            return fail(SAWATTN_ERR_INVALID_ARG, "variant.tiles_per_workgroup must be 0 (default), 1 or 2");
        if (v->launch != SAWATTN_LAUNCH_AUTO) launch = v->launch == SAWATTN_LAUNCH_GRID ? kLaunchGrid : kLaunchPersistent;
        decode = v->decode == SAWATTN_DECODE_LINEAR ? kDecodeLinear : kDecodeDomain;
        max_slots = v->slots_per_domain;
        if (v->tiles_per_workgroup) tiles_per_wg = v->tiles_per_workgroup;
        if (v->qo_streaming < 0 || v->qo_streaming > 4)
            return fail(SAWATTN_ERR_INVALID_ARG, "variant.qo_streaming must be 0 (default), 1 (O), 2 (Q), 3 (both) or 4 (neither)");
        if (v->align_rounds != 0 && v->align_rounds != 1)
            return fail(SAWATTN_ERR_INVALID_ARG, "variant.align_rounds must be 0 or 1");
        align_rounds = v->align_rounds == 1;
    }
    if (halves == 0) halves = default_kv_halves(B * H, N, d, causal, bf16);
    if (halves == 2) rows = 32;
    if (rows == 0) rows = default_rows_per_wavefront(B * H, N, d, causal, bf16);
    const int tile_q = rows == 64 ? 2 * kTileQ : (halves == 2 ? kTileQ / 2 : kTileQ);
    *out = launch_schedule(B * H, N, d, causal, tile_q, launch, decode, max_slots, tiles_per_wg, align_rounds);
    out->qo_streaming = v && v->qo_streaming ? v->qo_streaming : default_qo_streaming(N, d);
    return SAWATTN_OK;
}

// Whether bfloat16 inputs, converted to binary16, would run the wide variant: then a workspace pays.
int workspace_schedule(int B, int H, int N, int d, bool causal, bool bf16, const sawattn_variant* v, Schedule* out,
                       bool* use) {
    *use = false;
    if (!bf16 || d != 128) return SAWATTN_OK;
    Schedule s;
    const int rc = schedule_for(B, H, N, d, causal, false, v, &s);
    if (rc != SAWATTN_OK) return rc;
    if (s.tile_q > kTileQ) { *use = true; *out = s; }
    return SAWATTN_OK;
}

int run(const void* Q, const void* K, const void* V, void* O, int B, int H, int N, int d, float scale, int causal,
        int scan_order, int in_dtype, int o_dtype, void* hip_stream, const sawattn_variant* variant, int32_t* trace,
        int32_t* trace_count, void* workspace = nullptr, size_t workspace_bytes = 0) {
    int rc = check_shape(B, H, N, d);
    if (rc != SAWATTN_OK) return rc;
    if (!Q || !K || !V || !O) return fail(SAWATTN_ERR_INVALID_ARG, "Q, K, V and O must be non-null");
    if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)O) & 15u)
        return fail(SAWATTN_ERR_INVALID_ARG, "Q, K, V and O must be 16-byte aligned");
    if (!std::isfinite(scale)) return fail(SAWATTN_ERR_INVALID_ARG, "scale must be finite");
    if (scan_order != SAWATTN_SCAN_CYCLIC && scan_order != SAWATTN_SCAN_SAWTOOTH)
        return fail(SAWATTN_ERR_INVALID_ARG, "scan_order must be SAWATTN_SCAN_CYCLIC or SAWATTN_SCAN_SAWTOOTH");
    if (in_dtype != SAWATTN_F16 && in_dtype != SAWATTN_BF16)
        return fail(SAWATTN_ERR_INVALID_ARG, "in_dtype must be SAWATTN_F16 or SAWATTN_BF16");
    if (o_dtype != SAWATTN_F16 && o_dtype != SAWATTN_BF16 && o_dtype != SAWATTN_F32)
        return fail(SAWATTN_ERR_INVALID_ARG, "o_dtype must be SAWATTN_F16, SAWATTN_BF16 or SAWATTN_F32");
    if ((trace == nullptr) != (trace_count == nullptr))
        return fail(SAWATTN_ERR_INVALID_ARG, "trace and trace_count must be given together");
    Schedule sched;
    bool converted = false;   // bfloat16 inputs through binary16 copies of K and V in the caller's workspace
    if (workspace) {
        rc = workspace_schedule(B, H, N, d, causal != 0, in_dtype == SAWATTN_BF16, variant, &sched, &converted);
        if (rc != SAWATTN_OK) return rc;
    }
    if (!converted) {
        rc = schedule_for(B, H, N, d, causal != 0, in_dtype == SAWATTN_BF16, variant, &sched);
        if (rc != SAWATTN_OK) return rc;
    }
    {   // A workgroup writes its O rows while others still read Q, K, V: O may not share memory with them.
        const unsigned long long elems = (unsigned long long)B * H * N * d;
        const unsigned long long in_bytes = elems * 2u, out_bytes = elems * (o_dtype == SAWATTN_F32 ? 4u : 2u);
        const uintptr_t o0 = (uintptr_t)O, o1 = o0 + out_bytes;
        for (const void* in : {Q, K, V}) {
            const uintptr_t i0 = (uintptr_t)in, i1 = i0 + in_bytes;
            if (o0 < i1 && i0 < o1) return fail(SAWATTN_ERR_INVALID_ARG, "O must not overlap Q, K or V");
        }
        if (converted) {
            if ((uintptr_t)workspace & 15u) return fail(SAWATTN_ERR_INVALID_ARG, "workspace must be 16-byte aligned");
            if (workspace_bytes < 2 * in_bytes)
                return fail(SAWATTN_ERR_INVALID_ARG, "workspace is smaller than attn_fwd_workspace_bytes reports");
            const uintptr_t w0 = (uintptr_t)workspace, w1 = w0 + 2 * in_bytes;
            for (const void* in : {Q, K, V}) {
                const uintptr_t i0 = (uintptr_t)in, i1 = i0 + in_bytes;
                if (w0 < i1 && i0 < w1) return fail(SAWATTN_ERR_INVALID_ARG, "workspace must not overlap Q, K, V or O");
            }
            if (w0 < o1 && o0 < w1) return fail(SAWATTN_ERR_INVALID_ARG, "workspace must not overlap Q, K, V or O");
        }
    }

    Params p;
    p.Q = Q; p.K = K; p.V = V; p.O = O;
    p.trace = trace; p.trace_count = trace_count;
    p.N = N;
    p.o_dtype = o_dtype;
    p.sawtooth = scan_order == SAWATTN_SCAN_SAWTOOTH;
    p.negate_q = scale < 0.f;
    p.q_bf16 = converted;
    {
        p.stream_o = sched.qo_streaming == 1 || sched.qo_streaming == 3;
        p.stream_q = sched.qo_streaming == 2 || sched.qo_streaming == 3;
    }
    // Never zero: the kernels mask a key by giving it the score -inf and rely on -inf * c = -inf.  At this floor
    // every finite score times c is below 2^-60 in magnitude, so scale = 0 still gives exp2(0) = 1 for every visible key.
    p.c = std::fmax((float)(std::fabs((double)scale) * 1.4426950408889634074), 1e-30f);
    p.sched = sched;
    p.max_local = sched.local_iters;
    const int grid = sched.grid;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const bool bf = in_dtype == SAWATTN_BF16, ca = causal != 0;
    if (converted) {
        const size_t chunks = (size_t)B * H * N * d / 8;
        u4* K16 = static_cast<u4*>(workspace);
        u4* V16 = K16 + chunks;
        const unsigned blocks = (unsigned)std::min<size_t>((chunks + 255) / 256, 256 * 16);
        hipLaunchKernelGGL(bf16_to_f16_kernel, dim3(blocks), dim3(256), 0, stream, static_cast<const u4*>(K),
                           static_cast<const u4*>(V), K16, V16, chunks);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(SAWATTN_ERR_RUNTIME, "conversion kernel launch failed");
        p.K = K16;
        p.V = V16;
    }
    if (sched.tile_q > kTileQ) {
        if (bf && !converted) return ca ? launch<128, true, true, 2>(p, grid, stream) : launch<128, true, false, 2>(p, grid, stream);
        return ca ? launch<128, false, true, 2>(p, grid, stream) : launch<128, false, false, 2>(p, grid, stream);
    }
    if (sched.tile_q < kTileQ) {   // 64-row tiles: the two halves of the K/V scan at once
        if (d == 128) return bf ? launch_halves<128, true>(p, ca, grid, stream) : launch_halves<128, false>(p, ca, grid, stream);
        return bf ? launch_halves<64, true>(p, ca, grid, stream) : launch_halves<64, false>(p, ca, grid, stream);
    }
    if (d == 128) {
        if (bf) return ca ? launch_128<128, true, true>(p, grid, stream) : launch_128<128, true, false>(p, grid, stream);
        return ca ? launch_128<128, false, true>(p, grid, stream) : launch_128<128, false, false>(p, grid, stream);
    }
    if (bf) return ca ? launch_128<64, true, true>(p, grid, stream) : launch_128<64, true, false>(p, grid, stream);
    return ca ? launch_128<64, false, true>(p, grid, stream) : launch_128<64, false, false>(p, grid, stream);
}

// ---- scratch memory of attn_fwd_static: a fixed array in device memory instead of a caller's workspace.
// Every GPU the library runs on holds its own copy at its own address; host code never uses the array's name as
// an address, only what hipGetSymbolAddress returned for the device that was current.
constexpr size_t kStaticScratchBytes = (size_t)SAWATTN_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Address of `scratch` on the current device (looked up once per device).
int static_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return fail(SAWATTN_ERR_RUNTIME, "cannot query the current device (or its index is 64 or more)");
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            char msg[200];
            std::snprintf(msg, sizeof msg, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
            return fail(SAWATTN_ERR_RUNTIME, msg);
        }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return SAWATTN_OK;
}

// Argument checks shared by the queries that launch nothing.
int check_query(int B, int H, int N, int d, int in_dtype) {
    if (in_dtype != SAWATTN_F16 && in_dtype != SAWATTN_BF16)
        return fail(SAWATTN_ERR_INVALID_ARG, "in_dtype must be SAWATTN_F16 or SAWATTN_BF16");
    return check_shape(B, H, N, d);
}

}  // namespace sawattn

extern "C" {

int attn_fwd(const void* Q, const void* K, const void* V, void* O, int B, int H, int N, int d, float scale, int causal,
             int scan_order, int in_dtype, int o_dtype, void* hip_stream) {
    return sawattn::run(Q, K, V, O, B, H, N, d, scale, causal, scan_order, in_dtype, o_dtype, hip_stream, nullptr, nullptr,
                        nullptr);
}

int attn_fwd_variant(const void* Q, const void* K, const void* V, void* O, int B, int H, int N, int d, float scale,
                     int causal, int scan_order, int in_dtype, int o_dtype, void* hip_stream,
                     const sawattn_variant* variant, int32_t* trace, int32_t* trace_count) {
    return sawattn::run(Q, K, V, O, B, H, N, d, scale, causal, scan_order, in_dtype, o_dtype, hip_stream, variant, trace,
                        trace_count);
}

int attn_fwd_workspace(const void* Q, const void* K, const void* V, void* O, int B, int H, int N, int d, float scale,
                       int causal, int scan_order, int in_dtype, int o_dtype, void* hip_stream,
                       const sawattn_variant* variant, int32_t* trace, int32_t* trace_count, void* workspace,
                       size_t workspace_bytes) {
    return sawattn::run(Q, K, V, O, B, H, N, d, scale, causal, scan_order, in_dtype, o_dtype, hip_stream, variant, trace,
                        trace_count, workspace, workspace_bytes);
}

int attn_fwd_workspace_bytes(int B, int H, int N, int d, int causal, int in_dtype, const sawattn_variant* variant,
                             size_t* bytes, sawattn_launch_info* info) {
    using namespace sawattn;
    if (!bytes) return fail(SAWATTN_ERR_INVALID_ARG, "bytes must be non-null");
    int rc = check_query(B, H, N, d, in_dtype);
    if (rc != SAWATTN_OK) return rc;
    Schedule s;
    bool use = false;
    rc = workspace_schedule(B, H, N, d, causal != 0, in_dtype == SAWATTN_BF16, variant, &s, &use);
    if (rc != SAWATTN_OK) return rc;
    if (!use) {
        rc = schedule_for(B, H, N, d, causal != 0, in_dtype == SAWATTN_BF16, variant, &s);
        if (rc != SAWATTN_OK) return rc;
    }
    *bytes = use ? (size_t)B * H * N * d * 4 : 0;
    if (info) fill_info(s, d, info);
    return SAWATTN_OK;
}

int attn_fwd_static(const void* Q, const void* K, const void* V, void* O, int B, int H, int N, int d, float scale,
                    int causal, int scan_order, int in_dtype, int o_dtype, void* hip_stream) {
    using namespace sawattn;
    size_t need = 0;
    int rc = attn_fwd_workspace_bytes(B, H, N, d, causal, in_dtype, nullptr, &need, nullptr);
    if (rc != SAWATTN_OK) return rc;
    if (need > kStaticScratchBytes) {
        char msg[200];
        std::snprintf(msg, sizeof msg, "attn_fwd_static: this problem needs %zu bytes of scratch, the fixed array holds %zu "
                      "(4*B*H*N*d must not exceed it)", need, kStaticScratchBytes);
        return fail(SAWATTN_ERR_UNSUPPORTED, msg);
    }
    void* ws = nullptr;
    if (need) {
        rc = static_scratch(&ws);
        if (rc != SAWATTN_OK) return rc;
    }
    return run(Q, K, V, O, B, H, N, d, scale, causal, scan_order, in_dtype, o_dtype, hip_stream, nullptr, nullptr, nullptr,
               ws, need);
}

int attn_fwd_variant_launch_info(int B, int H, int N, int d, int causal, int in_dtype, const sawattn_variant* variant,
                                 sawattn_launch_info* out) {
    using namespace sawattn;
    if (!out) return fail(SAWATTN_ERR_INVALID_ARG, "out must be non-null");
    int rc = check_query(B, H, N, d, in_dtype);
    if (rc != SAWATTN_OK) return rc;
    Schedule s;
    rc = schedule_for(B, H, N, d, causal != 0, in_dtype == SAWATTN_BF16, variant, &s);
    if (rc != SAWATTN_OK) return rc;
    fill_info(s, d, out);
    return SAWATTN_OK;
}

int attn_fwd_launch_info(int B, int H, int N, int d, int causal, int scan_order, int in_dtype, sawattn_launch_info* out) {
    if (scan_order != SAWATTN_SCAN_CYCLIC && scan_order != SAWATTN_SCAN_SAWTOOTH)
        return sawattn::fail(SAWATTN_ERR_INVALID_ARG, "scan_order must be SAWATTN_SCAN_CYCLIC or SAWATTN_SCAN_SAWTOOTH");
    return attn_fwd_variant_launch_info(B, H, N, d, causal, in_dtype, nullptr, out);
}

int attn_fwd_plan(int B, int H, int N, int d, int causal, int scan_order, int in_dtype, const sawattn_variant* variant,
                  int32_t* trace, int32_t* trace_count) {
    using namespace sawattn;
    if (!trace || !trace_count) return fail(SAWATTN_ERR_INVALID_ARG, "trace and trace_count must be non-null");
    if (scan_order != SAWATTN_SCAN_CYCLIC && scan_order != SAWATTN_SCAN_SAWTOOTH)
        return fail(SAWATTN_ERR_INVALID_ARG, "scan_order must be SAWATTN_SCAN_CYCLIC or SAWATTN_SCAN_SAWTOOTH");
    int rc = check_query(B, H, N, d, in_dtype);
    if (rc != SAWATTN_OK) return rc;
    Schedule s;
    rc = schedule_for(B, H, N, d, causal != 0, in_dtype == SAWATTN_BF16, variant, &s);
    if (rc != SAWATTN_OK) return rc;
    // the kernel's outer loop, one workgroup at a time
    for (int wg = 0; wg < s.grid; ++wg) {
        int local = 0;
        for (int it = 0; it < s.local_iters; ++it) {
            const Work w = decode_work(s, wg, it, causal != 0, scan_order == SAWATTN_SCAN_SAWTOOTH);
            if (w.tile < 0) continue;
            const int nkv = visible_kv_tiles(s, w.tile, N, causal != 0);
            int32_t* rec = trace + ((size_t)wg * s.local_iters + local) * 4;
            rec[0] = w.head; rec[1] = w.tile; rec[2] = w.backward ? nkv - 1 : 0; rec[3] = w.backward ? 0 : nkv - 1;
            ++local;
        }
        trace_count[wg] = local;
    }
    return SAWATTN_OK;
}

const char* attn_last_error(void) { return sawattn::g_err; }
int attn_version(void) { return 212; }
const char* sawattn_last_error(void) { return attn_last_error(); }
int sawattn_version(void) { return attn_version(); }

}  // extern "C"
