// Split-K decode attention over resident KV (Sec. II-A: the query's similarity with the keys weights
// the values):  out[b,hq,:] = softmax_j(q[b,hq,:].K[b,h,j,:] / sqrt(D)) V[b,h,j,:],  h = hq / G.
//
// Partial kernel: one workgroup of 8 wavefronts (6 when D = 256) per (sequence, query-head group, token split).  Splits are cut for about one
// workgroup per compute unit; where that would leave them uneven for one to four of each (uniform batches), or for three (ragged ones);
// a batch with more pairs of sequence and KV head than that has a workgroup for each pair at least (attn_splits.hpp).  A step is a
// tile of 16 tokens (two tiles when D = 64); the steps of a split are handed out to the wavefronts on demand through a counter in LDS, so a wavefront whose loads come back
// late takes fewer steps and all of them reach the merge together (with a fixed round-robin the slowest
// wavefront, and the second workgroup of a compute unit, finished 2-4 us after the median).
//  * q K^T on the matrix cores: v_mfma_f32_16x16x32 with K as the 16 x 32 A operand (a lane holds 16 contiguous bytes of a
//    row) and the query heads of the group as the columns of B.  A 16-byte global load is exactly one operand register set, so K
//    never passes through LDS.
//    A load of K takes whole 128-byte lines, of 8 rows: two neighbouring rows of the operand hold the two halves of a line of one
//    token, and the columns of a head the two halves of its query in turn (beyond 8 heads: a product for each half), so a score is two
//    elements of the result.  With a row of the operand for each token a load took 64 bytes of 16 rows, and the other half of each line was a request of
//    its own to L2: reading alone 6.12 against 6.53 TB/s at head_dim 64 and 6.47 / 6.57 at 128, with two workgroups per compute unit 6.16 / 6.40
//    (200 MB per launch).  us per layer from a graph, 16 rows / 8 rows: 16 KV heads x 4 x 64, 7 sequences of 9000 49.6 / 45.2, paged of
//    6283-11718 57.6 / 52.6; 8 x 4 x 128, 8 of 1K-8K paged 31.5 / 30.0, 32K fp16 26.4 / 26.0, bf16 25.0 / 25.3 (the turn below takes 0.3 of both), 16K 16.8 / 16.0, 32 x 1, batch 32 of 528 46.4 / 45.0; 8 x 16 x 128, 12 of 2000
//    26.2 / 24.2; 5 x 5 x 256, 43 of 2354 97.4 / 87.9, 16 x 4, 4 of 8192 86.9 / 86.5 (paged fp16 85.7 / 86.6); shorter single sequences the same (32 layers of 4K 259.6 / 261.6, with
//    the 32-bit offsets below 260.5).
//  * The result leaves lane (column n, row group tg) with the scores of four tokens (tg, 4 + tg, 8 + tg, 12 + tg) for the column's query
//    head, which is the layout of the B operand of V^T P: probabilities never leave their lane.
//  * V^T P on the matrix cores as well: the 16 lanes of a row group load the V rows of their own 4 tokens, 16 bytes
//    per lane; byte permutes gather the 4 tokens of each of the lane's 8 columns, and that is the A operand.
//    A probability enters in parts, one product each: three bf16 terms, whose sum is the 32-bit value exactly, or two fp16
//    terms, which drop up to 2^-24 of it and whatever lies below 2^-36 of the reference.  The error against float64 is
//    that of the whole 32-bit factor or less (fp16, 1.5K tokens of N(0,1), relative to a head's 2-norm: at most 4.3e-7, with the whole
//    factor 4.6e-7; scores four times as steep 1.9e-6 both).
//    On the vector ALU this product cost 32 fused multiply-adds per query head and tile, so a workgroup took at most
//    4 heads, and only 1 or 2 of a group that 4 does not divide: 7 heads per KV head read K and V seven times
//    (8 KV heads x 32K tokens x 128, bf16, vector ALU / matrix cores: 7 heads 224 / 25.5 us, 3 heads 102 / 25.4, 16 heads 61 / 26.6; 4 heads are level).
//    A single head stays on the vector ALU (see the kernel).
//  * K and V are read once and never again: the loads are nontemporal.
// The wavefronts' softmax states of a head are merged through LDS and one fp32 partial per (b, hq, split) is
// written; the combine kernel merges the splits.  When every sequence is a single split the partial kernel writes the
// results itself (batch 32 x 32 heads of 512-544 tokens: 3.1 of 50.4 us).
// HBM-bound (G flop per byte).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "attn_splits.hpp"
#include "launch.hpp"
#include "plan.hpp"

namespace {

using namespace kvb;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Wavefronts of a workgroup.  A step is 8 KiB of K and V, at head_dim 256 16 KiB: eight wavefronts then have more loads in
// flight than HBM likes (8 KV heads x 4 x 8K tokens x 256, one query head each: 46.0 us with eight, 45.2 with six; at
// head_dim 128 eight and six are equal on long sequences and eight better on many short ones, 47.3 against 54.2 us).
constexpr int waves(int D) { return D >= 256 ? 6 : 8; }
constexpr float kEmptyMax = -1.0e30f; // running maximum of a row group that has seen no token
// How K and V are addressed: a strided view; a block pool whose blocks hold whole tiles (split starts are multiples of
// the tile); any other block pool; a strided view whose token rows lie kFarRows 16-byte vectors (256 MiB) or more apart, so that the offsets within a tile
// (15 rows and a row's own bytes) do not fit 32 bits.  An instance of its own: both kinds of
// address in one loop cost near rows 2 %, and the second pass, which has 64-bit addresses anyway, is 2 to 9 times slower.  us per layer, 129 rows 256 MiB apart,
// second pass / this: 1 KV head x 4 x 64 11.5 / 3.5, 4 x 128 12.3 / 3.8, 16 x 128 43.6 / 5.0, 4 x 256 14.5 / 5.9.
constexpr int kStrided = 0, kPagedTiles = 1, kPagedRows = 2, kStridedFar = 3;
constexpr unsigned long long kFarRows = 1ull << 24;
struct AttnParams {
    const int *seq_lens;   // device [B]
    float *part_acc;       // [B, Hq, n_splits, D]
    float *part_ml;        // [B, Hq, n_splits, 2]
    const long long *seq_off;  // strided layout, optional: element offset of each sequence (replaces b*sb)
    int n_pool;            // paged layout
    int direct_mode;       // >= 0: every sequence has one split, results go to `out` in this mode (store_out); -1: partials
    float scale_log2e;     // log2(e) / sqrt(D)
    void *out;             // [B, Hq, D]
    int n_splits;
    int max_len;           // host-checked bound on every sequence length
};

// Three strides below 2^40 vectors (16 TiB) in four words: 32 bits of each, and a word with 8 further bits of each.
struct Strides {
    unsigned long long ss, sh, sb;
};
struct PackedStrides {
    unsigned long long ss_sh;
    int sb, high;
};
// A further bit of `high`: sequences start at seq_off.
constexpr int kSeqOff = 1 << 24;
constexpr PackedStrides pack_strides(Strides s)
{
    return {(s.ss & 0xffffffffull) | s.sh << 32, (int)(unsigned)s.sb,
            (int)((unsigned)(s.ss >> 32 & 0xff) | (unsigned)(s.sh >> 32 & 0xff) << 8 | (unsigned)(s.sb >> 32 & 0xff) << 16)};
}
constexpr Strides unpack_strides(PackedStrides p)
{
    return {(p.ss_sh & 0xffffffffull) | (unsigned long long)(p.high & 0xff) << 32, p.ss_sh >> 32 | (unsigned long long)(p.high >> 8 & 0xff) << 32,
            (unsigned)p.sb | (unsigned long long)(p.high >> 16 & 0xff) << 32};
}
constexpr bool strides_survive(Strides s)
{
    const Strides u = unpack_strides(pack_strides(s));
    return u.ss == s.ss && u.sh == s.sh && u.sb == s.sb;
}
static_assert(strides_survive({16, 0x80000000ull, 0xffffffffffull}) && strides_survive({0xffffffffffull, 0x80ffffffffull, 0}) &&
              strides_survive({0x100000000ull, 0, 0x8080000000ull}), "pack_strides");
// What the partial kernel's first K and V addresses depend on.  These are arguments of their own, 14 words in all, because the
// command processor can place that many in registers before a wavefront starts; a struct it cannot, and the wavefront then
// waits for two scalar loads in turn before its first vector load.  us per layer from a graph, struct / arguments: 8 KV heads x 4 x 128, 1K tokens
// 7.2 / 7.1, 2K 7.8 / 7.6, 4K 8.9 / 8.75; 8 x 8, 4 sequences of 1K-3K 11.6 / 11.3; paged, 2 x 7, 4K 8.2 / 8.0; batches that
// take 16 us and more are within 1 %.
struct AttnHead {
    const u32x4 *K, *V;    // attention-side buffers of the layer
    const u32x4 *q;        // [B, Hq, D]
    int len_uniform;       // >= 0: every sequence has this length (saves the first dependent load); -1: read seq_lens
    int split_tokens;
    Strides strides;       // strided layout, in 16-byte vectors
    const int *table;      // paged layout
    int max_blocks, bt;
    int H, Hq, G, B;
    int gt, subs;          // query heads per workgroup (at most kMaxHeads); workgroups that share a KV head
    bool heads_first;      // table: grid (head group, item), not (item, head group)
};
// Numbers of heads fit 16 bits.  The sequences of a table fit 8; what other grids need of B is their z dimension.
inline unsigned pack16(int lo, int hi) { return (unsigned)lo | (unsigned)hi << 16; }
static_assert(kMaxHeads < 128 && kMaxTableSeqs < 256, "gt has 7 bits, B 8");

// Ragged batch: the r-th sequence of the grid's order, seq[r], owns work items [first[r], first[r + 1]), each of tokens[r] token rows
// (the last one shorter).  Entries past the batch are INT_MAX.
struct ItemTable {
    int first[kMaxTableSeqs], tokens[kMaxTableSeqs];
    unsigned char seq[kMaxTableSeqs];
};
// How many splits of each sequence the combine kernel reads.
struct CountTable {
    unsigned short splits[kMaxTableSeqs];
};
static_assert(kMaxSplits <= 0xffff, "CountTable");
// Every other batch: the grid is (split, head group, sequence).  The length and the split length are then scalar arguments, a workgroup looks nothing up,
// and the launch copies 1.2 KiB less (0.1 us of host time).
struct NoTable {};

template <bool BF16>
__device__ __forceinline__ void unpack8(u32x4 v, float f[8])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned w = v[i];
        if (BF16) {
            f[2 * i] = __uint_as_float(w << 16);
            f[2 * i + 1] = __uint_as_float(w & 0xffff0000u);
        } else {
            const f16x2 h = __builtin_bit_cast(f16x2, w);
            f[2 * i] = (float)h[0];
            f[2 * i + 1] = (float)h[1];
        }
    }
}

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float rdlane(float x, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
// Wavefront-wide maximum / sum over all 64 lanes, result uniform: four DPP steps inside each row of 16 lanes
// (vector-ALU speed, no trip through the LDS crossbar), then the four row results through scalar registers.
__device__ __forceinline__ float wave_max(float x)
{
    x = fmaxf(x, dpp_mov<0xB1>(x));   // quad_perm [1,0,3,2]
    x = fmaxf(x, dpp_mov<0x4E>(x));   // quad_perm [2,3,0,1]
    x = fmaxf(x, dpp_mov<0x141>(x));  // row_half_mirror
    x = fmaxf(x, dpp_mov<0x140>(x));  // row_mirror
    return fmaxf(fmaxf(rdlane(x, 0), rdlane(x, 16)), fmaxf(rdlane(x, 32), rdlane(x, 48)));
}
__device__ __forceinline__ float wave_sum(float x)
{
    x += dpp_mov<0xB1>(x);
    x += dpp_mov<0x4E>(x);
    x += dpp_mov<0x141>(x);
    x += dpp_mov<0x140>(x);
    return (rdlane(x, 0) + rdlane(x, 16)) + (rdlane(x, 32) + rdlane(x, 48));
}

// The same over the lanes of each half row.
__device__ __forceinline__ float half_row_max(float x)
{
    x = fmaxf(x, dpp_mov<0xB1>(x));
    x = fmaxf(x, dpp_mov<0x4E>(x));
    return fmaxf(x, dpp_mov<0x141>(x));
}
__device__ __forceinline__ float half_row_sum(float x)
{
    x += dpp_mov<0xB1>(x);
    x += dpp_mov<0x4E>(x);
    return x + dpp_mov<0x141>(x);
}

template <bool BF16>
__device__ __forceinline__ f32x4 mfma_16x16x32(u32x4 a, u32x4 b, f32x4 c)
{
    if (BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ unsigned short f32_to_bf16_rne(float f)
{
    unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40);  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// mode: 0 fp32, 1 fp16, 2 bf16, both rounded to nearest even.
__device__ __forceinline__ void store_out(void *out, long long i, int mode, float r)
{
    if (mode == 0) ((float *)out)[i] = r;
    else if (mode == 1) ((_Float16 *)out)[i] = (_Float16)r;
    else ((unsigned short *)out)[i] = f32_to_bf16_rne(r);
}
// C in a row (i is a multiple of C); the buffer itself need only be aligned to its elements.
template <int C>
__device__ __forceinline__ void store_outs(void *out, long long i, int mode, const float r[C])
{
    typedef float fv __attribute__((ext_vector_type(C)));
    typedef unsigned short hv __attribute__((ext_vector_type(C)));
    if (mode == 0 && !((uintptr_t)out & (4 * C - 1))) {
        fv v;
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = r[k];
        *(fv *)((float *)out + i) = v;
    } else if (mode != 0 && !((uintptr_t)out & (2 * C - 1))) {
        hv v;
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = mode == 1 ? __builtin_bit_cast(unsigned short, (_Float16)r[k]) : f32_to_bf16_rne(r[k]);
        *(hv *)((unsigned short *)out + i) = v;
    } else {
#pragma unroll
        for (int k = 0; k < C; ++k) store_out(out, i + k, mode, r[k]);
    }
}

// C += A B with the four tokens of a row group in a tile as the lane's share of the contracted index.
template <bool BF16>
__device__ __forceinline__ f32x4 mfma_16x16x16(u32x2 a, u32x2 b, f32x4 c)
{
    if (BF16)
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, a), __builtin_bit_cast(f16x4, b), c, 0, 0, 0);
}

// Maximum / sum over the four row groups (lanes n, n + 16, n + 32, n + 48), in every one of them.
__device__ __forceinline__ float rows_max(float x)
{
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}
__device__ __forceinline__ float rows_sum(float x)
{
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

// Sum over the two halves of the wavefront, in both of them.
__device__ __forceinline__ float halves_sum(float x)
{
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

// A probability in fp32 is the exact sum of three bf16 numbers (the upper half of its bits, twice of what is left), or
// of two fp16 numbers up to 2^-24 of itself; P V is one product per term.
template <bool BF16> constexpr int kTerms = BF16 ? 3 : 2;

template <bool BF16>
__device__ __forceinline__ void split2(float x, float y, unsigned out[kTerms<BF16>])   // two tokens per register
{
    if constexpr (BF16) {
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const unsigned a = __float_as_uint(x), b = __float_as_uint(y);
            out[t] = __builtin_amdgcn_perm(b, a, 0x07060302u);
            x -= __uint_as_float(a & 0xffff0000u);
            y -= __uint_as_float(b & 0xffff0000u);
        }
    } else {
        const f16x2 h = __builtin_convertvector(f32x2{x, y}, f16x2);
        const f16x2 l = __builtin_convertvector(f32x2{x - (float)h[0], y - (float)h[1]}, f16x2);
        out[0] = __builtin_bit_cast(unsigned, h);
        out[1] = __builtin_bit_cast(unsigned, l);
    }
}

// Probabilities are exp2(score - reference): the reference follows the running maximum only when a score passes it by
// kRise, so most tiles neither reduce a maximum over the row groups nor rescale the accumulators.
constexpr float kRise = 4.f;
// The exponent of a probability is one fused multiply-add (score x scale - reference), which rounds once; the reference is itself
// a rounded product.  Up to this magnitude that rounding shifts every exponent by at most 1/32, which cancels in the
// normalisation; far above it the shift would leave the range of the probabilities, and the split is done again.  (Rounding
// the products in the loop where the reference is large costs 2-3 % at head_dim 64 and 2 % on many short sequences.)
constexpr float kFusedRef = 1048576.f;
// fp16 terms are taken of 2^11 times the probability (up to 2^15), which puts what they drop below 2^-36 of the largest.
template <bool BF16> constexpr float kLift = BF16 ? 1.f : 2048.f;

// One head (NH = 1, head_dim 128 and 256): V^T P on the vector ALU.  On the matrix cores 15 of 16 columns would repeat the head,
// and its sums would lie in 4 lanes of 64, from where they cost eight 16-byte LDS stores per wavefront where these take two: 512 against 290 cycles in front of the merge
// of a split of 128 tokens.  us per layer from a graph, one query head each, matrix cores -> vector ALU: 8 KV heads of 128, 1K tokens
// 7.9 -> 7.6, 4K 9.1 -> 8.8, 32K 26.1 -> 25.8, batch 32 of 520 15.0 -> 14.3; of 256, 4K 15.9 -> 15.4, 16K 31.5 -> 30.7.  Two heads
// gain nothing (4K 9.0 / 9.0, of 256 16.1 / 16.4), and head_dim 64 had no faster vector kernel (4K 7.5 against 19).
template <int D, int NH, bool BF16, int LAYOUT, typename TAB>
__global__ void __launch_bounds__(64 * waves(D), D <= 128 ? 4 : 2) 
kv_attn_partial_kernel(const u32x4 *K, const u32x4 *V, const u32x4 *q,
                       typename std::conditional<std::is_same<TAB, ItemTable>::value, const int *, unsigned long long>::type lens_arg,
                       unsigned heads, unsigned shares,
                       typename std::conditional<LAYOUT == kPagedTiles || LAYOUT == kPagedRows, const int *, unsigned long long>::type addr_arg, int addr2, int addr3,
                       AttnParams p, TAB tab)
{
    constexpr int kWaves = waves(D), kThreads = 64 * kWaves;
    constexpr int NJ = D / 32;               // MFMA slices along D of q K^T
    constexpr int DV = D / 8;                // 16-byte vectors per row
    constexpr int E = D >= 128 ? 8 : 4;      // V elements per lane and load: 16 lanes hold a row of 16 * E
    constexpr int NV = D / (16 * E);         // loads per V row (1, or 2 when D = 256)
    constexpr int TI = tiles_per_step(D);    // tiles of one step
    constexpr int kStepTok = kTile * TI;
    constexpr int NT = kTerms<BF16>;
    constexpr bool VALU = NH == 1;
    constexpr int RG = VALU ? 4 : 1;         // states of a wavefront that meet in LDS: one per row group, or one
    constexpr int kCopies = VALU ? 1 : 16 / NH;   // matrix columns that carry the same query head
    constexpr bool HALVES = NH <= 8;         // a column holds one half of every 128-byte line of its query head
    constexpr int NQ = HALVES ? NJ / 2 : NJ;
    constexpr bool PAGED = LAYOUT == kPagedTiles || LAYOUT == kPagedRows, TILE_ID = LAYOUT == kPagedTiles;
    typedef unsigned vload_t __attribute__((ext_vector_type(E / 2)));

    int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int H = heads & 0xffff, G = heads >> 16, Hq = H * G, gt = shares & 0x7f, subs = shares >> 16;
    int split = blockIdx.x, gy = blockIdx.y, b = blockIdx.z, split_tokens = 0, len = 0;
    if constexpr (std::is_same<TAB, ItemTable>::value) {
        // Ragged batch: the grid counts only splits that hold tokens, sequence after sequence, each sequence cut into its own
        // number of equal splits.  Lane = sequence: table and lengths come with one memory latency, two beyond 64 sequences (us, a search
        // of scalar loads, each waiting for the one before / this: 8 sequences of 1K-8K tokens, 16 layers 501 / 495; 60 of 100-600, a layer 23.3 / 22.8).
        static_assert(kMaxTableSeqs == 128, "two sequences per lane");
        const int B = shares >> 8 & 0xff;
        const bool heads_first = shares & 0x80;
        const int item = heads_first ? blockIdx.y : blockIdx.x;
        gy = heads_first ? blockIdx.x : blockIdx.y;
        int first = tab.first[lane], tokens = tab.tokens[lane], seq = tab.seq[lane], n_tok = lens_arg[min(lane, B - 1)];
        int rank = __builtin_popcountll(__ballot(first <= item)) - 1;   // the last sequence that starts at or before this item
        int n_tok2 = 0;
        if (B > 64) {
            n_tok2 = lens_arg[min(64 + lane, B - 1)];
            const int first2 = tab.first[64 + lane], in2 = __builtin_popcountll(__ballot(first2 <= item));
            if (in2) {
                rank = in2 - 1;
                first = first2;
                tokens = tab.tokens[64 + lane];
                seq = tab.seq[64 + lane];
            }
        }
        b = __builtin_amdgcn_readlane(seq, rank);
        split = item - __builtin_amdgcn_readlane(first, rank);
        split_tokens = __builtin_amdgcn_readlane(tokens, rank);
        len = min(__builtin_amdgcn_readlane(b < 64 ? n_tok : n_tok2, b & 63), p.max_len);
    } else {
        split_tokens = (int)lens_arg;
        len = (int)(lens_arg >> 32);
        if (len < 0) len = min(p.seq_lens[b], p.max_len);
    }
    const int h = __builtin_expect(subs == 1, 1) ? gy : gy / subs, g0 = (gy - h * subs) * gt;
    const int hq0 = h * G + g0;
    const int ng = min(gt, G - g0);   // query heads of this workgroup
    int n = lane & 15;          // MFMA column (query head n / kCopies; columns past the last head repeat it); also the pair of K rows this lane loads from
    int tg = lane >> 4;         // row group: owns tokens tg, 4 + tg, 8 + tg and 12 + tg of a tile; also the D sub-slice of the operands

    const int t_begin = min(len, split * split_tokens);
    const int t_end = min(len, t_begin + split_tokens);

    // B operand: column n carries query head n / kCopies; this lane holds elements 32j + 8tg .. +7 of it, or (HALVES) those of its half of line j.
    u32x4 qv[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j)
        qv[j] = q[((long long)b * Hq + hq0 + (VALU ? 0 : min(n / kCopies, ng - 1))) * DV + (HALVES ? 8 * j + 4 * (n & 1) : 4 * j) + tg];

    float m = kEmptyMax, l = 0.f;     // reference (the same in the four row groups) and this row group's sum
    f32x4 acc[NV][E];                 // element (w, e)[i]: column d = w * 16E + (4tg + i) * E + e of this lane's query head
    float vacc[NV][E];                // VALU: column d = (w * 16 + n) * E + e, this row group's share
#pragma unroll
    for (int w = 0; w < NV; ++w)
#pragma unroll
        for (int e = 0; e < E; ++e) {
            acc[w][e] = f32x4{0.f, 0.f, 0.f, 0.f};
            vacc[w][e] = 0.f;
        }

    unsigned long long ss = 0;
    long long head_off = 0;
    const int *tbl = nullptr;
    if constexpr (PAGED) {
        tbl = addr_arg + (long long)b * addr2;
    } else {
        const Strides st = unpack_strides({addr_arg, addr2, addr3});
        ss = st.ss;
        long long seq_start = (long long)(b * st.sb);
        if (__builtin_expect(addr3 & kSeqOff, 0)) {
            int here = 0;
            asm volatile("" : "+s"(here));   // or the pointer is loaded, and waited for, ahead of the first addresses of every launch (only where the load stands rests on it)
            seq_start = (&p.seq_off)[here][b] / 8;
        }
        head_off = seq_start + (long long)(h * st.sh);
    }
    const int bt = addr3, bt_shift = (bt & (bt - 1)) == 0 ? __builtin_ctz((unsigned)bt) : -1;   // paged
    auto block_of = [&](int row) -> int { return bt_shift >= 0 ? (row >> bt_shift) : (row / bt); };
    // vector index of the first element of token row `row` (paged: in pool block blk; a block id outside the pool
    // reads block 0 and is masked)
    auto row_base = [&](int row, int blk) -> long long {
        if (PAGED) {
            const int slot = row - block_of(row) * bt;
            if ((unsigned)blk >= (unsigned)p.n_pool) blk = 0;
            return (((long long)blk * H + h) * bt + slot) * DV;
        }
        return head_off + (long long)row * ss;
    };
    // Which of a tile's tokens are whose: row group tg has tokens tg, 4 + tg, 8 + tg and 12 + tg, so that a load of V takes four rows that lie side by side.
    // K registers j = 2c and 2c + 1 hold line c (128 bytes) of one of the first and of one of the last eight tokens, the even lane of a pair the
    // first half of it and the odd lane the second.
    auto k_row = [&](int j) -> int { return 8 * (j & 1) + 4 * ((n >> 1) & 1) + (n >> 2); };
    auto k_vec = [&](int j) -> int { return 8 * (j >> 1) + 4 * (n & 1) + tg; };
    // Paged layout: the block ids of one step's rows are fetched ahead, so that the table lookup is off the load chain.
    // When the block size is a multiple of the tile a tile lies inside one block (kPagedTiles): one lookup per tile, the
    // same for the whole wavefront and so a scalar load.  Otherwise a lane looks up its two K rows and the 4 tokens of
    // its row group.
    struct Ids { int k[TI][TILE_ID ? 1 : 2], t[TI][TILE_ID ? 1 : 4], slot0[TI]; };   // slot0: the first row's place in its block
    // kPagedRows: the rows of a tile that a lane loads, two of K and four of V, as places from the start of the block in which the tile's first row has place
    // slot0 (past the end: that row's own), and those cut into blocks on from there and a place in the block.  One division for the tile and not one for each
    // row: above 16 tokens a block a place is at most one block on, below it the quotient of a number up to 29 comes from a product.  The branch
    // is one for all six rows: as a choice for each row it took 1-14 % more.  us per layer from a graph, a division for each row with a row of K per lane / with whole
    // lines of K / this: 16 x 4 x 64, 7 of 6283-11718, blocks of 24 75.4 / 79.9 / 59.5, of 10 77.4 / 81.8 / 61.3, of 8 66.6 / 65.1 / 60.3; 2 x 2 x 64, 256 tokens in 24 5.86 / 6.10
    // / 4.82; 8 x 4 x 128, 8 of 1K-8K in 24 35.1 / 35.6 / 30.4, 4K 8.93 / 8.84 / 8.64; 4 x 7 x 128, 48 of 200-4000 in 20 46.4 / 43.3 / 42.4; 8 x 4 x 256, 9 of 1K-5K in 24 48.1 / 44.3 / 43.4.
    constexpr int kLaneRows = 6;
    auto lane_places = [&](int slot0, int rem, int place[kLaneRows]) {
#pragma unroll
        for (int i = 0; i < kLaneRows; ++i) {
            const int r = i < 2 ? k_row(i) : 4 * (i - 2) + tg;
            place[i] = slot0 + (r < rem ? r : 0);
        }
    };
    const int bt_recip = 65536 / max(bt, 1) + 1;
    auto cut_places = [&](int place[kLaneRows], int on[kLaneRows]) {
        if (bt >= kTile) {
#pragma unroll
            for (int i = 0; i < kLaneRows; ++i) {
                on[i] = place[i] >= bt;
                place[i] -= on[i] ? bt : 0;
            }
        } else {
#pragma unroll
            for (int i = 0; i < kLaneRows; ++i) {
                on[i] = (int)(__umul24(place[i], bt_recip) >> 16);
                place[i] -= (int)__umul24(on[i], bt);
            }
        }
    };
    auto fetch_ids = [&](int Tw, Ids &ids) {
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            const int T0 = Tw + kTile * ti;
            const int fb = T0 < t_end ? T0 : Tw;   // a valid row of this tile's block (of the step's first tile when the tile is empty)
            if (TILE_ID) {
                ids.k[ti][0] = ids.t[ti][0] = tbl[block_of(fb)];
            } else {
                const int b0 = block_of(fb);
                int place[kLaneRows], on[kLaneRows];
                ids.slot0[ti] = fb - b0 * bt;
                lane_places(ids.slot0[ti], t_end - T0, place);
                cut_places(place, on);
#pragma unroll
                for (int i = 0; i < 2; ++i) ids.k[ti][i] = tbl[b0 + on[i]];
#pragma unroll
                for (int i = 0; i < 4; ++i) ids.t[ti][i] = tbl[b0 + on[2 + i]];
            }
        }
    };

    // One step in registers: the K tiles in A-operand order, the V rows of this row group's tokens, and which of them count.
    struct Step {
        u32x4 k[TI][NJ];
        vload_t v[TI][4][NV];
        bool ok[TI][4];
    };
    // Strided layout: head h starts a split whose steps are a power of two, 32 and more (128 at head_dim 256), with step h % 8.  All workgroups begin together and read at one pace,
    // and where the strides are powers of two the same step of every head lies at the same place modulo them.  us per layer, all heads from step 0 / from step h, otherwise the same
    // code: 8 x 4 x 128, 32 steps (16K tokens) 15.94 / 15.80, 64 (32K) 26.29 / 26.02, 8 x 16 x 128, 64 27.52 / 27.29, 8 x 4 x 64, 32 16.05 / 15.86; over 22 shapes of 32 and 64 steps
    // 0.5 % less (the worst, 32 KV heads of 32 steps, 15.63 / 16.11); 16 x 1 x 256, 128 steps 82.5 / 80.6.  Other splits gain nothing by it, or lose: 8 and 16 steps level or 1 % slower
    // (one sequence of 8 steps up to 0.8 % faster, two and four 0.5 % slower), 24, 40 and 56 up to 1 % slower; head_dim 256, 32 steps 26.79 / 27.21, 64 46.71 / 46.95
    // (profiles/attn_turn.md); any step of the split, by a hash: 16 x 1 x 256, 4 of 8192 84.8 / 92.2.
    const int n_steps = (t_end - t_begin + kStepTok - 1) / kStepTok;
    constexpr int kTurn = 8;
    const int first_step = (h + b) & (!PAGED && n_steps >= (D < 256 ? 4 : 16) * kTurn && !(n_steps & (n_steps - 1)) ? kTurn - 1 : 0);
    auto step_row = [&](int st) -> int {
        const int s = st + first_step;
        return t_begin + (PAGED || s < n_steps ? s : s - n_steps) * kStepTok;
    };
    // A lane's part of an address, a row number times the row length, is the same in every step and has 32 bits (rows of up to 256 MiB); what changes from tile to
    // tile is the wavefront's part, in scalar registers.  Rows past the end re-read the tile's first one, and are masked.  us per layer from a graph, 64-bit
    // addresses in every lane and the pointer to the sequences' starts waited for / this: 2 x 2 x 64, 256 tokens 4.18 / 3.77; 2 x 6 x 64, 2 of 1K-1.6K 6.65 / 6.48; paged
    // 8 x 4 x 128, 8 of 1K-8K 29.7 / 29.1; the others within 1 %.  (Both kinds of address in the loop: 8 x 4 x 128, 4K 8.50, with this one alone 8.29.)
    // At head_dim 64, fp16, strided, it takes 91 registers where 74 did, and with them the third workgroup of a compute unit: no slower on any shape tried (16 x 4 x 64, 7 of 9000 43.8 /
    // 43.1, 32 x 4, 64 of 500-700 51.6 / 51.8, 8 x 8, 96 of 300-2000 42.6 / 40.5).
    const unsigned row_bytes = PAGED ? 16u * DV : (unsigned)ss * 16u;
    const unsigned k_first = 16u * k_vec(0), v_first = 2u * E * n;
    unsigned k_off[2], v_off[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) k_off[i] = k_first + k_row(i) * row_bytes;
#pragma unroll
    for (int i = 0; i < 4; ++i) v_off[i] = v_first + (4 * i + tg) * row_bytes;
    auto load_step = [&](int st, const Ids &ids, Step &x) {
        const int Tw = step_row(st);
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            const int T0 = Tw + kTile * ti;
            const int R0 = T0 < t_end ? T0 : Tw;      // the tile's first row (an empty tile: the step's)
            const int rem = t_end - T0;
            if constexpr (LAYOUT == kStrided || TILE_ID) {
                const long long tb = row_base(R0, PAGED ? ids.k[ti][0] : 0);
                const bool in_pool = !PAGED || (unsigned)ids.k[ti][0] < (unsigned)p.n_pool;
                const char *const kt = (const char *)(K + tb), *const vt = (const char *)(V + tb);
                unsigned ko[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) ko[i] = k_row(0) < rem - 8 * i ? k_off[i] : k_first;
#pragma unroll
                for (int j = 0; j < NJ; ++j) x.k[ti][j] = __builtin_nontemporal_load((const u32x4 *)(kt + 128 * (j >> 1) + ko[j & 1]));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = tg < rem - 4 * i;
                    x.ok[ti][i] = in_pool && in;
                    const unsigned vo = in ? v_off[i] : v_first;
#pragma unroll
                    for (int w = 0; w < NV; ++w) x.v[ti][i][w] = __builtin_nontemporal_load((const vload_t *)(vt + 32 * E * w + vo));
                }
            } else {
                int place[kLaneRows], on[kLaneRows];
                long long at[kLaneRows];   // the lane's rows, as vector indices
                lane_places(PAGED ? ids.slot0[ti] : 0, rem, place);
                if (PAGED) cut_places(place, on);
#pragma unroll
                for (int i = 0; i < kLaneRows; ++i) {
                    int blk = PAGED ? (i < 2 ? ids.k[ti][i] : ids.t[ti][i - 2]) : 0;
                    if ((unsigned)blk >= (unsigned)p.n_pool) blk = 0;
                    at[i] = PAGED ? (((long long)blk * H + h) * bt + place[i]) * DV : row_base(R0 + place[i], 0);
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j) x.k[ti][j] = __builtin_nontemporal_load(K + at[j & 1] + k_vec(j));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 4 * i + tg, blk = ids.t[ti][i];
                    x.ok[ti][i] = r < rem && (!PAGED || (unsigned)blk < (unsigned)p.n_pool);
                    const vload_t *vp = (const vload_t *)(V + at[2 + i]) + n;
#pragma unroll
                    for (int w = 0; w < NV; ++w) x.v[ti][i][w] = __builtin_nontemporal_load(vp + w * 16);
                }
            }
        }
    };
    const unsigned odd = -(unsigned)(n & 1);   // a mask and not a condition, of which the compiler makes three selects by the element's number
    auto attend = [&](const Step &x) {
        // ---- scores of 16 tokens x 16 columns per tile on the matrix cores
        f32x4 sc[TI];
        float mx = -INFINITY;
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            f32x4 c = {0.f, 0.f, 0.f, 0.f};
            // Rows 4tg + 2i and 4tg + 2i + 1 of u[k] are the first and the second half of token 8k + 4i + tg, each against the columns' halves of the query.
            if constexpr (HALVES) {
                f32x4 u[2] = {c, c};
#pragma unroll
                for (int j = 0; j < NJ; ++j) u[j & 1] = mfma_16x16x32<BF16>(x.k[ti][j], qv[j >> 1], u[j & 1]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float half = __uint_as_float((__float_as_uint(u[i >> 1][2 * (i & 1) + 1]) & odd) | (__float_as_uint(u[i >> 1][2 * (i & 1)]) & ~odd));
                    c[i] = half + dpp_mov<0xB1>(half);   // quad_perm [1,0,3,2]: the other half, from the neighbouring column
                }
            } else {
                f32x4 u[2][2] = {{c, c}, {c, c}};
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int f = 0; f < 2; ++f) u[j & 1][f] = mfma_16x16x32<BF16>(x.k[ti][j], qv[(j & ~1) + f], u[j & 1][f]);
#pragma unroll
                for (int i = 0; i < 4; ++i) c[i] = u[i >> 1][0][2 * (i & 1)] + u[i >> 1][1][2 * (i & 1) + 1];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sc[ti][i] = x.ok[ti][i] ? c[i] : -INFINITY;
                mx = fmaxf(mx, sc[ti][i]);
            }
        }
        // ---- the reference follows the maximum when some score has left it too far behind
        mx *= p.scale_log2e;
        if (__any(mx > m + kRise)) {
            const float mn = fmaxf(m, rows_max(mx));
            const float alpha = exp2f(m - mn);
            l *= alpha;
            m = mn;
#pragma unroll
            for (int w = 0; w < NV; ++w)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    if constexpr (VALU) vacc[w][e] *= alpha;
                    else acc[w][e] *= alpha;
                }
        }
        if constexpr (VALU) {
            // a tile's sum is formed first and enters the accumulator by one addition, as on the matrix cores
            float pr[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) pr[i] = __builtin_amdgcn_exp2f(fmaf(sc[0][i], p.scale_log2e, -m));
            l += (pr[0] + pr[1]) + (pr[2] + pr[3]);
#pragma unroll
            for (int w = 0; w < NV; ++w) {
                float vf[4][8];
#pragma unroll
                for (int i = 0; i < 4; ++i) unpack8<BF16>(x.v[0][i][w], vf[i]);
#pragma unroll
                for (int e = 0; e < E; ++e)
                    vacc[w][e] += fmaf(pr[3], vf[3][e], fmaf(pr[2], vf[2][e], fmaf(pr[1], vf[1][e], pr[0] * vf[0][e])));
            }
            return;
        }
        // ---- probabilities, as sums of 16-bit terms: the B operand (row = token, column = query head)
        unsigned pt[NT][2 * TI];
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
#pragma unroll
            for (int i2 = 0; i2 < 2; ++i2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[ti][2 * i2], p.scale_log2e, -m));
                const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[ti][2 * i2 + 1], p.scale_log2e, -m));
                l += p0 + p1;
                unsigned t[NT];
                split2<BF16>(p0 * kLift<BF16>, p1 * kLift<BF16>, t);
#pragma unroll
                for (int k = 0; k < NT; ++k) pt[k][2 * ti + i2] = t[k];
            }
        // ---- acc += V^T P: A operand row n holds column d = w * 16E + n * E + e of V for this row group's tokens,
        // which this lane has loaded; four tokens of one column are gathered from four registers by byte permutes.
        // Each tile's sum goes into the accumulator by one addition, so that what a tile adds is rounded once at the
        // accumulator's magnitude.  The largest term first: within one operation the matrix core drops what lies far
        // below the largest summand.  For the same reason bf16 terms do not share a product; the two fp16 terms of one tile do
        // (V twice as the A operand).  Products that follow each other in one accumulator are of one shape on purpose: a
        // 16x16x32 product three instructions after a 16x16x16 product whose result it added to once read the last two rows
        // of that result too early here, always the same ones.  Whether the compiler's waits or the source were at fault was
        // not found; no such pair is in the code that the compiler makes, and a test of that code looks for one.
        // Four columns at a time: eight would take the kernel past 128 registers and with that cost the second workgroup of
        // a compute unit (bf16, batch 32 x 32 heads of 512-544 tokens: 10 % more time).
        constexpr int kCols = 4;
#pragma unroll
        for (int w = 0; w < NV; ++w)
#pragma unroll
            for (int e0 = 0; e0 < E; e0 += kCols) {
                unsigned av[kCols][2 * TI];
                f32x4 t[kCols];
#pragma unroll
                for (int e = 0; e < kCols; ++e) {
                    t[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
                        for (int i2 = 0; i2 < 2; ++i2)
                            av[e][2 * ti + i2] = __builtin_amdgcn_perm(x.v[ti][2 * i2 + 1][w][(e0 + e) / 2], x.v[ti][2 * i2][w][(e0 + e) / 2],
                                                                       (e & 1) ? 0x07060302u : 0x05040100u);
                }
                if constexpr (TI == 1 && NT == 2) {
#pragma unroll
                    for (int e = 0; e < kCols; ++e)
                        t[e] = mfma_16x16x32<BF16>(u32x4{av[e][0], av[e][1], av[e][0], av[e][1]},
                                                   u32x4{pt[0][0], pt[0][1], pt[1][0], pt[1][1]}, t[e]);
                } else {
#pragma unroll
                    for (int k = 0; k < NT; ++k)
#pragma unroll
                        for (int e = 0; e < kCols; ++e) {
                            if constexpr (TI == 2)
                                t[e] = mfma_16x16x32<BF16>(u32x4{av[e][0], av[e][1], av[e][2], av[e][3]},
                                                           u32x4{pt[k][0], pt[k][1], pt[k][2], pt[k][3]}, t[e]);
                            else
                                t[e] = mfma_16x16x16<BF16>(u32x2{av[e][0], av[e][1]}, u32x2{pt[k][0], pt[k][1]}, t[e]);
                        }
                }
#pragma unroll
                for (int e = 0; e < kCols; ++e) acc[w][e0 + e] += t[e];
            }
    };

    // Steps are handed out in order, on demand.  A wavefront always knows its current and its next step; the
    // one after that is claimed (one LDS atomic by lane 0) right after the current step's loads are issued,
    // so neither the atomic nor, for the paged layout, the block-table lookup sits on the load chain.
    __shared__ int sh_next;
    // steps 0 .. 2*kWaves-1 are preassigned: w and w + kWaves to wavefront w; a split that has no more needs no counter and
    // no barrier in front of its first loads
    const bool claims = n_steps > 2 * kWaves;
    if (claims) {
        if (threadIdx.x == 0) sh_next = 2 * kWaves;
        __syncthreads();
    }
    int s_cur = wave, s_nxt = wave + kWaves;
    Ids ids{};
    if (PAGED && s_cur < n_steps) fetch_ids(step_row(s_cur), ids);
    while (s_cur < n_steps) {
        Step x;
        load_step(s_cur, ids, x);
        int s_new = n_steps;
        if (claims) {
            if (lane == 0) s_new = atomicAdd(&sh_next, 1);
            s_new = __builtin_amdgcn_readfirstlane(s_new);
        }
        if (PAGED && s_nxt < n_steps) fetch_ids(step_row(s_nxt), ids);
        attend(x);
        s_cur = s_nxt;
        s_nxt = s_new;
    }

    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // formed again: kept through the loop they cost three registers, which the largest instances do not have
    lane = tid & 63;
    n = lane & 15;
    tg = lane >> 4;

    // ---- merge: a wavefront is one softmax state (m, l, acc[D]) per head; the states meet in LDS
    constexpr int DP = D + 4 * kCopies;   // padding: the 16-byte stores of 8 neighbouring lanes fall into different banks
    __shared__ __attribute__((aligned(16))) float sh_acc[kWaves][RG][NH][DP];
    __shared__ f32x2 sh_ml[kWaves][RG * NH];
    auto far = [](float ref) { return fabsf(ref) > kFusedRef && ref != kEmptyMax; };
    constexpr int C = D == 64 ? 1 : D == 256 ? 4 : (NH <= 4 ? 1 : 2), kUnits = D / (64 * C);   // columns of a lane in the merge
    typedef float cols_t __attribute__((ext_vector_type(C)));
    // A wavefront's first states are on their way while the references are looked at.  us per layer from a graph, after / before that: 8 x 4 x 128, 4K tokens 8.21 / 8.15,
    // 1K 6.46 / 6.42; 2 x 2 x 64, 256 3.62 / 3.57; 2 x 6 x 64, 2 of 1K-1.6K 6.54 / 6.43; paged 16 x 8 x 64, 4 of 700 7.73 / 7.62; 8 x 16 x 128, 4K 9.70 / 9.81.  (Over 32 layers of 4K each,
    // 260.8 us / 260.5: level.)
    constexpr bool kEarly = !VALU && NH <= 8;
    f32x2 ml;
    cols_t part[kWaves];
    auto load_unit = [&](int u) {   // the states of 64 * C columns of one head
        const int g = u / kUnits, d = (u % kUnits) * 64 * C + lane * C;
        ml = lane < kWaves ? sh_ml[lane][g] : f32x2{kEmptyMax, 0.f};
#pragma unroll
        for (int k = 0; k < kWaves; ++k) part[k] = *(const cols_t *)&sh_acc[k][0][g][d];
    };
    bool again;   // some accumulated value is not finite, or some reference beyond kFusedRef: the split is done again
    f32x2 state = {kEmptyMax, 0.f};   // VALU: lane = state
    if constexpr (VALU) {
        // position ((2w + e4) * 16 + n) * 4 + k of a state holds column (w * 16 + n) * 8 + 4 * e4 + k: contiguous 16-byte stores
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NV; ++w)
#pragma unroll
            for (int e4 = 0; e4 < 2; ++e4) {
                const float *a = &vacc[w][4 * e4];
                sum += (a[0] + a[1]) + (a[2] + a[3]);
                *(f32x4 *)&sh_acc[wave][tg][0][((2 * w + e4) * 16 + n) * 4] = f32x4{a[0], a[1], a[2], a[3]};
            }
        // an infinite reference in LDS stands for values that are not finite: the references are read anyway, a flag would
        // be one more trip to LDS
        const bool bad = __any(!(fabsf(sum) < INFINITY));
        if (n == 0) sh_ml[wave][tg] = f32x2{bad ? INFINITY : m, l};
        __syncthreads();
        if (lane < RG * kWaves) state = (&sh_ml[0][0])[lane];
        again = __any(far(state[0]));
    } else {
        // A head's columns of the matrix hold the same sums: each of them writes its share.  (Written by one of four, with three of four
        // lanes idle, the stores took four times as many LDS cycles, in front of the barrier.)
        l = rows_sum(l);
        const int g = n / kCopies, copy = n % kCopies;
        constexpr int kParts = NV * E / kCopies;   // 16-byte stores of a lane
        float nf = far(m) ? 1.f : 0.f;   // not 0 (or NaN): again
#pragma unroll
        for (int s = 0; s < kParts; ++s) {
            f32x4 v;
#pragma unroll
            for (int c = 0; c < kCopies; ++c) {
                const int j = s * kCopies + c, w = j / E, i = j % E / (E / 4), e4 = j % (E / 4) * 4;
                const f32x4 u{acc[w][e4][i], acc[w][e4 + 1][i], acc[w][e4 + 2][i], acc[w][e4 + 3][i]};
                if (c == 0) v = u;
                else v = copy == c ? u : v;
            }
            const int j = s * kCopies + copy;
            nf += ((v[0] + v[1]) + (v[2] + v[3])) * 0.f;
            if (g < ng) *(f32x4 *)&sh_acc[wave][0][g][(j / E) * 16 * E + tg * 4 * E + (j % E) * 4] = v;
        }
        const bool bad = __any(!(nf == 0.f));
        if (tg == 0 && copy == 0 && g < ng) sh_ml[wave][g] = f32x2{bad ? INFINITY : m, l};
        __syncthreads();
        if constexpr (kEarly) load_unit(min(wave, ng * kUnits - 1));
        bool some = false;
#pragma unroll
        for (int j0 = 0; j0 < kWaves * NH; j0 += 64) {
            const int j = j0 + lane;
            if (j < kWaves * NH && j % NH < ng) some = some || far((&sh_ml[0][0])[j][0]);
        }
        again = __any(some);
    }

    auto head_out = [&](int g) { return ((long long)b * Hq + hq0 + g) * D; };
    auto head_part = [&](int g) { return ((long long)b * Hq + hq0 + g) * p.n_splits + split; };
    if (__builtin_expect(again, 0)) {   // out of the way of what every launch runs through
        // V (or K, or q) holds infinities or NaNs, or scores are beyond kFusedRef.  The terms of a probability meet an infinite
        // V one by one, and one that is zero or negative turns it into a NaN, so the split is done again with the
        // probability as one factor, and with exponents from score differences: a wavefront takes every kWaves-th run of 8
        // tokens, whose loads are in flight together, for 4 heads at a time, and leaves its states in their places in LDS.
        // (fp16, 8 KV heads x 32K x 128 with one infinity per KV head: 101 us at 4 heads, 62 at one; 539 and 511 with a
        // wavefront per head and a token at a time.)
        constexpr int C = D / 64, kRun = 8, kHeads = NH < 4 ? NH : 4;
        typedef typename std::conditional<BF16, __bf16, _Float16>::type elem_t;
        for (int h0 = 0; h0 < ng; h0 += kHeads) {
            if (h0 == 0) __syncthreads();   // the states' references have been read
            float qs[kHeads][C], a[kHeads][C], ms[kHeads], ls[kHeads];
#pragma unroll
            for (int g = 0; g < kHeads; ++g) {
                const elem_t *qp = (const elem_t *)(q + ((long long)b * Hq + hq0 + min(h0 + g, ng - 1)) * DV);
                ms[g] = kEmptyMax;
                ls[g] = 0.f;
#pragma unroll
                for (int c = 0; c < C; ++c) { qs[g][c] = (float)qp[c * 64 + lane]; a[g][c] = 0.f; }
            }
            for (int t0 = t_begin + kRun * wave; t0 < t_end; t0 += kRun * kWaves) {
                elem_t kv[kRun][C], vv[kRun][C];
                bool ok[kRun];
#pragma unroll
                for (int i = 0; i < kRun; ++i) {   // rows past the end re-read the split's last row; masked below
                    const int t = min(t0 + i, t_end - 1), blk = PAGED ? tbl[block_of(t)] : 0;
                    ok[i] = t0 + i < t_end && (!PAGED || (unsigned)blk < (unsigned)p.n_pool);
                    const long long rb = row_base(t, blk);
                    const elem_t *kp = (const elem_t *)(K + rb), *vp = (const elem_t *)(V + rb);
#pragma unroll
                    for (int c = 0; c < C; ++c) { kv[i][c] = kp[c * 64 + lane]; vv[i][c] = vp[c * 64 + lane]; }
                }
#pragma unroll
                for (int g = 0; g < kHeads; ++g) {
                    if (h0 + g >= ng) continue;
                    float s[kRun], mn = ms[g];
#pragma unroll
                    for (int i = 0; i < kRun; ++i) {
                        float dot = 0.f;
#pragma unroll
                        for (int c = 0; c < C; ++c) dot = fmaf(qs[g][c], (float)kv[i][c], dot);
                        s[i] = wave_sum(dot);
                        if (ok[i]) mn = fmaxf(mn, s[i]);
                    }
                    const float al = exp2f((ms[g] - mn) * p.scale_log2e);
                    ms[g] = mn;
                    ls[g] *= al;
#pragma unroll
                    for (int c = 0; c < C; ++c) a[g][c] *= al;
#pragma unroll
                    for (int i = 0; i < kRun; ++i) {
                        if (!ok[i]) continue;   // its row may be another sequence's, or infinite: not even times zero
                        const float pr = exp2f((s[i] - mn) * p.scale_log2e);
                        ls[g] += pr;
#pragma unroll
                        for (int c = 0; c < C; ++c) a[g][c] = fmaf(pr, (float)vv[i][c], a[g][c]);
                    }
                }
            }
#pragma unroll
            for (int g = 0; g < kHeads; ++g) {
                if (h0 + g >= ng) continue;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const int d = c * 64 + lane;
                    if constexpr (VALU) {
                        const int pos = ((2 * (d / 128) + ((d >> 2) & 1)) * 16 + ((d >> 3) & 15)) * 4 + (d & 3);
                        sh_acc[wave][0][h0 + g][pos] = a[g][c];
#pragma unroll
                        for (int r = 1; r < RG; ++r) sh_acc[wave][r][h0 + g][pos] = 0.f;
                    } else {
                        sh_acc[wave][0][h0 + g][d] = a[g][c] * kLift<BF16>;
                    }
                }
                if (VALU) {
                    if (lane < RG) sh_ml[wave][lane] = f32x2{ms[g] * p.scale_log2e, lane == 0 ? ls[g] : 0.f};
                } else if (lane == 0) {
                    sh_ml[wave][h0 + g] = f32x2{ms[g] * p.scale_log2e, ls[g]};
                }
            }
        }
        __syncthreads();
        if (VALU && lane < RG * kWaves) state = (&sh_ml[0][0])[lane];
        if constexpr (kEarly) load_unit(min(wave, ng * kUnits - 1));
    }
    if constexpr (VALU) {
        // 64 positions per wavefront, which forms the states' weights itself (lane = state) and takes them from the lanes by readlane
        for (int base = wave * 64; base < D; base += kThreads) {
            const int pos = base + lane, d = ((pos / 128) * 16 + ((pos >> 2) & 15)) * 8 + ((pos >> 6) & 1) * 4 + (pos & 3);
            const float M = wave_max(state[0]);
            const float wgt = exp2f(state[0] - M);
            const float L = wave_sum(state[1] * wgt);
            float A = 0.f;
#pragma unroll
            for (int k = 0; k < kWaves; ++k)
                A = fmaf((sh_acc[k][0][0][pos] + sh_acc[k][1][0][pos]) + (sh_acc[k][2][0][pos] + sh_acc[k][3][0][pos]), rdlane(wgt, RG * k), A);
            if (p.direct_mode >= 0) {
                store_out(p.out, head_out(0) + d, p.direct_mode, L == 0.f ? 0.f : A / L);
            } else {
                p.part_acc[head_part(0) * D + d] = A;
                if (pos == 0) *(f32x2 *)&p.part_ml[head_part(0) * 2] = f32x2{M, L};
            }
        }
        return;
    }
    // A wavefront forms 64 * C columns of one head at a time: lane = state for the weights, which it then takes from the lanes
    // by readlane, one weight's exponential per lane in place of every state's in every lane.  us per layer from a graph, together with the stores above:
    // 8 KV heads x 4 x 128, 1K tokens 7.1 / 6.7, 4K 8.75 / 8.3; 2 x 2 x 64, 256 tokens 4.4 / 3.95; 4 x 2 x 256, 2 sequences of 3000
    // 11.3 / 10.7; paged, 2 x 7, 4K 8.0 / 7.7; 32K and larger batches within 1 %.
    static_assert(kWaves <= 8, "half a row of lanes");
    for (int u = wave; u < ng * kUnits; u += kWaves) {
        const int g = u / kUnits, d = (u % kUnits) * 64 * C + lane * C;
        if (!kEarly || u != wave) load_unit(u);
        const float Ml = half_row_max(ml[0]);
        const float wgt = exp2f(ml[0] - Ml);
        const float M = rdlane(Ml, 0), L = rdlane(half_row_sum(ml[1] * wgt), 0);
        float A[C] = {};
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            const float f = rdlane(wgt, k) * (1.f / kLift<BF16>);
#pragma unroll
            for (int c = 0; c < C; ++c) A[c] = fmaf(part[k][c], f, A[c]);
        }
        if (p.direct_mode >= 0) {   // the only split of its sequence: the result itself
#pragma unroll
            for (int c = 0; c < C; ++c) A[c] = L == 0.f ? 0.f : A[c] / L;
            store_outs<C>(p.out, head_out(g) + d, p.direct_mode, A);
        } else {
            cols_t v;
#pragma unroll
            for (int c = 0; c < C; ++c) v[c] = A[c];
            *(cols_t *)&p.part_acc[head_part(g) * D + d] = v;
            if (d == 0) *(f32x2 *)&p.part_ml[head_part(g) * 2] = f32x2{M, L};
        }
    }
}

// out_mode: 0 fp32, 1 fp16, 2 bf16.  One workgroup of W wavefronts per (hq, b).  A lane loads 16 bytes of a partial row, so a load of a
// wavefront is one, two or four rows (head_dim 256, 128, 64), and a round of a wavefront 8, 8 or 16 rows.  Every
// wavefront forms the split weights exp2(m_s - M) itself (lane = split, 64 at a time, the maximum carried along)
// and takes them from the lanes by readlane.  The loads of the (m, l) pairs and of the first round do not depend on each other
// and are issued together, and every further round while the one before is added: up to a round of splits the kernel is one memory latency
// long.  The wavefronts' sums are added through LDS; up to 8 (16) splits are one wavefront's work, without LDS or barrier, and up to
// twice as many two wavefronts'.  us per layer from a graph, four wavefronts that load 4 bytes per lane / this: 8 KV heads x 4 x 128, 4K tokens (32 splits)
// 8.3 / 8.1; 1 x 8 x 128, 16K (64) 10.35 / 10.0; 4 x 2 x 256, 2 of 3000 (32) 10.7 / 10.3; paged, 48 sequences, 4 x 7 x 128 (up to 7) 43.7 / 42.9,
// 24 sequences, 8 x 8 x 64 24.8 / 24.0.  With four wavefronts for few splits as well, the last two are 44.5 and 25.7.
constexpr int combine_loads(int D) { return D == 256 ? 8 : 4; }                      // loads of a wavefront per round
constexpr int combine_rows(int D) { return combine_loads(D) * (D >= 256 ? 1 : 256 / D); }   // partial rows of a wavefront per round

template <int D, int W, typename TAB>
__global__ void __launch_bounds__(64 * W)
kv_attn_combine_kernel(const float *__restrict__ part_acc, const float *__restrict__ part_ml,
                       void *__restrict__ out, const int *__restrict__ seq_lens, int Hq, int n_splits_alloc, int out_mode,
                       int n_uniform, int max_len, int split_tokens, TAB tab)
{
    constexpr int kRowLanes = D / 4, RPL = 64 / kRowLanes;    // lanes of a row, rows of a load
    constexpr int kLoads = combine_loads(D), kRound = W * kLoads * RPL;
    static_assert(kLoads * RPL == combine_rows(D), "rows of a round");
    constexpr bool kSkips = W == 1 || std::is_same<TAB, CountTable>::value;   // a round is often not full: loads past its last row are left out
    const int hq = blockIdx.x, b = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = lane / kRowLanes, d = (lane % kRowLanes) * 4;
    const long long o = ((long long)b * Hq + hq) * n_splits_alloc;
    // only the splits that hold tokens of this sequence were written (and matter)
    int n_splits;
    if constexpr (std::is_same<TAB, CountTable>::value) {
        n_splits = tab.splits[b];
    } else {
        n_splits = n_uniform;   // every sequence has as many; a division here would be on the way to the first load
        if (n_splits < 0) n_splits = min(n_splits_alloc, splits_of(max(0, min(seq_lens[b], max_len)), split_tokens));
    }

    const float *const pa = part_acc + o * D;
    const f32x2 *const pm = (const f32x2 *)part_ml + o;
    // Loads are not masked (each would be a branch): what lies past the last split re-reads the first one and is dropped when it is used.
    auto load_ml = [&](int s0) { return pm[(unsigned)(s0 + lane < n_splits ? s0 + lane : 0)]; };
    auto load_rows = [&](int s0, f32x4 rows[kLoads]) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int s_first = s0 + (i * W + wave) * RPL, s = s_first + sub;
            if (kSkips && s_first >= n_splits) break;
            rows[i] = *(const f32x4 *)&pa[(unsigned)((s < n_splits ? s : 0) * D + d)];
        }
    };
    f32x2 ml = load_ml(0);
    f32x4 rows[kLoads];
    load_rows(0, rows);                                  // independent of the weights
    f32x4 A = {0.f, 0.f, 0.f, 0.f};
    float M = kEmptyMax, L = 0.f;
    for (int s0 = 0; s0 < n_splits; s0 += 64) {          // 64 splits at a time: lane = split
        f32x2 ml_next;
        if (s0 + 64 < n_splits) ml_next = load_ml(s0 + 64);
        if (s0 + lane >= n_splits) ml = f32x2{kEmptyMax, 0.f};
        const float Mn = fmaxf(M, wave_max(ml[0])), rescale = exp2f(M - Mn), wgt = exp2f(ml[0] - Mn);
        M = Mn;
        A *= rescale;
        L = fmaf(ml[1], wgt, L * rescale);
#pragma unroll
        for (int r0 = 0; r0 < 64; r0 += kRound) {        // the next rows are on their way while these are added
            if (s0 + r0 >= n_splits) break;
            f32x4 next[kLoads];
            if (s0 + r0 + kRound < n_splits) load_rows(s0 + r0 + kRound, next);
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const int j = r0 + (i * W + wave) * RPL;
                if (kSkips && s0 + j >= n_splits) break;
                float w = rdlane(wgt, j);
#pragma unroll
                for (int k = 1; k < RPL; ++k) {
                    const float wk = rdlane(wgt, j + k);
                    w = sub == k ? wk : w;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) A[k] = fmaf(s0 + j + sub < n_splits ? rows[i][k] : 0.f, w, A[k]);
            }
#pragma unroll
            for (int i = 0; i < kLoads; ++i) rows[i] = next[i];
        }
        ml = ml_next;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (RPL == 4) A[k] = rows_sum(A[k]);
        if (RPL == 2) A[k] = halves_sum(A[k]);
    }
    L = wave_sum(L);
    if constexpr (W > 1) {
        __shared__ __attribute__((aligned(16))) float sums[W][D];
        if (sub == 0) *(f32x4 *)&sums[wave][d] = A;
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int k = 1; k < W; ++k) A += *(const f32x4 *)&sums[k][d];
    }
    if (sub == 0) {
        float r[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = L == 0.f ? 0.f : A[k] / L;   // nothing attended: zeros; a NaN score: NaN
        store_outs<4>(out, ((long long)b * Hq + hq) * D + d, out_mode, r);
    }
}

AttnShape attn_shape(const kv_plan *p)
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cus = n;
        else
            cus = 256;
    }
    return AttnShape{p->B, p->H, p->Hq, p->D, cus};
}

template <int D, int NH, bool BF16, typename TAB>
void launch_partial(dim3 grid, hipStream_t st, const AttnHead &c, const AttnParams &a, const TAB &t)
{
    const unsigned heads = pack16(c.H, c.G), shares = pack16(c.gt, c.subs) | (std::is_same<TAB, ItemTable>::value ? (unsigned)c.heads_first << 7 | (unsigned)c.B << 8 : 0u);
    typename std::conditional<std::is_same<TAB, ItemTable>::value, const int *, unsigned long long>::type lens;
    if constexpr (std::is_same<TAB, ItemTable>::value) lens = a.seq_lens;
    else lens = (unsigned)c.split_tokens | (unsigned long long)(unsigned)c.len_uniform << 32;
    const dim3 block(64 * waves(D));
    if (!c.table) {
        const PackedStrides ps = pack_strides(c.strides);
        const int high = ps.high | (a.seq_off ? kSeqOff : 0);
        if (c.strides.ss < kFarRows)
            (void)kvb::launch_kernel(kv_attn_partial_kernel<D, NH, BF16, kStrided, TAB>, grid, block, st, c.K, c.V, c.q, lens, heads, shares,
                               ps.ss_sh, ps.sb, high, a, t);
        else
            (void)kvb::launch_kernel(kv_attn_partial_kernel<D, NH, BF16, kStridedFar, TAB>, grid, block, st, c.K, c.V, c.q, lens, heads, shares,
                               ps.ss_sh, ps.sb, high, a, t);
    } else if (c.bt % kTile == 0) {
        (void)kvb::launch_kernel(kv_attn_partial_kernel<D, NH, BF16, kPagedTiles, TAB>, grid, block, st, c.K, c.V, c.q, lens, heads, shares,
                           c.table, c.max_blocks, c.bt, a, t);
    } else {
        (void)kvb::launch_kernel(kv_attn_partial_kernel<D, NH, BF16, kPagedRows, TAB>, grid, block, st, c.K, c.V, c.q, lens, heads, shares,
                           c.table, c.max_blocks, c.bt, a, t);
    }
}

template <int D, int NH, typename TAB>
void launch_partial_type(bool bf16, dim3 grid, hipStream_t st, const AttnHead &c, const AttnParams &a, const TAB &t)
{
    if (bf16) launch_partial<D, NH, true>(grid, st, c, a, t);
    else launch_partial<D, NH, false>(grid, st, c, a, t);
}

template <int D, typename TAB>
void launch_partial_nh(bool bf16, dim3 grid, hipStream_t st, const AttnHead &c, const AttnParams &a, const TAB &t)
{
    if constexpr (D >= 128) {
        if (c.gt == 1) return launch_partial_type<D, 1>(bf16, grid, st, c, a, t);
    }
    if (c.gt <= 4) launch_partial_type<D, 4>(bf16, grid, st, c, a, t);   // from here on NH only sizes the merge's LDS
    else if (c.gt <= 8) launch_partial_type<D, 8>(bf16, grid, st, c, a, t);
    else launch_partial_type<D, kMaxHeads>(bf16, grid, st, c, a, t);
}

template <typename TAB>
void launch_partial_d(int D, bool bf16, dim3 grid, hipStream_t st, const AttnHead &c, const AttnParams &a, const TAB &t)
{
    if (D == 64) launch_partial_nh<64>(bf16, grid, st, c, a, t);
    else if (D == 128) launch_partial_nh<128>(bf16, grid, st, c, a, t);
    else launch_partial_nh<256>(bf16, grid, st, c, a, t);
}

template <typename TAB>
void launch_combine(int D, dim3 grid, hipStream_t st, const AttnHead &c, const AttnParams &a, int out_mode, const TAB &t)
{
    const int n_uniform = c.len_uniform < 0 ? -1 : std::min(a.n_splits, splits_of(c.len_uniform, c.split_tokens));
#define KV_COMBINE_W(DD, W)                                                                                      \
    (void)kvb::launch_kernel(kv_attn_combine_kernel<DD, W, TAB>, grid, dim3(64 * W), st, a.part_acc, a.part_ml, a.out, \
                       a.seq_lens, c.Hq, a.n_splits, out_mode, n_uniform, a.max_len, c.split_tokens, t)
#define KV_COMBINE(DD) { if (a.n_splits <= combine_rows(DD)) KV_COMBINE_W(DD, 1); else if (a.n_splits <= 2 * combine_rows(DD)) KV_COMBINE_W(DD, 2); else KV_COMBINE_W(DD, 4); }
    if (D == 64) KV_COMBINE(64)
    else if (D == 128) KV_COMBINE(128)
    else KV_COMBINE(256)
#undef KV_COMBINE
#undef KV_COMBINE_W
}

}  // namespace

extern "C" size_t kv_decode_attn_workspace(const kv_plan_t *p, int n_splits, int max_len)
{
    if (!p || n_splits < 0 || max_len < 0) return 0;
    const int ns = n_splits > 0 ? n_splits : max_auto_splits(attn_shape(p), max_len);
    return (size_t)p->B * p->Hq * ns * (p->D + 2) * sizeof(float);
}

namespace {

// Checks, split choice and the two launches; shared by both entry points.  Allocates nothing.
int decode_attn(const kv_plan_t *p, const kv_view_t *kv, int layer, const void *q, void *out, int out_dtype,
                int n_splits, void *workspace, size_t ws_bytes, void *hip_stream)
{
    if (!p || !kv || !q || !out || !workspace) return KV_EINVAL;
    if (out_dtype != KV_OUT_F32 && out_dtype != KV_OUT_SAME) return KV_EINVAL;
    if (n_splits < 0 || n_splits > kMaxSplits) return KV_EINVAL;
    if (p->D != 64 && p->D != 128 && p->D != 256) return KV_EINVAL;
    if (!kv->k_layers || !kv->v_layers || !kv->seq_lens_host || !kv->seq_lens_dev) return KV_EINVAL;
    if (layer < 0 || layer >= p->L || layer >= kv->n_layers) return KV_ERANGE;
    const void *K = kv->k_layers[layer], *V = kv->v_layers[layer];
    if (!K || !V) return KV_EINVAL;
    if (((uintptr_t)K | (uintptr_t)V | (uintptr_t)q | (uintptr_t)workspace) & 15) return KV_EINVAL;
    if (p->B > 65535 || p->Hq > 65535) return KV_EINVAL;

    int max_len = 0;
    for (int b = 0; b < p->B; ++b) {
        const int len = kv->seq_lens_host[b];
        if (len < 0) return KV_EINVAL;
        max_len = std::max(max_len, len);
    }
    AttnHead c{};
    AttnParams a{};
    const bool paged = kv->layout == KV_LAYOUT_PAGED;
    if (kv->layout == KV_LAYOUT_BHSD) {
        if (kv->stride_b < 0 || kv->stride_h < 0 || kv->stride_s < p->D) return KV_EINVAL;
        if ((kv->stride_b | kv->stride_h | kv->stride_s) & 7) return KV_EINVAL;
        if (max_len > kv->s_alloc) return KV_ERANGE;
        if ((kv->seq_off_host == nullptr) != (kv->seq_off_dev == nullptr)) return KV_EINVAL;
        for (int b = 0; b < p->B; ++b) {  // the last element any sequence reads must lie inside the buffer
            const int len = kv->seq_lens_host[b];
            if (len == 0) continue;
            if (kv->seq_off_host && (kv->seq_off_host[b] < 0 || (kv->seq_off_host[b] & 7))) return KV_EINVAL;
            const uint64_t base = kv->seq_off_host ? (uint64_t)kv->seq_off_host[b] : (uint64_t)b * kv->stride_b;
            const uint64_t max_elem = base + (uint64_t)(p->H - 1) * kv->stride_h + (uint64_t)(len - 1) * kv->stride_s + p->D;
            if (max_elem * 2 > kv->layer_bytes) return KV_ERANGE;
        }
        c.strides = Strides{(unsigned long long)kv->stride_s / 8, (unsigned long long)kv->stride_h / 8, (unsigned long long)kv->stride_b / 8};
        a.seq_off = (const long long *)kv->seq_off_dev;
    } else if (paged) {
        if (!kv->block_table || kv->block_tokens < 1 || kv->n_pool_blocks < 0) return KV_EINVAL;
        if ((uint64_t)kv->n_pool_blocks * p->H * kv->block_tokens * p->D * 2 > kv->layer_bytes) return KV_ERANGE;
        if (kvb::ceil_div((uint64_t)max_len, (uint64_t)kv->block_tokens) > (uint64_t)kv->max_blocks_per_seq)
            return KV_ERANGE;
        if (max_len > 0 && kv->n_pool_blocks < 1) return KV_ERANGE;
        c.table = kv->block_table;
        c.max_blocks = kv->max_blocks_per_seq;
        c.bt = kv->block_tokens;
        a.n_pool = kv->n_pool_blocks;
    } else {
        return KV_EINVAL;
    }

    c.len_uniform = max_len;
    for (int b = 0; b < p->B; ++b)
        if (kv->seq_lens_host[b] != max_len) c.len_uniform = -1;

    // Splits.  A uniform batch takes one split length for all sequences and the grid (split, query-head group, sequence).  A ragged batch of up
    // to kMaxTableSeqs sequences launches workgroups only for splits that hold tokens: its grid walks a table of per-sequence
    // split counts.
    AttnCut cut{};
    if (!cut_tokens(attn_shape(p), kv->seq_lens_host, n_splits, ws_bytes, &cut)) return KV_ENOSPC;
    const SplitTable &tab = cut.tab;
    const bool use_table = cut.use_table;
    const int ns = cut.ns, G = p->Hq / p->H;
    c.split_tokens = cut.split_tokens;
    c.subs = cut.subs;
    c.gt = (G + c.subs - 1) / c.subs;
    c.K = (const u32x4 *)K; c.V = (const u32x4 *)V; c.q = (const u32x4 *)q;
    a.seq_lens = kv->seq_lens_dev;
    a.part_acc = (float *)workspace;
    a.part_ml = a.part_acc + (size_t)p->B * p->Hq * ns * p->D;
    c.H = p->H; c.Hq = p->Hq; c.G = G; c.B = p->B;
    a.n_splits = ns;
    a.max_len = max_len;
    a.scale_log2e = (float)(1.4426950408889634 / std::sqrt((double)p->D));

    hipStream_t st = (hipStream_t)hip_stream;
    const bool bf16 = p->dtype == KV_BF16;
    const int out_mode = out_dtype == KV_OUT_F32 ? 0 : (bf16 ? 2 : 1);
    // One split per sequence: there is nothing to combine, and the partial kernel writes the results.  (In the table's
    // grid a sequence without tokens has no workgroup that could write its zeros.)
    bool direct = ns == 1 && max_len > 0;
    for (int b = 0; use_table && b < p->B; ++b) direct = direct && kv->seq_lens_host[b] > 0;
    a.direct_mode = direct ? out_mode : -1;
    a.out = out;
    const long long n_items = use_table ? tab.first[p->B] : (max_len > 0 ? (long long)ns * p->B : 0);
    const unsigned groups = (unsigned)(p->H * c.subs);
    if (n_items > 0) {
        if (use_table) {
            ItemTable items;
            for (int r = 0, first = 0; r < kMaxTableSeqs; ++r) {
                const int b = r < p->B ? cut.order[r] : 0;
                items.first[r] = r < p->B ? first : INT_MAX;
                items.tokens[r] = tab.tokens[b];
                items.seq[r] = (unsigned char)b;
                first += tab.first[b + 1] - tab.first[b];
            }
            c.heads_first = cut.longest_first;
            const dim3 grid = cut.longest_first ? dim3(groups, (unsigned)n_items, 1u) : dim3((unsigned)n_items, groups, 1u);
            launch_partial_d(p->D, bf16, grid, st, c, a, items);
        } else {
            launch_partial_d(p->D, bf16, dim3((unsigned)ns, groups, (unsigned)p->B), st, c, a, NoTable{});
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { kvb::set_hip_error((int)e); return KV_EHIP; }
    }

    if (direct) return KV_OK;
    const dim3 cgrid((unsigned)p->Hq, (unsigned)p->B, 1u);
    if (use_table) {
        CountTable counts{};
        for (int b = 0; b < p->B; ++b) counts.splits[b] = (unsigned short)(tab.first[b + 1] - tab.first[b]);
        launch_combine(p->D, cgrid, st, c, a, out_mode, counts);
    } else {
        launch_combine(p->D, cgrid, st, c, a, out_mode, NoTable{});
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { kvb::set_hip_error((int)e); return KV_EHIP; }
    return KV_OK;
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each GPU, resolved on the first call there

}  // namespace

// Split partials of kv_decode_attn_static: every GPU the library runs on holds its own copy of this array
// until the process ends.  In host code the name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[KV_ATTN_SCRATCH_BYTES];

extern "C" int kv_decode_attn_splits(const kv_plan_t *p, const int32_t *seq_lens_host, int n_splits, int *n_splits_out,
                                     int *first, int *tokens)
{
    if (!p || !seq_lens_host || !n_splits_out) return KV_EINVAL;
    if (n_splits < 0 || n_splits > kMaxSplits) return KV_EINVAL;
    if (p->D != 64 && p->D != 128 && p->D != 256) return KV_EINVAL;
    for (int b = 0; b < p->B; ++b)
        if (seq_lens_host[b] < 0) return KV_EINVAL;
    SplitTable tab{};
    bool use_table = false;
    int st = 0;
    *n_splits_out = plan_splits(attn_shape(p), planned_parts(p->Hq / p->H), seq_lens_host, n_splits, kMaxSplits, &use_table, &tab, &st);
    int acc = 0;
    for (int b = 0; b < p->B; ++b) {
        if (first) first[b] = acc;
        if (tokens) tokens[b] = use_table ? tab.tokens[b] : st;
        acc += use_table ? tab.first[b + 1] - tab.first[b] : std::min(*n_splits_out, splits_of(seq_lens_host[b], st));
    }
    if (first) first[p->B] = acc;
    return KV_OK;
}

extern "C" int kv_decode_attn(const kv_plan_t *p, const kv_view_t *kv, int layer, const void *q, void *out,
                              int out_dtype, int n_splits, void *workspace, size_t ws_bytes, void *hip_stream)
{
    return decode_attn(p, kv, layer, q, out, out_dtype, n_splits, workspace, ws_bytes, hip_stream);
}

extern "C" int kv_decode_attn_static(const kv_plan_t *p, const kv_view_t *kv, int layer, const void *q, void *out,
                                     int out_dtype, int n_splits, void *hip_stream)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) { kvb::set_hip_error((int)e); return KV_EHIP; }
    if (dev < 0 || dev >= kMaxDevices) return KV_EINVAL;
    void *ws = nullptr;
    {
        std::lock_guard<std::mutex> g(g_scratch_mu);
        if (!g_scratch_ptr[dev]) {
            // the array's name is a host-side stand-in; its device address on the current GPU is looked up once
            void *ptr = nullptr;
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !ptr) { kvb::set_hip_error((int)e); return KV_EHIP; }
            g_scratch_ptr[dev] = ptr;
        }
        ws = g_scratch_ptr[dev];
    }
    // decode_attn answers KV_ENOSPC when the partials of this call do not fit the array
    return decode_attn(p, kv, layer, q, out, out_dtype, n_splits, ws, (size_t)KV_ATTN_SCRATCH_BYTES, hip_stream);
}
