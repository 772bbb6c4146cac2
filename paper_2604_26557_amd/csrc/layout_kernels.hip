// Pack / unpack: the byte permutation between the attention-side KV layout (strided [B,H,S,D] or a
// paged block pool) and extent order, the row-major (S, B*H, D) array of Sec. IV-B.
//
// The innermost D row (D*2 bytes, a multiple of 16) is preserved by the permutation, so the kernels
// move whole 16-byte vectors: one lane = one global_load_dwordx4 + one global_store_dwordx4.
// Threads are laid out as (rx, ty): rx walks the vectors of one extent row (consecutive lanes ->
// consecutive extent bytes and whole head rows of the source), ty walks token rows.  The (b, h, d)
// decomposition of a row position is done once per thread per row position and reused for every token, so
// the inner loop is adds, U independent 16-byte loads, then U stores.  HBM-bound: 2 bytes of traffic per
// payload byte, no reuse, no LDS.  Where a plain copy reaches 6.3 TB/s, launches of 128 MiB and more run at
// 5.5-6.3 (strided, rows to 4 KiB), 5.0-5.9 (strided, wider rows of 128- and 256-wide heads; 64-wide 4.6-4.9)
// and 4.5-6.0 (paged; 32 heads x 128, batch 4 of 2000: 5.6).  32 layers of 8 heads x 4K tokens x 128 out of one launch pair: 169 us for 1 GiB of traffic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "launch.hpp"
#include "plan.hpp"

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kMaxSegs = 32;
constexpr int kTblStage = 64;  // block-table entries one workgroup can stage in LDS

// Attention-side addressing, in 16-byte vectors.
struct SrcDesc {
    long long sb, sh, ss;  // strided layout: vectors per batch / head / token step
    const int *table;      // paged layout
    int max_blocks, bt, bt_shift, n_pool;
    int H, dvec;           // heads, vectors per head row
};

// One contiguous run of token rows of one (sub-)extent inside the image buffer.
struct Seg {
    unsigned long long img_off;  // vector index in the image of row 0 of this run
    unsigned long long pad_off;  // vector index of the first pad vector (pack only)
    unsigned int pad_vecs;       // zero vectors to write (pack only)
    int b;                       // sequence, or -1: the batch index is part of the row position
    int tok0, ntok;
    u32x4 *base;                 // the attention-side buffer this run belongs to (K or V of some layer)
};

// Grid (tiles of the longest run, run): workgroups past a shorter run's end return at once.
struct SegTable {
    static constexpr bool kDense = false;
    Seg seg[kMaxSegs];
};
// The runs lie one after the other in the grid's x dimension, run i in [first[i], first[i + 1]), and a workgroup looks up its run.
struct DenseSegTable {
    static constexpr bool kDense = true;
    Seg seg[kMaxSegs];
    int first[kMaxSegs + 1];
    int n;
};

// Every byte is touched once: nontemporal loads and stores keep the streams out of each other's way in L2.
__device__ __forceinline__ u32x4 ld(const u32x4 *p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void st(u32x4 *p, u32x4 v) { __builtin_nontemporal_store(v, p); }

// PACK: source -> image.  !PACK: image -> source.  U = token rows in flight per thread.
template <bool PACK, bool PAGED, int U, typename TAB>
__global__ void __launch_bounds__(kThreads)
kv_layout_kernel(SrcDesc s, u32x4 *__restrict__ img, TAB segs, int rowv, int rx_log2, int tpb, int rchunk)
{
    int run = blockIdx.y, tile = blockIdx.x, n_tiles = gridDim.x;
    if constexpr (TAB::kDense) {
        int lo = 0, hi = segs.n;   // the last run that starts at or before this workgroup
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (segs.first[mid] <= tile) lo = mid; else hi = mid;
        }
        run = lo;
        n_tiles = segs.first[run + 1] - segs.first[run];
        tile -= segs.first[run];
    }
    const Seg sg = segs.seg[run];
    const int tid = threadIdx.x;
    u32x4 *const base = sg.base;

    if (PACK && sg.pad_vecs && blockIdx.z == 0) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        for (unsigned int i = tile * kThreads + tid; i < sg.pad_vecs; i += n_tiles * kThreads)
            img[sg.pad_off + i] = z;
    }

    const int t_begin = tile * tpb;
    if (t_begin >= sg.ntok) return;
    const int t_end = min(sg.ntok, t_begin + tpb);

    const int RX = 1 << rx_log2;
    const int TY = kThreads >> rx_log2;
    const int rx = tid & (RX - 1);
    const int ty = tid >> rx_log2;
    const int hd = s.H * s.dvec;

    // Paged source, one sequence per segment: the few block-table entries this tile touches are staged in
    // LDS once, so the per-token lookup is not a second dependent trip to memory.  Where a thread has one token the lookup is one trip
    // anyway, and staging only adds the way through LDS and a barrier to the short life of a workgroup (16 heads x 256, batch 4: 361 / 357 us for
    // 6 layers staged, 303 / 314 not; pack / unpack).
    __shared__ int sh_tbl[kTblStage];
    int j_first = 0;
    bool tbl_in_lds = false;
    if (PAGED && sg.b >= 0 && tpb > TY) {
        j_first = (sg.tok0 + t_begin) / s.bt;
        const int nj = (sg.tok0 + t_end - 1) / s.bt - j_first + 1;
        if (nj <= kTblStage) {  // uniform over the workgroup
            const int *row = s.table + (long long)sg.b * s.max_blocks;
            for (int i = tid; i < nj; i += kThreads) sh_tbl[i] = row[j_first + i];
            __syncthreads();
            tbl_in_lds = true;
        }
    }

    // this workgroup's share of the row positions (a wide row is cut into chunks, so that a tile spans fewer
    // source head rows and more tokens of each)
    const int r_begin = blockIdx.z * rchunk, r_end = min(rowv, r_begin + rchunk);
    for (int r = r_begin + rx; r < r_end; r += RX) {
        int b, rem;
        if (sg.b >= 0) { b = sg.b; rem = r; } else { b = r / hd; rem = r - b * hd; }
        const int h = rem / s.dvec;
        const int dv = rem - h * s.dvec;
        const long long row_off = PAGED ? 0 : (long long)b * s.sb + (long long)h * s.sh + dv;
        const int *tbl = PAGED ? s.table + (long long)b * s.max_blocks : nullptr;

        for (int t0 = t_begin + ty; t0 < t_end; t0 += TY * U) {
            u32x4 v[U];
            long long a[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + u * TY;
                ok[u] = t < t_end;
                a[u] = 0;
                if (ok[u]) {
                    const int tok = sg.tok0 + t;
                    if (PAGED) {
                        const int j = s.bt_shift >= 0 ? (tok >> s.bt_shift) : (tok / s.bt);
                        const int slot = tok - j * s.bt;
                        const int blk = tbl_in_lds ? sh_tbl[j - j_first] : tbl[j];
                        ok[u] = (unsigned)blk < (unsigned)s.n_pool;  // ids outside the pool are skipped
                        a[u] = (((long long)blk * s.H + h) * s.bt + slot) * s.dvec + dv;
                    } else {
                        a[u] = row_off + (long long)tok * s.ss;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned long long i = sg.img_off + (unsigned long long)(t0 + u * TY) * rowv + r;
                if (ok[u]) v[u] = PACK ? ld(base + a[u]) : ld(img + i);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned long long i = sg.img_off + (unsigned long long)(t0 + u * TY) * rowv + r;
                if (PACK) {
                    // a skipped block id still owns its bytes of the image: they read as zero
                    const bool in = (t0 + u * TY) < t_end;
                    const u32x4 z = {0u, 0u, 0u, 0u};
                    if (in) st(img + i, ok[u] ? v[u] : z);
                } else if (ok[u]) {
                    st(base + a[u], v[u]);
                }
            }
        }
    }
}

// The newest token rows of many tensors and sequences, one workgroup column per row: a decode step's write-back is a few
// KiB per tensor, so what it costs is launches and copies, not bytes.  The tables go by value: 32 layers and 128
// sequences per launch (one launch for 512 rows of 2 KiB, where segments of 32 rows took 16 launches).  The rows are
// written where the host reads them: into pinned memory, 16 bytes per lane and whole rows per workgroup, without a
// staging copy (the runtime's 1 MiB device-to-host copy alone takes 20 us behind the last launch).
constexpr int kRowLayers = 32, kRowSeqs = 128;
struct RowTable {
    const u32x4 *base[2 * kRowLayers];  // K, V of each layer
    int tok[kRowSeqs];                  // the row of each sequence
};

template <bool PAGED>
__global__ void __launch_bounds__(kThreads)
kv_rows_kernel(SrcDesc s, u32x4 *__restrict__ dst, RowTable t, int rowv, int nseq, int b_first)
{
    const int tok = t.tok[blockIdx.x];
    const u32x4 *const base = t.base[blockIdx.y];
    const int hd = s.H * s.dvec;
    u32x4 *const row = dst + ((long long)blockIdx.y * nseq + blockIdx.x) * rowv;
    for (int r = blockIdx.z * blockDim.x + threadIdx.x; r < rowv; r += gridDim.z * blockDim.x) {
        const int b = b_first >= 0 ? b_first + (int)blockIdx.x : r / hd;   // token-major: a row holds all sequences
        const int rem = b_first >= 0 ? r : r - b * hd;
        const int h = rem / s.dvec, dv = rem - h * s.dvec;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (PAGED) {
            const int j = s.bt_shift >= 0 ? (tok >> s.bt_shift) : (tok / s.bt);
            const int blk = s.table[(long long)b * s.max_blocks + j];
            if ((unsigned)blk < (unsigned)s.n_pool)   // ids outside the pool are skipped: their bytes read as zero
                v = ld(base + (((long long)blk * s.H + h) * s.bt + (tok - j * s.bt)) * s.dvec + dv);
        } else {
            v = ld(base + (long long)b * s.sb + (long long)h * s.sh + (long long)tok * s.ss + dv);
        }
        st(row + r, v);
    }
}

int check_view(const kv_plan *p, const kv_view_t *v, int layer)
{
    if (!v || !v->k_layers || !v->v_layers || !v->seq_lens_host) return KV_EINVAL;
    if (layer < 0 || layer >= p->L || layer >= v->n_layers) return KV_ERANGE;
    if (!v->k_layers[layer] || !v->v_layers[layer]) return KV_EINVAL;
    if (((uintptr_t)v->k_layers[layer] | (uintptr_t)v->v_layers[layer]) & 15) return KV_EINVAL;
    if (v->seq_off_host || v->seq_off_dev) return KV_EINVAL;  // per-sequence offsets are for attention only
    if (v->layout == KV_LAYOUT_BHSD) {
        if (v->stride_b < 0 || v->stride_h < 0 || v->stride_s < 0 || v->s_alloc < 0) return KV_EINVAL;
        if ((v->stride_b | v->stride_h | v->stride_s) & 7) return KV_EINVAL;
        if (v->stride_s < p->D) return KV_EINVAL;
    } else if (v->layout == KV_LAYOUT_PAGED) {
        if (!v->block_table || v->block_tokens < 1 || v->n_pool_blocks < 0 || v->max_blocks_per_seq < 0)
            return KV_EINVAL;
        const uint64_t pool = (uint64_t)v->n_pool_blocks * p->H * v->block_tokens * p->D * 2;
        if (pool > v->layer_bytes) return KV_ERANGE;
    } else {
        return KV_EINVAL;
    }
    return KV_OK;
}

// Rows [tok0, tok0+ntok) of sequence b (or of every sequence when b < 0) must exist in the view.
int check_rows(const kv_plan *p, const kv_view_t *v, int b, int tok0, int ntok)
{
    const int b0 = b < 0 ? 0 : b, b1 = b < 0 ? p->B : b + 1;
    const long long last = (long long)tok0 + ntok;  // one past the last row
    if (ntok == 0) return KV_OK;
    if (v->layout == KV_LAYOUT_BHSD) {
        if (last > v->s_alloc) return KV_ERANGE;
        const uint64_t max_elem = (uint64_t)(b1 - 1) * v->stride_b + (uint64_t)(p->H - 1) * v->stride_h +
                                  (uint64_t)(last - 1) * v->stride_s + p->D;
        if (max_elem * 2 > v->layer_bytes) return KV_ERANGE;
    } else {
        for (int i = b0; i < b1; ++i) {
            if (last > v->seq_lens_host[i]) return KV_ERANGE;
            if (kvb::ceil_div((uint64_t)last, (uint64_t)v->block_tokens) > (uint64_t)v->max_blocks_per_seq)
                return KV_ERANGE;
        }
    }
    return KV_OK;
}

u32x4 *tensor_base(const kv_view_t *v, int layer, int which)
{
    return (u32x4 *)(which == 0 ? v->k_layers[layer] : v->v_layers[layer]);
}

SrcDesc make_src(const kv_plan *p, const kv_view_t *v)
{
    SrcDesc s{};
    s.H = p->H;
    s.dvec = p->D / 8;
    if (v->layout == KV_LAYOUT_BHSD) {
        s.sb = v->stride_b / 8; s.sh = v->stride_h / 8; s.ss = v->stride_s / 8;
    } else {
        s.table = v->block_table;
        s.max_blocks = v->max_blocks_per_seq;
        s.bt = v->block_tokens;
        s.bt_shift = (s.bt & (s.bt - 1)) == 0 ? __builtin_ctz((unsigned)s.bt) : -1;
        s.n_pool = v->n_pool_blocks;
    }
    return s;
}

// Launch shape.  rx_cap: most lanes (log2) along an extent row; unroll: token rows in flight per thread (1 or 2);
// tile_bytes: extent bytes one workgroup moves; run_bytes: consecutive source bytes per head row a tile should reach when
// the row is cut into chunks (0: one sweep of the lanes), which takes precedence over tile_bytes.
struct Shape {
    int rx_cap, unroll, tile_bytes, run_bytes;
};

// Many small workgroups, one or two vectors per lane in flight, beat fewer and larger ones at every shape measured: the launch
// order then walks both sides nearly in order, so what is in flight at one time is a compact window of memory, where 16-64 KiB
// tiles with 4-8 vectors per lane kept hundreds of scattered streams open.  What differs is which way a workgroup lies in the
// permutation (us, 32-64 KiB tiles as they were -> now; pack / unpack; heads of 128 unless stated):
//  * strided, rows of up to 4 KiB: one head row by the workgroup's tokens (4 KiB of one head's stream).  8 heads x 4K tokens,
//    32 layers in one launch pair 188 / 188 -> 171 / 171; x 32K, 8 layers 381 / 372 -> 367 / 355; 30001 tokens 374 / 347 -> 331 / 330; ragged
//    batch of 8 472 / 458 -> 422 / 420.  Whole rows (16 KiB) are as good at 4K but alias at power-of-two strides (32K: 411).
//  * strided, wider rows: 4 KiB of the row by one token (heads of 128), by two (256: 8 KiB) or by eight (64: 32 KiB), one after the
//    other.  us per layer: 16 heads, batch 4 of 4096 47.3 / 48.8 -> 48.4 / 46.7 (by four tokens 50.2 / 49.4), of 3500 43.4 / 44.0 -> 41.0 / 40.5
//    (43.1 / 42.8); 20 heads, batch 3 39.2 / 38.6 -> 34.6 / 33.6 (37.5 / 35.9); 16 heads x 256, batch 2 38.7 / 39.2 -> 34.2 / 34.6 (by one
//    token 34.9 / 33.8); 4 heads x 64, batch 28 38.6 / 37.9 -> 25.4 / 25.2; 8 x 64, batch 8 of 4096 37.9 / 37.8 -> 27.6 / 27.9 (by one 29.4 / 27.9).
//  * paged, rows of up to 4 KiB: whole rows, since a pool block holds all heads of its tokens.  Ragged batch of 8 438 / 480 -> 413 / 449;
//    8 heads x 256, batch 6 404 / 515 -> 376 / 391; one sequence of 8000 243 / 250 -> 219 / 226; 5 heads, where the lanes do not divide the
//    row, 38.6 / 41.4 -> 36.4 / 38.2 per layer.
//  * paged, wider rows: 4 KiB of one token's row, or 8 KiB where 4 do not divide the row (the last workgroup of a row would have little
//    to do: 9 heads x 256, batch 4, unpack 218 against 200). Such a workgroup needs one block id and does not stage the table (see the
//    kernel); with that, tiles of two head rows by one block's tokens (8 KiB), which 64- and 128-wide heads had, are no longer better.
//    us for 6 layers, as it was -> now, pack / unpack: 32 heads x 128, batch 4 of 1K-3K 293 / 274 -> 243 / 247, 20 heads, batch 3 149 / 151 ->
//    144 / 142; 16 heads x 256, batch 4 of 2K-3K 361 / 358 -> 305 / 317, 9 heads 272 / 265 -> 204 / 200; 64 heads x 64 (2 layers) 98 / 92 ->
//    82 / 83.  Rows of up to 4 KiB gain nothing from 4 KiB tiles: 8 heads x 128, ragged batch of 8 (8 layers) 407 / 451, with them 418 / 443; 5 heads
//    121 / 123, with them 138 / 137.
Shape pick_shape(bool paged, int rowv, int dvec)
{
    if (paged && rowv > 256) return Shape{8, 1, rowv % 256 == 0 ? 4 * 1024 : 8 * 1024, 0};
    if (paged) return Shape{8, 2, 8 * 1024, 4 * 1024};
    if (rowv > 256) return Shape{8, 1, 4 * 1024, dvec == 16 ? 0 : 1024};
    int lanes = 4;   // one head row, at least 16 lanes
    while ((1 << lanes) < dvec && lanes < 8) ++lanes;
    return Shape{lanes, 1, 4 * 1024, 2 * 1024};
}

// A ragged batch whose tiles fill little of the grid (tiles of the longest run, run) takes the dense one.  The lookup costs a workgroup
// some percent, one that returns at once costs about a tenth of one that moves a tile.  us per layer, first grid / dense, by how much
// is filled: 4 % (32 sequences, one of 16K tokens and the others of about 200; 8 heads x 128) strided 131 / 38, paged 80 / 39; strided 18 %
// (32 sequences, the others at 15 % of the longest; 2 heads x 128, 8 x 64) 15.6 / 13.2 and 22.4 / 22.1, 27 % 18.8 / 17.8 and 29.6 / 31.4;
// paged 18 % 16.6 / 14.5 and 22.0 / 23.2.
bool dense_grid(bool paged, unsigned total, unsigned most, int n) { return (unsigned long long)total * (paged ? 8 : 5) < (unsigned long long)most * n; }

template <bool PACK, bool PAGED, typename TAB>
void launch_u(int U, dim3 grid, hipStream_t stream, const SrcDesc &s, void *img, const TAB &tab, int rowv, int rx_log2,
              int tpb, int rchunk)
{
    if (U == 1) (void)kvb::launch_kernel(kv_layout_kernel<PACK, PAGED, 1, TAB>, grid, dim3(kThreads), stream, s, (u32x4 *)img, tab, rowv, rx_log2, tpb, rchunk);
    else (void)kvb::launch_kernel(kv_layout_kernel<PACK, PAGED, 2, TAB>, grid, dim3(kThreads), stream, s, (u32x4 *)img, tab, rowv, rx_log2, tpb, rchunk);
}

template <bool PACK>
int launch(const kv_plan *p, const kv_view_t *v, const Seg *segs, int nseg, void *img, hipStream_t stream)
{
    const int rowv = (int)(p->row_bytes / 16);
    const bool paged = v->layout == KV_LAYOUT_PAGED;
    const Shape sh = pick_shape(paged, rowv, p->D / 8);
    int rx_log2 = 0;
    while ((1 << rx_log2) < rowv && rx_log2 < sh.rx_cap) ++rx_log2;
    const int TY = kThreads >> rx_log2;
    const int U = sh.unroll;
    const long long tile_bytes = sh.tile_bytes;
    // Tile = tpb token rows x rchunk row positions, about tile_bytes of extent.  A row wider than one sweep of
    // the workgroup is cut into chunks of row positions, and the tile gets more tokens instead, so that every
    // source head row it touches contributes at least run_bytes of consecutive tokens.
    const long long head_row_bytes = (long long)p->D * 2;
    long long want_tok = tile_bytes / (long long)p->row_bytes;
    if (rowv > (1 << rx_log2)) want_tok = std::max<long long>(want_tok, sh.run_bytes / head_row_bytes);
    int tpb = (int)std::max<long long>(1, want_tok);
    // a grid has fewer than 2^32 threads in a dimension: at most 2^18 tiles of a run, times kMaxSegs runs, times kThreads
    int max_tok = 0, min_tok = INT_MAX;
    for (int i = 0; i < nseg; ++i) {
        max_tok = std::max(max_tok, segs[i].ntok);
        min_tok = std::min(min_tok, segs[i].ntok);
    }
    tpb = std::max(tpb, (int)(((long long)max_tok + (1 << 18) - 1) >> 18));
    tpb = (tpb + TY * U - 1) / (TY * U) * (TY * U);
    const int RXv = 1 << rx_log2;
    long long chunk = std::max<long long>(RXv, tile_bytes / 16 / tpb);
    chunk = std::max<long long>(chunk, (rowv + 65534) / 65535);   // at most 65535 chunks in the grid
    chunk = (chunk + RXv - 1) / RXv * RXv;
    const int rchunk = (int)std::min<long long>(chunk, (rowv + RXv - 1) / RXv * RXv);
    const unsigned n_rchunks = (unsigned)((rowv + rchunk - 1) / rchunk);
    const SrcDesc s = make_src(p, v);
    auto tiles_of = [&](int ntok) { return std::max(1u, ((unsigned)ntok + (unsigned)tpb - 1u) / (unsigned)tpb); };   // a run without rows may have a pad

    for (int g0 = 0; g0 < nseg; g0 += kMaxSegs) {
        const int n = std::min(kMaxSegs, nseg - g0);
        unsigned most = tiles_of(max_tok), total = most * (unsigned)n;
        if (min_tok != max_tok) {
            most = total = 0;
            for (int i = 0; i < n; ++i) {
                const unsigned tiles = tiles_of(segs[g0 + i].ntok);
                total += tiles;
                most = std::max(most, tiles);
            }
        }
        if (dense_grid(paged, total, most, n)) {
            DenseSegTable tab{};
            for (int i = 0; i < n; ++i) {
                tab.seg[i] = segs[g0 + i];
                tab.first[i + 1] = tab.first[i] + (int)tiles_of(segs[g0 + i].ntok);
            }
            tab.n = n;
            const dim3 grid(total, 1u, n_rchunks);
            if (paged) launch_u<PACK, true>(U, grid, stream, s, img, tab, rowv, rx_log2, tpb, rchunk);
            else launch_u<PACK, false>(U, grid, stream, s, img, tab, rowv, rx_log2, tpb, rchunk);
        } else {
            SegTable tab{};
            for (int i = 0; i < n; ++i) tab.seg[i] = segs[g0 + i];
            const dim3 grid(most, (unsigned)n, n_rchunks);
            if (paged) launch_u<PACK, true>(U, grid, stream, s, img, tab, rowv, rx_log2, tpb, rchunk);
            else launch_u<PACK, false>(U, grid, stream, s, img, tab, rowv, rx_log2, tpb, rchunk);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { kvb::set_hip_error((int)e); return KV_EHIP; }
    }
    return KV_OK;
}

// Runs of the whole extent image of tensor (layer, which) placed at byte img_off of the image buffer: rows
// [0, len_b) of every sequence and the zero pad up to each (sub-)extent's end.
int whole_extent_segs(const kv_plan *p, const kv_view_t *v, int layer, int which, uint64_t img_off, std::vector<Seg> *segs)
{
    const uint64_t sec = (uint64_t)p->sector;
    const uint64_t image = p->tensor_blocks * sec;
    if (p->mode == KV_TOKEN_MAJOR) {
        const int len = v->seq_lens_host[0];
        for (int b = 0; b < p->B; ++b)
            if (v->seq_lens_host[b] != len) return KV_EINVAL;
        if (len < 0 || len > p->cap[0]) return KV_ERANGE;
        int rc = check_rows(p, v, -1, 0, len);
        if (rc != KV_OK) return rc;
        Seg s{};
        s.img_off = img_off / 16;
        s.b = -1; s.tok0 = 0; s.ntok = len; s.base = tensor_base(v, layer, which);
        s.pad_off = s.img_off + (uint64_t)len * p->row_bytes / 16;
        s.pad_vecs = (unsigned)((image - (uint64_t)len * p->row_bytes) / 16);
        segs->push_back(s);
        return KV_OK;
    }
    for (int b = 0; b < p->B; ++b) {
        const int len = v->seq_lens_host[b];
        if (len < 0 || len > p->cap[b]) return KV_ERANGE;
        int rc = check_rows(p, v, b, 0, len);
        if (rc != KV_OK) return rc;
        const uint64_t sub_bytes = kvb::round_up((uint64_t)p->cap[b] * p->row_bytes, sec);
        Seg s{};
        s.img_off = (img_off + p->seq_base[b] * sec) / 16;
        s.b = b; s.tok0 = 0; s.ntok = len; s.base = tensor_base(v, layer, which);
        s.pad_off = s.img_off + (uint64_t)len * p->row_bytes / 16;
        s.pad_vecs = (unsigned)((sub_bytes - (uint64_t)len * p->row_bytes) / 16);
        if (len > 0 || s.pad_vecs > 0) segs->push_back(s);
    }
    return KV_OK;
}

// Whole extent images of K and V of layers [layer_begin, layer_end), back to back in tensor-id order (layer
// ascending, K before V), in as few launches as the segment table allows: a small layer alone is too short a
// launch to reach HBM speed.
template <bool PACK>
int run_layers(const kv_plan *p, int layer_begin, int layer_end, const kv_view_t *v, void *img, size_t img_bytes,
               void *hip_stream)
{
    if (!p || !img || ((uintptr_t)img & 15)) return KV_EINVAL;
    if (layer_begin < 0 || layer_end > p->L || layer_begin > layer_end) return KV_ERANGE;
    if (p->row_bytes / 16 > (uint64_t)INT_MAX) return KV_EINVAL;
    const uint64_t image = p->tensor_blocks * (uint64_t)p->sector;
    if (img_bytes < (uint64_t)(layer_end - layer_begin) * 2 * image) return KV_ENOSPC;
    std::vector<Seg> segs;
    for (int l = layer_begin; l < layer_end; ++l) {
        int rc = check_view(p, v, l);
        if (rc != KV_OK) return rc;
        for (int w = 0; w < 2; ++w) {
            rc = whole_extent_segs(p, v, l, w, ((uint64_t)(l - layer_begin) * 2 + (uint64_t)w) * image, &segs);
            if (rc != KV_OK) return rc;
        }
    }
    if (!PACK)
        for (Seg &s : segs) s.pad_vecs = 0;
    if (segs.empty()) return KV_OK;
    return launch<PACK>(p, v, segs.data(), (int)segs.size(), img, (hipStream_t)hip_stream);
}

template <bool PACK>
int run(const kv_plan *p, int layer, int kind, const kv_view_t *v, int seq, int tok0, int ntok, void *img,
        size_t img_bytes, void *hip_stream)
{
    if (!p || !img) return KV_EINVAL;
    if (kind != KV_K && kind != KV_V && kind != KV_KV) return KV_EINVAL;
    if ((uintptr_t)img & 15) return KV_EINVAL;
    int rc = check_view(p, v, layer);
    if (rc != KV_OK) return rc;
    if (p->row_bytes / 16 > (uint64_t)INT_MAX) return KV_EINVAL;
    hipStream_t stream = (hipStream_t)hip_stream;
    const uint64_t sec = (uint64_t)p->sector;
    const int first = kind == KV_V ? 1 : 0, last = kind == KV_K ? 0 : 1;  // KV_KV: K image, then V image
    const uint64_t n_img = (uint64_t)(last - first + 1);

    std::vector<Seg> segs;
    if (seq == KV_SEQ_ALL && tok0 == 0 && ntok == 0) {
        // Whole extent image(s).
        const uint64_t image = p->tensor_blocks * sec;
        if (img_bytes < n_img * image) return KV_ENOSPC;
        for (int w = first; w <= last; ++w) {
            rc = whole_extent_segs(p, v, layer, w, (uint64_t)(w - first) * image, &segs);
            if (rc != KV_OK) return rc;
        }
    } else {
        kvb::RowRange r;
        rc = kvb::resolve_rows(p, seq, tok0, ntok, &r);
        if (rc != KV_OK) return rc;
        // with KV_KV the V range follows the K range at req_bytes
        if (img_bytes < (n_img - 1) * r.req_bytes + (PACK ? r.req_bytes : r.payload)) return KV_ENOSPC;
        const int b = p->mode == KV_TOKEN_MAJOR ? -1 : r.b;
        rc = check_rows(p, v, b, tok0, ntok);
        if (rc != KV_OK) return rc;
        for (int w = first; w <= last; ++w) {
            Seg s{};
            s.img_off = (uint64_t)(w - first) * r.req_bytes / 16;
            s.b = b; s.tok0 = tok0; s.ntok = ntok; s.base = tensor_base(v, layer, w);
            s.pad_off = s.img_off + r.payload / 16;
            s.pad_vecs = (unsigned)((r.req_bytes - r.payload) / 16);
            segs.push_back(s);
        }
    }
    if (!PACK)
        for (Seg &s : segs) s.pad_vecs = 0;
    if (segs.empty()) return KV_OK;
    return launch<PACK>(p, v, segs.data(), (int)segs.size(), img, stream);
}

}  // namespace

namespace kvb {
// The newest token row (row len_b - 1, len_b = v->seq_lens_host[b]) of every tensor of layers
// [layer_begin, layer_end) and every sequence, in extent order, packed back to back at dst in the order
// (layer, K then V, sequence) -- one row of all sequences per tensor in token-major mode.  No sector
// alignment rule and no padding: the decode append merges the rows into their sectors on the host.
// dst: device memory or pinned host memory, which the kernel writes through the link.
int pack_last_rows(const kv_plan *p, const kv_view_t *v, int layer_begin, int layer_end, void *dst, size_t dst_bytes,
                   hipStream_t stream)
{
    if (!p || !dst || ((uintptr_t)dst & 15)) return KV_EINVAL;
    if (layer_begin < 0 || layer_end > p->L || layer_begin >= layer_end) return KV_ERANGE;
    if (p->row_bytes / 16 > (uint64_t)INT_MAX) return KV_EINVAL;
    const int nseq = p->mode == KV_TOKEN_MAJOR ? 1 : p->B;
    const uint64_t n_rows = (uint64_t)(layer_end - layer_begin) * 2 * (uint64_t)nseq;
    if (dst_bytes < n_rows * p->row_bytes) return KV_ENOSPC;
    for (int l = layer_begin; l < layer_end; ++l) {
        const int rc = check_view(p, v, l);
        if (rc != KV_OK) return rc;
    }
    for (int i = 0; i < nseq; ++i) {   // the same for every layer
        const int len = v->seq_lens_host[i];
        if (len < 1 || len > p->cap[i]) return KV_ERANGE;
        const int rc = check_rows(p, v, p->mode == KV_TOKEN_MAJOR ? -1 : i, len - 1, 1);
        if (rc != KV_OK) return rc;
    }
    const SrcDesc s = make_src(p, v);
    const int rowv = (int)(p->row_bytes / 16);
    const int threads = std::min(kThreads, (rowv + 63) / 64 * 64);
    const unsigned gz = (unsigned)std::min((rowv + threads - 1) / threads, 65535);
    for (int l0 = layer_begin; l0 < layer_end; l0 += kRowLayers) {
        const int nl = std::min(kRowLayers, layer_end - l0);
        for (int b0 = 0; b0 < nseq; b0 += kRowSeqs) {
            const int nb = std::min(kRowSeqs, nseq - b0);
            RowTable t{};
            for (int i = 0; i < 2 * nl; ++i) t.base[i] = tensor_base(v, l0 + i / 2, i % 2);
            for (int i = 0; i < nb; ++i) t.tok[i] = v->seq_lens_host[b0 + i] - 1;
            u32x4 *out = (u32x4 *)dst + ((size_t)(l0 - layer_begin) * 2 * nseq + b0) * rowv;
            const dim3 grid((unsigned)nb, (unsigned)(2 * nl), gz);
            const int b_first = p->mode == KV_TOKEN_MAJOR ? -1 : b0;
            if (v->layout == KV_LAYOUT_PAGED)
                (void)kvb::launch_kernel(kv_rows_kernel<true>, grid, dim3(threads), stream, s, out, t, rowv, nseq, b_first);
            else
                (void)kvb::launch_kernel(kv_rows_kernel<false>, grid, dim3(threads), stream, s, out, t, rowv, nseq, b_first);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) { kvb::set_hip_error((int)e); return KV_EHIP; }
        }
    }
    return KV_OK;
}
}

extern "C" int kv_offload_pack(const kv_plan_t *plan, int layer, int kind, const kv_view_t *src, int seq, int tok0,
                               int ntok, void *dst_dev, size_t dst_bytes, void *hip_stream)
{
    return run<true>(plan, layer, kind, src, seq, tok0, ntok, dst_dev, dst_bytes, hip_stream);
}

extern "C" int kv_reload_unpack(const kv_plan_t *plan, int layer, int kind, const void *src_dev, size_t src_bytes,
                                const kv_view_t *dst, int seq, int tok0, int ntok, void *hip_stream)
{
    return run<false>(plan, layer, kind, dst, seq, tok0, ntok, const_cast<void *>(src_dev), src_bytes, hip_stream);
}

extern "C" int kv_offload_pack_layers(const kv_plan_t *plan, int layer_begin, int layer_end, const kv_view_t *src,
                                      void *dst_dev, size_t dst_bytes, void *hip_stream)
{
    return run_layers<true>(plan, layer_begin, layer_end, src, dst_dev, dst_bytes, hip_stream);
}

extern "C" int kv_reload_unpack_layers(const kv_plan_t *plan, int layer_begin, int layer_end, const void *src_dev,
                                       size_t src_bytes, const kv_view_t *dst, void *hip_stream)
{
    return run_layers<false>(plan, layer_begin, layer_end, dst, const_cast<void *>(src_dev), src_bytes, hip_stream);
}
