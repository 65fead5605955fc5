// Heavy rows accumulated straight from a chunk-major copy of B, with no
// expansion in memory.
//
// C's columns are cut into chunks of TILE_COLS = 2^14. The B rows that the
// heavy rows use (the slices) are copied once into chunk-major order: chunk c
// holds, slice by slice, the part of every slice's row that falls in the
// chunk, with 16-bit chunk-local columns. A region is a heavy row of C
// restricted to one chunk (or, for sparse rows, to several adjacent chunks);
// its products are the parts that the row's A entries meet in it, scaled. The
// non-empty parts of every region are listed once (start, length, A entry);
// then a wave or a work group per region reads its parts and accumulates them
// in LDS, counting distinct columns in the symbolic phase and summing values
// in the numeric phase.
//
// Why: writing the products out, splitting them by column and reading them
// back twice moves about 34 bytes per product through HBM. Here a product
// costs 2 bytes of reads in the symbolic and 10 in the numeric phase, about half
// of them or more served by the L2s (regions of more than 2048 products of an
// R-MAT 22 panel: 59 to 84 % hits in the symbolic, 41 to 63 % in the numeric
// kernels, which take 4.5 to 5.6 TB/s of lines from behind them) because regions
// run in chunk order and share the chunk's part of B.
// The price is one visit per (A entry, chunk), so the path is taken when the
// entries' parts are long enough (use_tiles in plan.hip).
#include <algorithm>
#include <type_traits>

#include "host.hpp"
#include "rank.hpp"

namespace gm {

namespace {

constexpr int TWORDS = TILE_COLS / 32;
constexpr int TU = 4;                       // products per lane in flight (8: the same times)
constexpr int TWIN = GM_WAVE * TU;          // products of one wave window
constexpr int TLONG = 256;                  // longer parts are shared by the work group's waves
constexpr int TLONG_CAP = 128;              // parts the shared list holds

// ------------------------------------------------------------- chunk-major B
constexpr int TR_WAVES = 4, TR_ILP = 8, TR_STREAM = 4096, TR_PER = 4;

// Elements of every slice's B row per chunk: cnt[s * nc + c]. One wave per
// slice. Rows of at most TR_STREAM elements are read once and counted by runs
// (a sorted row meets every chunk in one run per 64 elements); longer rows
// take the chunk bounds by binary searches, TR_PER per lane stepping together.
template <typename CI>
__global__ __launch_bounds__(TR_WAVES * GM_WAVE) void k_tile_row_counts(CsrV<CI, NoV> B, const int32_t *slice_k,
                                                                        int64_t ns, int nc, uint16_t *cnt) {
    extern __shared__ uint32_t tr_hist[];  // TR_WAVES * (nc + 1)
    const int lane = threadIdx.x & (GM_WAVE - 1);
    uint32_t *hist = tr_hist + (threadIdx.x / GM_WAVE) * (nc + 1);
    const int64_t nwaves = (int64_t)gridDim.x * TR_WAVES;
    for (int64_t s = blockIdx.x * (int64_t)TR_WAVES + threadIdx.x / GM_WAVE; s < ns; s += nwaves) {
        const int32_t k = slice_k[s];
        const int64_t b0 = B.rp[k], len = B.rp[k + 1] - b0;
        const CI *row = B.ci + b0;
        uint16_t *out = cnt + s * nc;
        if (len <= TR_STREAM) {  // uniform over the wave
            for (int f = lane; f < nc; f += GM_WAVE) hist[f] = 0;
            wave_lds_fence();
            for (int p0 = 0; p0 < (int)len; p0 += GM_WAVE * TR_ILP) {
                int fc[TR_ILP];
#pragma unroll
                for (int u = 0; u < TR_ILP; ++u) {
                    const int p = p0 + u * GM_WAVE + lane;
                    const int64_t f = p < (int)len ? ((int64_t)row[p] >> TILE_LOG2) : -1;
                    fc[u] = f < nc ? (int)f : nc - 1;
                }
#pragma unroll
                for (int u = 0; u < TR_ILP; ++u) {
                    const int fp = prev_lane(fc[u], -2);
                    const uint64_t starts = ballot(fc[u] >= 0 && fc[u] != fp);
                    if (fc[u] >= 0 && ((starts >> lane) & 1)) {
                        const uint64_t above = starts & ~((lanemask_lt() << 1) | 1ull);
                        const int left = (int)len - (p0 + u * GM_WAVE);
                        const int end = above ? __ffsll((long long)above) - 1 : (left < GM_WAVE ? left : GM_WAVE);
                        atomicAdd(&hist[fc[u]], (uint32_t)(end - lane));
                    }
                }
            }
            wave_lds_fence();
            for (int f = lane; f < nc; f += GM_WAVE) out[f] = (uint16_t)hist[f];
            wave_lds_fence();  // the counters are read before the next slice clears them
            continue;
        }
        for (int f0 = 0; f0 <= nc; f0 += TR_PER * GM_WAVE) {
            int64_t lo[TR_PER], hi[TR_PER];
#pragma unroll
            for (int j = 0; j < TR_PER; ++j) {
                const int f = f0 + lane + j * GM_WAVE;
                lo[j] = f < nc ? 0 : len;  // bound nc is the row's end
                hi[j] = len;
            }
            for (int st = 64 - __clzll((long long)len); st > 0; --st) {
#pragma unroll
                for (int j = 0; j < TR_PER; ++j) {
                    const int64_t mid = (lo[j] + hi[j]) >> 1;
                    const bool go = lo[j] < hi[j];
                    const int64_t col = go ? (int64_t)row[mid] : 0;
                    if (go) {
                        if (col < ((int64_t)(f0 + lane + j * GM_WAVE) << TILE_LOG2))
                            lo[j] = mid + 1;
                        else
                            hi[j] = mid;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < TR_PER; ++j) {
                const int f = f0 + lane + j * GM_WAVE;
                if (f <= nc) hist[f] = (uint32_t)lo[j];
            }
        }
        wave_lds_fence();
        for (int f = lane; f < nc; f += GM_WAVE) out[f] = (uint16_t)(hist[f + 1] - hist[f]);
        wave_lds_fence();
    }
}

// out[c * rows + r] = in[r * cols + c], 64 x 64 tiles through LDS.
constexpr int TT = 64;
template <typename T>
__global__ __launch_bounds__(256) void k_tile_transpose(const T *in, int64_t rows, int64_t cols, uint32_t *out) {
    __shared__ uint32_t t[TT][TT + 1];
    const int64_t n_rt = (rows + TT - 1) / TT;
    const int64_t r0 = (blockIdx.x % n_rt) * TT, c0 = (blockIdx.x / n_rt) * TT;
    const int x = threadIdx.x & (TT - 1), y0 = threadIdx.x / TT;
    for (int y = y0; y < TT; y += 256 / TT)
        if (r0 + y < rows && c0 + x < cols) t[y][x] = in[(r0 + y) * cols + c0 + x];
    __syncthreads();
    for (int y = y0; y < TT; y += 256 / TT)
        if (c0 + y < cols && r0 + x < rows) out[(c0 + y) * rows + r0 + x] = t[x][y];
}

// In-place exclusive scan of uint32 values (sums below 2^32).
constexpr int SC_BLOCK = 256, SC_ITEMS = 16;
constexpr int64_t SC_TILE = SC_BLOCK * SC_ITEMS;

GM_DEV void sc_load(const uint32_t *a, int64_t base, int64_t n, uint32_t (&v)[SC_ITEMS]) {
    if (base + SC_ITEMS <= n) {  // base is a multiple of 16 and the array 16-byte aligned
#pragma unroll
        for (int j = 0; j < SC_ITEMS; j += 4) {
            const uint4 q = *(const uint4 *)(a + base + j);
            v[j] = q.x;
            v[j + 1] = q.y;
            v[j + 2] = q.z;
            v[j + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < SC_ITEMS; ++j) v[j] = base + j < n ? a[base + j] : 0u;
    }
}

__global__ __launch_bounds__(SC_BLOCK) void k_tile_scan_sums(const uint32_t *a, int64_t n, uint32_t *sums) {
    __shared__ uint32_t sm[SC_BLOCK / GM_WAVE];
    uint32_t v[SC_ITEMS];
    sc_load(a, blockIdx.x * SC_TILE + (int64_t)threadIdx.x * SC_ITEMS, n, v);
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < SC_ITEMS; ++j) s += v[j];
    const uint32_t tot = block_reduce_sum<SC_BLOCK>(s, sm);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_tile_scan_mid(uint32_t *sums, int64_t n) {
    __shared__ uint32_t sm[1024 / GM_WAVE];
    uint32_t carry = 0;
    for (int64_t b = 0; b < n; b += 1024) {
        const int64_t i = b + threadIdx.x;
        const uint32_t x = i < n ? sums[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_excl_scan<1024>(x, sm, &tot);
        if (i < n) sums[i] = carry + ex;
        carry += tot;
    }
}

// (also writes the total at a[n])
__global__ __launch_bounds__(SC_BLOCK) void k_tile_scan_apply(uint32_t *a, int64_t n, const uint32_t *sums) {
    __shared__ uint32_t sm[SC_BLOCK / GM_WAVE];
    const int64_t base = blockIdx.x * SC_TILE + (int64_t)threadIdx.x * SC_ITEMS;
    uint32_t v[SC_ITEMS];
    sc_load(a, base, n, v);
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < SC_ITEMS; ++j) s += v[j];
    uint32_t run = sums[blockIdx.x] + block_excl_scan<SC_BLOCK>(s, sm);
#pragma unroll
    for (int j = 0; j < SC_ITEMS; ++j) {
        const uint32_t x = v[j];
        v[j] = run;
        run += x;
    }
    if (base + SC_ITEMS <= n) {
#pragma unroll
        for (int j = 0; j < SC_ITEMS; j += 4) *(uint4 *)(a + base + j) = make_uint4(v[j], v[j + 1], v[j + 2], v[j + 3]);
    } else {
#pragma unroll
        for (int j = 0; j < SC_ITEMS; ++j)
            if (base + j < n) a[base + j] = v[j];
    }
    if (base <= n - 1 && n - 1 < base + SC_ITEMS) a[n] = run;
}

// Copies elements [p0, p1) of a slice's row (part: its parts' starts) into the chunk-major arrays, one
// wave: an element's place is its part's start plus its index in the part.
// `run_f`, `run_at`: the chunk that is open at p0 and the row index where it
// starts (run_f = -1: none).
template <typename CI, typename V>
GM_DEV void tile_copy_row(const CI *row, const V *val, int64_t p0, int64_t p1, int nc, const uint32_t *part,
                          int64_t n_elems, int run_f, int64_t run_at, uint16_t *out_col, V *out_val) {
    constexpr int U = 4;
    const int lane = threadIdx.x & (GM_WAVE - 1);
    const uint64_t le_mask = lanemask_lt() | (uint64_t(1) << lane);
    for (int64_t b = p0; b < p1; b += GM_WAVE * U) {
        CI c[U];
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = b + u * GM_WAVE + lane;
            c[u] = row[p < p1 ? p : p1 - 1];
            v[u] = val[p < p1 ? p : p1 - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = b + u * GM_WAVE;
            if (q >= p1) break;  // uniform
            const int64_t p = q + lane;
            const bool in = p < p1;
            int64_t f64 = (int64_t)c[u] >> TILE_LOG2;
            const int f = f64 < nc ? (int)f64 : nc - 1;
            const int fp = prev_lane(f, run_f);
            const uint64_t heads = ballot(in && f != fp);
            const uint64_t mine = heads & le_mask;
            const int64_t at = mine ? q + 63 - __clzll((long long)mine) : run_at;
            if (in) {
                const int64_t d = (int64_t)part[f] + (p - at);
                if (d < n_elems) {  // (always, for canonical rows)
                    out_col[d] = (uint16_t)((int64_t)c[u] & (TILE_COLS - 1));
                    out_val[d] = v[u];
                }
            }
            const int last = p1 - q < GM_WAVE ? (int)(p1 - q) - 1 : GM_WAVE - 1;
            run_f = __builtin_amdgcn_readlane(f, last);
            if (heads) run_at = q + 63 - __clzll((long long)heads);
        }
    }
}

constexpr int TF_WAVES = 4;
constexpr int64_t TF_LONG = 2048;  // longer rows are copied in pieces of this many elements, a wave each

// Rows of at most TF_LONG elements, one wave each; of longer ones the pieces
// (slice, first element / TF_LONG) are listed.
// (A work group per 64 consecutive slices, whose parts share lines in every
// chunk: 0.79 instead of 0.64 ms, the rows' lengths being too uneven.)
template <typename CI, typename V>
__global__ __launch_bounds__(TF_WAVES * GM_WAVE) void k_tile_fill(CsrV<CI, V> B, const int32_t *slice_k, int64_t ns,
                                                                  int nc, const uint32_t *part, int64_t n_elems,
                                                                  uint16_t *out_col, V *out_val, int32_t *n_pieces,
                                                                  int2 *pieces) {
    const int64_t nwaves = (int64_t)gridDim.x * TF_WAVES;
    for (int64_t s = blockIdx.x * (int64_t)TF_WAVES + threadIdx.x / GM_WAVE; s < ns; s += nwaves) {
        const int32_t k = slice_k[s];
        const int64_t b0 = B.rp[k], len = B.rp[k + 1] - b0;
        if (len > TF_LONG) {
            const int lane = threadIdx.x & (GM_WAVE - 1), n = (int)((len + TF_LONG - 1) / TF_LONG);
            int at = 0;
            if (lane == 0) at = atomicAdd(n_pieces, n);
            at = __builtin_amdgcn_readfirstlane(at);
            for (int q = lane; q < n; q += GM_WAVE) pieces[at + q] = make_int2((int)s, q);
            continue;
        }
        tile_copy_row<CI, V>(B.ci + b0, B.v + b0, 0, len, nc, part + s * nc, n_elems, -1, 0, out_col, out_val);
    }
}

// The listed pieces, one wave each. (A list of rows, 32 waves a row: 5.5 ms for
// 3.3e4 rows of 3072 elements, two of whose 32 waves had work; so 1.4.)
template <typename CI, typename V>
__global__ __launch_bounds__(TF_WAVES * GM_WAVE) void k_tile_fill_long(CsrV<CI, V> B, const int32_t *slice_k,
                                                                       int64_t ns, int nc, const uint32_t *part,
                                                                       int64_t n_elems, uint16_t *out_col, V *out_val,
                                                                       const int32_t *n_pieces, const int2 *pieces) {
    const int lane = threadIdx.x & (GM_WAVE - 1);
    const int n = *n_pieces, nwaves = (int)gridDim.x * TF_WAVES;
    for (int i = (int)blockIdx.x * TF_WAVES + (int)(threadIdx.x / GM_WAVE); i < n; i += nwaves) {
        const int2 piece = pieces[i];
        const int64_t s = piece.x, p0 = piece.y * TF_LONG;
        const int32_t k = slice_k[s];
        const int64_t b0 = B.rp[k], len = B.rp[k + 1] - b0;
        const CI *row = B.ci + b0;
        // chunk open at p0 and where it starts in the row: 64 bounds a step
        // (a chain of binary search steps took longer than the copy)
        const int64_t f64 = (int64_t)row[p0] >> TILE_LOG2;
        int64_t lo = 0, hi = p0;  // the answer is in [lo, hi]
        while (hi > lo) {
            const int64_t span = hi - lo, x = lo + span * lane / GM_WAVE;
            const uint64_t below = ballot(((int64_t)row[x] >> TILE_LOG2) < f64);
            const int c = __popcll(below);  // (a prefix: the row is sorted)
            if (c == 0) {
                hi = lo;
                break;
            }
            const int64_t nlo = lo + span * (c - 1) / GM_WAVE + 1;
            if (c < GM_WAVE) hi = lo + span * c / GM_WAVE;
            lo = nlo;
        }
        const int64_t p1 = p0 + TF_LONG < len ? p0 + TF_LONG : len;
        tile_copy_row<CI, V>(row, B.v + b0, p0, p1, nc, part + s * nc, n_elems, (int)(f64 < nc ? f64 : nc - 1), lo, out_col,
                             out_val);
    }
}

// ------------------------------------------------------ entries and regions
// The heavy rows' entries in row order. The rows of a work group's entries are
// found once and their starts kept in LDS, so that an entry's row takes no
// search in memory.
constexpr int EN_BLOCK = 256, EN_ITEMS = 8, EN_ROWS = 512;
template <typename CI, typename V>
__global__ __launch_bounds__(EN_BLOCK) void k_tile_entries(CsrV<CI, V> A, const int64_t *heavy_rows, int64_t n_heavy,
                                                           int64_t r0, const int64_t *a_heavy_ptr, int64_t total,
                                                           const int32_t *k_to_slice, int32_t *es, int32_t *eh, V *ea,
                                                           unsigned long long *n_kept) {
    __shared__ int64_t s_ptr[EN_ROWS + 1], s_at[EN_ROWS];
    __shared__ int64_t rows[2];
    __shared__ int32_t sm[EN_BLOCK / GM_WAVE];
    const int64_t e0 = blockIdx.x * (int64_t)(EN_BLOCK * EN_ITEMS);
    const int64_t e1 = e0 + EN_BLOCK * EN_ITEMS < total ? e0 + EN_BLOCK * EN_ITEMS : total;
    if (threadIdx.x == 0) rows[0] = find_row(a_heavy_ptr, 0, n_heavy + 1, e0);
    if (threadIdx.x == GM_WAVE) rows[1] = find_row(a_heavy_ptr, 0, n_heavy + 1, e1 - 1);
    __syncthreads();
    const int64_t ha = rows[0], nr = rows[1] - ha + 1;
    const bool staged = nr <= EN_ROWS;  // uniform
    if (staged) {
        for (int64_t q = threadIdx.x; q <= nr; q += EN_BLOCK) s_ptr[q] = a_heavy_ptr[ha + q];
        for (int64_t q = threadIdx.x; q < nr; q += EN_BLOCK) s_at[q] = A.rp[r0 + heavy_rows[ha + q]];
    }
    __syncthreads();
    int64_t j[EN_ITEMS];
    int32_t h[EN_ITEMS], sl[EN_ITEMS];
    int32_t kept = 0;
#pragma unroll
    for (int u = 0; u < EN_ITEMS; ++u) {
        const int64_t e = e0 + u * EN_BLOCK + threadIdx.x < e1 ? e0 + u * EN_BLOCK + threadIdx.x : e1 - 1;
        if (staged) {
            const int64_t q = find_row(s_ptr, 0, nr + 1, e);
            h[u] = (int32_t)(ha + q);
            j[u] = s_at[q] + (e - s_ptr[q]);
        } else {
            const int64_t hh = find_row(a_heavy_ptr, ha, ha + nr + 1, e);
            h[u] = (int32_t)hh;
            j[u] = A.rp[r0 + heavy_rows[hh]] + (e - a_heavy_ptr[hh]);
        }
    }
    CI k[EN_ITEMS];
    V v[EN_ITEMS];
#pragma unroll
    for (int u = 0; u < EN_ITEMS; ++u) {
        k[u] = A.ci[j[u]];
        v[u] = A.v[j[u]];
    }
#pragma unroll
    for (int u = 0; u < EN_ITEMS; ++u) sl[u] = k_to_slice[(int64_t)k[u]];
#pragma unroll
    for (int u = 0; u < EN_ITEMS; ++u) {
        const int64_t e = e0 + u * EN_BLOCK + threadIdx.x;
        if (e < e1) {
            es[e] = sl[u];
            eh[e] = h[u];
            ea[e] = v[u];
            kept += sl[u] >= 0;
        }
    }
    kept = block_reduce_sum<EN_BLOCK>(kept, sm);
    if (threadIdx.x == 0 && kept) atomicAdd(n_kept, (unsigned long long)kept);
}

// cls[k] = 0 for the B rows that the heavy rows' entries meet and that are not
// empty (the slices), by plain stores of one value (counting each slice's
// entries with atomics, as the slice order needs, takes 0.43 ms for 2e6 entries
// of R-MAT scale 17, whose hub columns stand in most rows).
template <typename CI>
__global__ void k_tile_mark(CsrV<CI, NoV> A, const int64_t *b_rp, const int64_t *heavy_rows, int64_t n_heavy, int64_t r0,
                            const int64_t *a_heavy_ptr, int64_t total, uint8_t *cls) {
    constexpr int U = 8;
    const int64_t e0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) * U;
    if (e0 >= total) return;
    int64_t h = find_row(a_heavy_ptr, 0, n_heavy + 1, e0), h_end = a_heavy_ptr[h + 1];
    int64_t base = A.rp[r0 + heavy_rows[h]] - a_heavy_ptr[h];
    int64_t k[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t e = e0 + u < total ? e0 + u : total - 1;
        while (e >= h_end) {
            ++h;
            h_end = a_heavy_ptr[h + 1];
            base = A.rp[r0 + heavy_rows[h]] - a_heavy_ptr[h];
        }
        k[u] = (int64_t)A.ci[base + e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (cls[k[u]] && b_rp[k[u] + 1] > b_rp[k[u]]) cls[k[u]] = 0;
}

__global__ void k_tile_slices(const int64_t *b_rp, const int64_t *perm, int64_t ns, int32_t *slice_k, int64_t *len,
                              int32_t *k_to_slice) {
    for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < ns; s += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = perm[s];
        slice_k[s] = (int32_t)k;
        len[s] = b_rp[k + 1] - b_rp[k];
        k_to_slice[k] = (int32_t)s;
    }
}

// Places of a region (c, h): its item id is c * nh + h (regions of one chunk
// together, so that concurrent work groups share the chunk's part of B); its
// list of parts is number (c / S * nh + h) * S + c % S (S = 2^slog chunks of a
// row next to each other, so that their lists can be read as one).
GM_DEV int64_t list_of(int64_t c, int64_t h, int64_t nh, int slog) {
    return ((((c >> slog) * nh) + h) << slog) + (c & ((1 << slog) - 1));
}

// Products and non-empty parts of every list (size: parts << 32 | products).
// A work group takes TE_BLOCK consecutive entries, a thread one chunk of a
// contiguous group of them, so the chunk sizes of a slice are read coalesced;
// one atomic per (row, chunk) and group.
constexpr int TE_BLOCK = 256, TE_U = 8, TE_PER = 16;
__global__ __launch_bounds__(TE_BLOCK) void k_tile_sizes(const int32_t *es, const int32_t *eh, int64_t n_ent,
                                                         const uint16_t *cnt, int nc, int ncb, int64_t nh, int slog,
                                                         unsigned long long *size) {
    __shared__ int32_t s_s[TE_BLOCK], s_h[TE_BLOCK];
    const int64_t e0 = blockIdx.x * (int64_t)TE_BLOCK;
    const int ne = (int)(n_ent - e0 < TE_BLOCK ? n_ent - e0 : TE_BLOCK);
    const int tid = threadIdx.x;
    if (tid < ne) {
        s_s[tid] = es[e0 + tid];
        s_h[tid] = eh[e0 + tid];
    }
    __syncthreads();
    // (few chunks: TE_PER entries a thread all the same, for fewer atomics)
    const int per = ncb > TE_PER ? ncb : TE_PER;
    const int i0 = (tid / ncb) * per, i1 = i0 + per < ne ? i0 + per : ne;
    const int c = blockIdx.y * ncb + tid % ncb;
    if (i0 >= i1 || c >= nc) return;
    int cur = s_h[i0];
    uint32_t sum = 0, n = 0;
    auto flush = [&]() {
        if (n) atomicAdd(&size[list_of(c, cur, nh, slog)], ((unsigned long long)n << 32) | sum);
        sum = n = 0;
    };
    for (int i = i0; i < i1; i += TE_U) {
        uint32_t v[TE_U];
#pragma unroll
        for (int u = 0; u < TE_U; ++u) {
            const int q = i + u < i1 ? i + u : i1 - 1;
            const int32_t s = s_s[q];
            v[u] = s >= 0 && i + u < i1 ? cnt[(int64_t)s * nc + c] : 0u;
        }
#pragma unroll
        for (int u = 0; u < TE_U; ++u) {
            if (i + u >= i1) break;
            if (s_h[i + u] != cur) {
                flush();
                cur = s_h[i + u];
            }
            sum += v[u];
            n += v[u] > 0;
        }
    }
    flush();
}

// The lists: seg = (start of the part in the chunk-major B, its length | its
// chunk within the S chunks << 16), seg_e = A entry; cursor[l] starts at list
// l's first place and ends one past its last. Tiles of 64 entries x C
// chunks pass through LDS: read a slice at a time (coalesced), written a
// chunk at a time with an entry per lane, so that a row's parts go out as one
// contiguous store (writing them a thread per chunk, 8 bytes at a time into
// as many lists as threads, took 3.1 ms instead of 1.9 for 1e8 parts).
// C chunks a work group: the smallest of 8, 16, 32, 64 that holds them all, for
// the LDS and the idle lanes that more would take (8 chunks, R-MAT 17 panels:
// 103 -> 76 us a panel in tiles of 8 instead of 64; 256 and 512 chunks: 64 and 32
// measure the same).
constexpr int TL_BLOCK = 256, TL_U = 8;
template <int C>
__global__ __launch_bounds__(TL_BLOCK) void k_tile_lists(const int32_t *es, const int32_t *eh, int64_t n_ent,
                                                         const uint16_t *cnt, const uint32_t *part, int nc, int64_t nh,
                                                         int slog, uint32_t *cursor, uint2 *seg, uint32_t *seg_e) {
    __shared__ uint32_t t_st[GM_WAVE][C + 1];
    __shared__ uint16_t t_len[GM_WAVE][C + 2];
    __shared__ int32_t s_s[GM_WAVE];
    const int tid = threadIdx.x, lane = tid & (GM_WAVE - 1), w = tid / GM_WAVE;
    const int64_t e0 = blockIdx.x * (int64_t)GM_WAVE;
    const int c0 = blockIdx.y * C, ncc = nc - c0 < C ? nc - c0 : C;
    const int64_t e = e0 + lane;
    const int32_t h = e < n_ent ? eh[e] : -1;
    if (w == 0) s_s[lane] = e < n_ent ? es[e] : -1;
    __syncthreads();
    {
        constexpr int RPB = TL_BLOCK / C;  // slices read at a time, RU times
        constexpr int RU = GM_WAVE / RPB < TL_U ? GM_WAVE / RPB : TL_U;
        const int c = tid & (C - 1);
        for (int i0 = tid / C; i0 < GM_WAVE; i0 += RPB * RU) {
            uint32_t len[RU], st[RU];
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                const int32_t s = s_s[i0 + u * RPB];
                const bool ok = s >= 0 && c < ncc;
                len[u] = ok ? cnt[(int64_t)s * nc + c0 + c] : 0u;
                st[u] = ok ? part[(int64_t)s * nc + c0 + c] : 0u;
            }
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                t_len[i0 + u * RPB][c] = (uint16_t)len[u];
                t_st[i0 + u * RPB][c] = st[u];
            }
        }
    }
    __syncthreads();
    const uint64_t le_mask = lanemask_lt() | (uint64_t(1) << lane);
    const int32_t hp = prev_lane(h, -2);
    const uint64_t heads = ballot(h != hp);  // lane 0 always starts a run
    const int first = 63 - __clzll((long long)(heads & le_mask));
    const uint64_t above = heads & ~le_mask;
    const int end = above ? __ffsll((long long)above) - 1 : GM_WAVE;  // lane after the run
    const uint64_t run = (end == GM_WAVE ? ~0ull : (uint64_t(1) << end) - 1) & ~((uint64_t(1) << first) - 1);
    constexpr int NW = TL_BLOCK / GM_WAVE, CU = C / NW < TL_U ? C / NW : TL_U;
    // CU chunks at a time: their reservations are in flight together
    for (int cb = w; cb < ncc; cb += CU * NW) {
        uint32_t len[CU], at[CU];
        uint64_t full[CU];
#pragma unroll
        for (int u = 0; u < CU; ++u) {
            const int c = cb + u * NW;
            len[u] = c < ncc ? t_len[lane][c] : 0u;
            full[u] = ballot(len[u] > 0) & run;
            at[u] = 0;
            if (lane == first && full[u])
                at[u] = atomicAdd(&cursor[list_of(c0 + c, h, nh, slog)], (uint32_t)__popcll(full[u]));
        }
#pragma unroll
        for (int u = 0; u < CU; ++u) {
            const int c = cb + u * NW;
            const uint32_t q = (uint32_t)__shfl((int32_t)at[u], first, GM_WAVE) +
                               (uint32_t)__popcll(full[u] & lanemask_lt());
            if (len[u] > 0) {
                seg[q] = make_uint2(t_st[lane][c], len[u] | (uint32_t)((c0 + c) & ((1 << slog) - 1)) << 16);
                seg_e[q] = (uint32_t)e;
            }
        }
    }
}

// Regions, bins and list lengths. The S chunks of a row are cut into aligned
// groups of a power of two of chunks that hold at most TILE_MERGE products
// together (one region each, at the group's first chunk; grp = its chunks), so
// that sparse rows make few regions; chunks above that stay alone.
template <int S>
__global__ void k_tile_classes(const unsigned long long *size, int64_t nh, int64_t n_lists, uint8_t *cls, uint8_t *grp,
                               uint32_t *list_len) {
    for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n_lists / S;
         g += (int64_t)gridDim.x * blockDim.x) {
        uint32_t sum[S];
        uint8_t len[S];
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const unsigned long long x = size[g * S + q];
            sum[q] = (uint32_t)x;
            len[q] = 1;
            list_len[g * S + q] = (uint32_t)(x >> 32);
        }
#pragma unroll
        for (int w = 2; w <= S; w *= 2)
#pragma unroll
            for (int q = 0; q < S; q += w) {
                // (a sum that passed TILE_MERGE is never merged further)
                const uint32_t a = sum[q], b = sum[q + w / 2];
                if (len[q] == w / 2 && len[q + w / 2] == w / 2 && a <= (uint32_t)TILE_MERGE &&
                    b <= (uint32_t)TILE_MERGE && a + b <= (uint32_t)TILE_MERGE) {
                    sum[q] = a + b;
                    sum[q + w / 2] = 0;
                    len[q] = (uint8_t)w;
                    len[q + w / 2] = 0;
                }
            }
        const int64_t C = g / nh, h = g - C * nh;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const uint32_t z = sum[q];
            const int64_t i = (C * S + q) * nh + h;
            grp[i] = len[q];
            cls[i] = z == 0             ? TILE_EMPTY
                     : z <= TILE_T_MAX  ? TILE_T
                     : z <= TILE_S_MAX  ? TILE_S
                     : z <= TILE_MERGE  ? TILE_L
                     : z <= TILE_M_MAX  ? TILE_M
                     : z <= TILE_D_MAX  ? TILE_D
                                        : TILE_D_BIG;
        }
    }
}

__global__ void k_tile_total(const uint32_t *v, int64_t *out) { *out = (int64_t)*v; }

// ------------------------------------------------------------- accumulation
// What a region's kernel reads. The regions' records are built in launch
// order beforehand, so that a region starts from one load instead of a chain
// (id -> chunks -> list ends -> parts); with the scales loaded beside the parts
// the small regions' numeric kernels went from 1.92 to 1.70 ms for a panel of
// 2e9 R-MAT 22 products and from 6.9 to 6.0 for 1.5e9 of R-MAT 23.
template <typename V>
struct TileArgs {
    const uint16_t *col;
    const V *val;
    const uint2 *seg;          // the regions' parts: start, length | chunk within its S chunks << 16
    const uint32_t *seg_e;     // A entry of a part
    const V *ea;
    const TileTask *tasks;     // the bin's regions
    int64_t n;
    uint32_t *bitmap;          // TWORDS words per region of more than TILE_MERGE products
};

// Records of the regions items[0 .. n) (ids c * nh + h): symbolic.
__global__ void k_tile_tasks_sym(const int64_t *items, int64_t n, const uint8_t *grp, const uint32_t *seg_end,
                                 int64_t nh, int64_t ncp, int slog, TileTask *tasks) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t id = items[i], c = id / nh, h = id - c * nh;
        const int64_t l = list_of(c, h, nh, slog);
        TileTask t;
        t.id = id;
        t.out = h * ncp + c;
        t.q0 = l > 0 ? seg_end[l - 1] : 0u;
        t.q1 = seg_end[l + grp[id] - 1];
        t.c = (int32_t)c;
        t.want = 0;
        t.at = (uint32_t)i;
        t.sub0 = (uint16_t)(c & ((1 << slog) - 1));
        t.chunks = grp[id];
        tasks[i] = t;
    }
}

// ... numeric: the place in C and the distinct columns, the first n_large
// regions in the order of `perm` (by distinct columns).
__global__ void k_tile_tasks_num(const TileTask *sym, int64_t n, const int64_t *perm, int64_t n_large, int64_t nh,
                                 const uint32_t *nnz, const int64_t *slot, const int64_t *heavy_rows,
                                 const int64_t *c_row_ptr, TileTask *tasks) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        TileTask t = sym[i < n_large ? perm[i] : i];
        const int64_t h = t.id - (int64_t)t.c * nh;
        t.want = nnz[t.id];
        t.out = c_row_ptr[heavy_rows[h]] + slot[t.out];
        tasks[i] = t;
    }
}

// Numeric bin of the large regions by distinct columns.
__global__ void k_tile_large_classes(const TileTask *sym, int64_t n, const uint32_t *nnz, uint8_t *cls) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t z = nnz[sym[i].id];
        cls[i] = z > TILE_RANK_MAX ? 0 : z > TILE_RANK_MID ? 1 : z > TILE_RANK_MIN ? 2 : 3;
    }
}

// Calls f(column, product) for the parts held one per lane (start
// `st`, `len` elements, scale `a`; the lanes past the last part hold len = 0),
// in windows of TWIN products. A product's part is the number of parts that
// end before it: the parts' last products are marked in `ends` (one bit per
// product of the window) and counted below the lane.
constexpr int TENDS = TWIN / 32;
template <bool NUM, typename V, class F>
GM_DEV void wave_parts(const uint16_t *col, const V *val, uint32_t st, uint32_t len, V a, uint32_t *ends, F &&f) {
    const int lane = threadIdx.x & (GM_WAVE - 1);
    const uint32_t inc = wave_incl_scan<uint32_t>(len);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, GM_WAVE - 1);
    const uint32_t rel = st - (inc - len);
    const uint32_t st0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)st);
    uint32_t ended = 0;  // parts that end before the window
    for (uint32_t w0 = 0; w0 < total; w0 += TWIN) {
        if (lane < TENDS) ends[lane] = 0u;
        wave_lds_fence();
        const uint32_t d = inc - 1 - w0;
        if (d < (uint32_t)TWIN)
            __hip_atomic_fetch_or(&ends[d >> 5], 1u << (d & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        wave_lds_fence();
        uint32_t own[TU], pos[TU];
#pragma unroll
        for (int u = 0; u < TU; ++u) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)ends[2 * u]);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)ends[2 * u + 1]);
            own[u] = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, ended));
            ended += (uint32_t)(__popc(lo) + __popc(hi));
            const uint32_t t = w0 + u * GM_WAVE + lane;
            const uint32_t p = (uint32_t)__shfl((int)rel, (int)own[u], GM_WAVE) + t;
            pos[u] = t < total ? p : st0;
        }
        uint32_t c[TU];
        V v[TU];
#pragma unroll
        for (int u = 0; u < TU; ++u) {
            c[u] = col[pos[u]];
            if (NUM) v[u] = val[pos[u]];
        }
#pragma unroll
        for (int u = 0; u < TU; ++u) {
            V p = (V)0;
            if (NUM) p = __shfl(a, (int)own[u], GM_WAVE) * v[u];
            const uint32_t t = w0 + u * GM_WAVE + lane;
            if (t < total) f(c[u], p);
        }
    }
}

// Shared list of the tails of a region's long parts.
template <typename V>
struct LongParts {
    int32_t n;
    uint32_t st[TLONG_CAP], len[TLONG_CAP];
    V a[TLONG_CAP];
};

// Calls f(column, product) for all products of a region of one chunk, for a
// work group of NW waves: wave w takes parts w, w + NW, ... (the longest B
// rows sit next to each other in a row's entries); what a part holds past
// TLONG elements goes to the list, whose windows the waves then share. Called
// by every thread; the list must be empty (n = 0) and a barrier behind it;
// ends without a barrier.
template <int NW, bool NUM, typename V, class F>
GM_DEV void tile_products(const TileArgs<V> &t, const TileTask &g, uint32_t *ends, LongParts<V> *lp, F &&f) {
    const int lane = threadIdx.x & (GM_WAVE - 1);
    const uint32_t w = threadIdx.x / GM_WAVE;
    for (uint32_t jb = g.q0 + w; jb < g.q1; jb += GM_WAVE * NW) {
        const uint32_t q = jb + lane * NW;
        uint32_t st = 0, len = 0;
        V a = (V)0;
        if (q < g.q1) {
            const uint2 sg = t.seg[q];
            st = sg.x;
            len = sg.y & 0xffffu;
            if (NUM) a = t.ea[t.seg_e[q]];
        }
        if (len > TLONG) {
            const int i = atomicAdd(&lp->n, 1);
            if (i < TLONG_CAP) {
                lp->st[i] = st + TLONG;
                lp->len[i] = len - TLONG;
                if (NUM) lp->a[i] = a;
                len = TLONG;
            }
        }
        wave_parts<NUM>(t.col, t.val, st, len, a, ends, f);
    }
    __syncthreads();
    const int n = lp->n < TLONG_CAP ? lp->n : TLONG_CAP;
    uint32_t k = w;  // next window of this wave, counted over the listed parts
    for (int i = 0; i < n; ++i) {
        const uint32_t st = lp->st[i], len = lp->len[i];
        const V a = NUM ? lp->a[i] : (V)0;
        const uint32_t nwin = (len + TWIN - 1) / TWIN;
        for (; k < nwin; k += NW) {
            uint32_t cc[TU];
            V v[TU];
#pragma unroll
            for (int u = 0; u < TU; ++u) {
                const uint32_t x = k * TWIN + u * GM_WAVE + lane;
                const uint32_t p = st + (x < len ? x : len - 1);
                cc[u] = t.col[p];
                if (NUM) v[u] = t.val[p];
            }
#pragma unroll
            for (int u = 0; u < TU; ++u)
                if (k * TWIN + u * GM_WAVE + lane < len) f(cc[u], NUM ? (V)(a * v[u]) : (V)0);
        }
        k -= nwin;
    }
}

GM_DEV void bit_or(uint32_t *bits, uint32_t c) {
    __hip_atomic_fetch_or(&bits[c >> 5], 1u << (c & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Regions of at most TILE_MERGE products (rank.hpp): the parts come from the
// lists, their columns relative to the region's first chunk.
template <typename V>
struct TileParts {
    typedef uint32_t Pos;
    typedef uint32_t Col;
    const TileArgs<V> &t;
    const TileTask &g;
    GM_DEV int64_t np() const { return g.q1 - g.q0; }
    GM_DEV uint32_t part(int64_t q, int64_t *st, uint32_t *aux) const {
        const uint2 sg = t.seg[g.q0 + q];
        *st = sg.x;
        *aux = ((sg.y >> 16) - (uint32_t)g.sub0) << TILE_LOG2;
        return sg.y & 0xffffu;
    }
    GM_DEV V scale(int64_t q) const { return t.ea[t.seg_e[g.q0 + q]]; }
    GM_DEV RankWord pack(int64_t st, uint32_t off, uint32_t aux) const { return RankWord{(uint32_t)st - off, aux}; }
    GM_DEV Pos at(const RankWord &p, uint32_t x, uint32_t *col) const {
        *col = p.rank;
        return p.bits + x;
    }
    GM_DEV Col col(Pos p) const { return t.col[p]; }
    GM_DEV V val(Pos p) const { return t.val[p]; }
    GM_DEV uint32_t local(Col c) const { return c; }
};

// Symbolic of small regions.
template <int BLOCK, int CAP, int REGS>
__global__ __launch_bounds__(BLOCK * REGS) void k_tile_sym_small(TileArgs<float> t, uint32_t *nnz,
                                                                 int64_t *slot) {
    static_assert(REGS == 1 || BLOCK == GM_WAVE, "several regions per work group are one wave each");
    __shared__ __align__(16) RankLds<BLOCK, CAP, false, float> L[REGS];
    const int reg = REGS > 1 ? threadIdx.x / GM_WAVE : 0, tid = REGS > 1 ? threadIdx.x & (GM_WAVE - 1) : threadIdx.x;
    const int64_t i = blockIdx.x * (int64_t)REGS + reg;
    if (i >= t.n) return;  // the whole wave (one region: the whole work group)
    const TileTask g = t.tasks[i];
    const uint32_t n = rank_region<BLOCK, CAP, false, float>(TileParts<float>{t, g}, (uint32_t)g.chunks << TILE_LOG2, L[reg],
                                                             tid, [](uint32_t, uint32_t) {});
    if (tid == 0) {
        nnz[g.id] = (uint32_t)n;
        slot[g.out] = n;
    }
}

// Symbolic, one work group per region; the bitmap is kept for the numeric phase.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_tile_sym(TileArgs<float> t, uint32_t *nnz, int64_t *slot) {
    constexpr int NW = BLOCK / GM_WAVE;
    __shared__ __align__(16) uint32_t bits[TWORDS];
    __shared__ __align__(16) uint32_t ends[NW][TENDS];
    __shared__ LongParts<float> lp;
    __shared__ int32_t scan[NW];
    for (int q = threadIdx.x; q < TWORDS; q += BLOCK) bits[q] = 0;
    if (threadIdx.x == 0) lp.n = 0;
    const TileTask g = t.tasks[blockIdx.x];
    __syncthreads();
    tile_products<NW, false, float>(t, g, ends[threadIdx.x / GM_WAVE], &lp,
                                    [&](uint32_t c, float) {
                                        // (most products of a large region meet a column already marked, and
                                        // atomics of several lanes on one word take turns)
                                        if (!(lds_peek(&bits[c >> 5]) & (1u << (c & 31)))) bit_or(bits, c);
                                    });
    __syncthreads();
    int32_t n = 0;
    uint32_t *bm = t.bitmap + g.at * (int64_t)TWORDS;
    for (int q = threadIdx.x; q < TWORDS; q += BLOCK) {
        const uint32_t x = bits[q];
        bm[q] = x;
        n += __popc(x);
    }
    n = block_reduce_sum<BLOCK>(n, scan);
    if (threadIdx.x == 0) {
        nnz[g.id] = (uint32_t)n;
        slot[g.out] = n;
    }
}

// C's arrays.
template <typename CI, typename V>
struct TileOut {
    CI *c_col;
    V *c_val;
    int32_t *err;
    GM_DEV CI base(const TileTask &g) const { return (CI)g.c << TILE_LOG2; }
};

// Numeric of small regions.
template <int BLOCK, int CAP, int REGS, typename CI, typename V>
__global__ __launch_bounds__(BLOCK * REGS) void k_tile_num_small(TileArgs<V> t, TileOut<CI, V> o) {
    static_assert(REGS == 1 || BLOCK == GM_WAVE, "several regions per work group are one wave each");
    __shared__ __align__(16) RankLds<BLOCK, CAP, true, V> L_all[REGS];
    const int reg = REGS > 1 ? threadIdx.x / GM_WAVE : 0, tid = REGS > 1 ? threadIdx.x & (GM_WAVE - 1) : threadIdx.x;
    const int64_t i = blockIdx.x * (int64_t)REGS + reg;
    if (i >= t.n) return;  // the whole wave (one region: the whole work group)
    const TileTask g = t.tasks[i];
    RankLds<BLOCK, CAP, true, V> &L = L_all[reg];
    const int want = (int)g.want;
    const int64_t dst = g.out;
    const CI cb = o.base(g);
    const int total = (int)rank_region<BLOCK, CAP, true, V>(TileParts<V>{t, g}, (uint32_t)g.chunks << TILE_LOG2, L, tid,
                                                            [&](uint32_t rk, uint32_t c) {
                                                                if ((int)rk < want) o.c_col[dst + rk] = cb + (CI)c;
                                                            });
    if (tid == 0 && total != want) atomicOr(o.err, 4);
    const int m = total < want ? total : want;
    for (int q = tid; q < m; q += BLOCK) o.c_val[dst + q] = L.vals[q];
}

// Adds v at its column's rank.
template <int CAP, typename V>
GM_DEV void rank_add(const RankWord *words, V *vals, uint32_t col, V v) {
    const uint32_t rk = rank_of(words[col >> 5], col & 31);
    if (rk < (uint32_t)CAP) __hip_atomic_fetch_add(&vals[rk], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// cols[rank] = column for the present columns of words [w0, w0 + n)
template <int CAP>
GM_DEV void rank_columns(const RankWord *words, uint16_t *cols, int w0, int n) {
    for (int wd = w0; wd < w0 + n; ++wd) {
        const RankWord x = words[wd];
        uint32_t b = x.bits, rk = x.rank;
        while (b) {
            if (rk < (uint32_t)CAP) cols[rk] = (uint16_t)(wd * 32 + __ffs((int)b) - 1);
            b &= b - 1;
            ++rk;
        }
    }
}

// Numeric of larger regions of at most CAP distinct columns: the ranks come
// from the bitmap the symbolic phase kept, so the products are read once. One
// launch per size of the value array, so that a small one leaves room for
// more work groups on a CU. (Panel of 2e9 R-MAT 22 products, these launches
// and the dense one: 6.65 ms with 1024 threads for all regions of more than
// 4096 products, each kernel leaving the other's regions at once; 5.58 ms with
// the regions sorted into the four launches.)
template <int BLOCK, int CAP, typename CI, typename V>
__global__ __launch_bounds__(BLOCK) void k_tile_num_rank(TileArgs<V> t, TileOut<CI, V> o) {
    constexpr int NW = BLOCK / GM_WAVE, WPT = TWORDS > BLOCK ? TWORDS / BLOCK : 1;
    static_assert(WPT == 1 || WPT * BLOCK == TWORDS, "bitmap words per thread");
    __shared__ __align__(16) RankWord words[TWORDS];
    __shared__ __align__(16) V vals[CAP];
    __shared__ __align__(16) uint32_t ends[NW][TENDS];
    __shared__ LongParts<V> lp;
    __shared__ int32_t scan[NW];
    const int tid = threadIdx.x, w0 = tid * WPT;
    const TileTask g = t.tasks[blockIdx.x];
    const int want = (int)g.want;
    if (want > CAP) return;  // (uniform; such regions are in another bin)
    uint32_t bw[WPT];
    int32_t cnt = 0;
#pragma unroll
    for (int q = 0; q < WPT; ++q) {
        bw[q] = w0 + q < TWORDS ? t.bitmap[g.at * (int64_t)TWORDS + w0 + q] : 0u;
        cnt += __popc(bw[q]);
    }
    for (int q = tid; q < want; q += BLOCK) vals[q] = (V)0;
    if (tid == 0) lp.n = 0;
    int32_t total;
    uint32_t rank = (uint32_t)block_excl_scan<BLOCK>(cnt, scan, &total);
#pragma unroll
    for (int q = 0; q < WPT; ++q)
        if (w0 + q < TWORDS) {
            words[w0 + q] = RankWord{bw[q], rank};
            rank += (uint32_t)__popc(bw[q]);
        }
    __syncthreads();
    tile_products<NW, true, V>(t, g, ends[tid / GM_WAVE], &lp,
                               [&](uint32_t c, V v) { rank_add<CAP>(words, vals, c, v); });
    __syncthreads();
    if (tid == 0 && total != want) atomicOr(o.err, 4);
    const int m = total < want ? total : want;
    const CI cb = o.base(g);
    const int64_t dst = g.out;
    for (int q = tid; q < m; q += BLOCK) o.c_val[dst + q] = vals[q];
    __syncthreads();  // the values' place is reused for the columns
    uint16_t *cols = (uint16_t *)vals;
    if (w0 < TWORDS) rank_columns<CAP>(words, cols, w0, WPT);
    __syncthreads();
    for (int q = tid; q < m; q += BLOCK) o.c_col[dst + q] = cb + (CI)cols[q];
}

// Numeric of regions of more than TILE_RANK_MAX distinct columns: one value per
// column of the chunk.
template <int BLOCK, typename CI, typename V>
__global__ __launch_bounds__(BLOCK) void k_tile_num_dense(TileArgs<V> t, TileOut<CI, V> o) {
    constexpr int NW = BLOCK / GM_WAVE;
    constexpr int SPAN = TILE_COLS / NW;  // columns a wave writes out
    __shared__ __align__(16) V vals[TILE_COLS];
    __shared__ __align__(16) uint32_t bits[TWORDS];
    __shared__ __align__(16) uint32_t ends[NW][TENDS];
    __shared__ LongParts<V> lp;
    __shared__ int32_t scan[NW];
    const int tid = threadIdx.x, lane = tid & (GM_WAVE - 1), w = tid / GM_WAVE;
    const TileTask g = t.tasks[blockIdx.x];
    const int want = (int)g.want;
    static_assert(BLOCK >= TWORDS, "one bitmap word per thread");
    if (tid < TWORDS) bits[tid] = t.bitmap[g.at * (int64_t)TWORDS + tid];
    for (int q = tid; q < TILE_COLS; q += BLOCK) vals[q] = (V)0;
    if (tid == 0) lp.n = 0;
    __syncthreads();
    tile_products<NW, true, V>(t, g, ends[w], &lp, [&](uint32_t c, V v) {
        __hip_atomic_fetch_add(&vals[c], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    });
    __syncthreads();
    // present columns in order: wave w owns columns [w * SPAN, w * SPAN + SPAN)
    static_assert(SPAN % GM_WAVE == 0 && SPAN / 32 <= GM_WAVE, "a wave's columns in whole ballots");
    int32_t cnt = lane < SPAN / 32 ? __popc(bits[w * (SPAN / 32) + lane]) : 0;
    cnt = wave_reduce_sum<int32_t>(cnt);
    int32_t total;
    int32_t at = block_excl_scan<BLOCK>(lane == 0 ? cnt : 0, scan, &total);
    at = __builtin_amdgcn_readfirstlane(at);
    if (tid == 0 && total != want) atomicOr(o.err, 2);
    const CI cb = o.base(g);
    const int64_t dst = g.out;
    for (int x0 = 0; x0 < SPAN; x0 += GM_WAVE) {
        const int x = w * SPAN + x0 + lane;
        const bool p = (bits[x >> 5] >> (x & 31)) & 1u;
        const uint64_t m = ballot(p);
        const int pos = at + __popcll(m & lanemask_lt());
        if (p && pos < want) {
            o.c_col[dst + pos] = cb + (CI)x;
            o.c_val[dst + pos] = vals[x];
        }
        at += __popcll(m);
    }
}

// Regions of at most TILE_RANK_MID distinct columns take small work groups, of
// which many share a CU. When all of them fit the chip as 16-wave groups (two a
// CU on 256 CUs), each takes all those waves instead: whole products of 64 rows,
// 2.3e6 products and 2048 columns each, 3.70 -> 1.80 ms, of 16 rows of 2.2e7
// products 35.5 -> 16.3; of 500 rows of 3600 products the same either way.
constexpr int64_t RANK_FEW = 512;

template <class K, class... Args>
void launch_regions(K kernel, int block, int64_t groups, hipStream_t s, Args... args) {
    if (groups <= 0) return;
    // (cannot happen below 2^32 products, which the rule admits)
    GM_REQUIRE(groups * block < (int64_t)1 << 32, GMAGNUS_ERROR_UNSUPPORTED, "too many regions for one launch");
    hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(block), 0, s, args...);
    GM_CHECK_LAUNCH();
}

template <typename V>
TileArgs<V> tile_args(const TileHeavy &t, const TileTask *tasks, int64_t b0, int64_t b1) {
    return TileArgs<V>{t.col,       static_cast<const V *>(t.val), t.seg,  t.seg_e, static_cast<const V *>(t.ea),
                       tasks + b0, b1 - b0,                        t.bitmap};
}

void scan_u32(uint32_t *a, int64_t n, uint32_t *scratch, hipStream_t s) {
    const int64_t tiles = (n + SC_TILE - 1) / SC_TILE;
    hipLaunchKernelGGL(k_tile_scan_sums, dim3((unsigned)tiles), dim3(SC_BLOCK), 0, s, a, n, scratch);
    GM_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_tile_scan_mid, dim3(1), dim3(1024), 0, s, scratch, tiles);
    GM_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_tile_scan_apply, dim3((unsigned)tiles), dim3(SC_BLOCK), 0, s, a, n, scratch);
    GM_CHECK_LAUNCH();
}

}  // namespace

int tile_chunks(int64_t c_m) { return (int)std::min<int64_t>((c_m + TILE_COLS - 1) / TILE_COLS, 1 << 20); }

void tile_parts(const Csr &B, const int32_t *slice_k, const TileHeavy &t, uint32_t *cm, hipStream_t s) {
    if (t.ns <= 0) return;
    with_index_type(B.ci64, [&](auto ci) {
        using CI = decltype(ci);
        hipLaunchKernelGGL(k_tile_row_counts<CI>, dim3(grid_for(t.ns, TR_WAVES, 65536)), dim3(TR_WAVES * GM_WAVE),
                           TR_WAVES * (t.nc + 1) * sizeof(uint32_t), s, typed<CI, NoV>(B), slice_k, t.ns, t.nc, t.cnt);
        GM_CHECK_LAUNCH();
    });
    // starts of the parts: the counts chunk-major, scanned, back beside the slices
    const int64_t tiles = ((t.ns + TT - 1) / TT) * ((t.nc + TT - 1) / TT);
    GM_REQUIRE(tiles < (int64_t)1 << 31, GMAGNUS_ERROR_UNSUPPORTED, "too many slices");
    hipLaunchKernelGGL(k_tile_transpose<uint16_t>, dim3((unsigned)tiles), dim3(256), 0, s, t.cnt, t.ns, (int64_t)t.nc, cm);
    GM_CHECK_LAUNCH();
    scan_u32(cm, t.ns * t.nc, t.scan, s);
    hipLaunchKernelGGL(k_tile_transpose<uint32_t>, dim3((unsigned)tiles), dim3(256), 0, s, cm, (int64_t)t.nc, t.ns, t.part);
    GM_CHECK_LAUNCH();
}

int64_t tile_scan_words(int64_t n) { return (n + SC_TILE - 1) / SC_TILE + 1; }

// The rows in pieces hold more than TF_LONG elements each: fewer than twice as many pieces as whole TF_LONGs.
int64_t tile_most_pieces(int64_t n_elems) { return n_elems > TF_LONG ? 2 * (n_elems / TF_LONG) + 1 : 0; }
int64_t tile_piece_words(int64_t n_elems) { return 2 + 2 * tile_most_pieces(n_elems); }

void tile_fill(const Csr &B, const int32_t *slice_k, const TileHeavy &t, int32_t *piece_words, hipStream_t s) {
    if (t.ns <= 0) return;
    int2 *pieces = reinterpret_cast<int2 *>(piece_words + 2);
    fill<int32_t>(piece_words, 0, 1, s);
    with_types(B, [&](auto ci, auto v) {
        using CI = decltype(ci);
        using V = decltype(v);
        V *ov = static_cast<V *>(t.val);
        hipLaunchKernelGGL((k_tile_fill<CI, V>), dim3(grid_for(t.ns, TF_WAVES, 65536)), dim3(TF_WAVES * GM_WAVE), 0, s,
                           typed<CI, V>(B), slice_k, t.ns, t.nc, t.part, t.n_elems, t.col, ov, piece_words, pieces);
        GM_CHECK_LAUNCH();
        const int64_t most = tile_most_pieces(t.n_elems);
        if (most == 0) return;
        hipLaunchKernelGGL((k_tile_fill_long<CI, V>), dim3(grid_for(most, TF_WAVES, 16384)), dim3(TF_WAVES * GM_WAVE), 0,
                           s, typed<CI, V>(B), slice_k, t.ns, t.nc, t.part, t.n_elems, t.col, ov, piece_words, pieces);
        GM_CHECK_LAUNCH();
    });
}

void tile_entries(const Csr &A, const int64_t *heavy_rows, int64_t r0, const int32_t *k_to_slice, const TileHeavy &t,
                  unsigned long long *n_kept, hipStream_t s) {
    if (t.n_ent <= 0) return;
    with_types(A, [&](auto ci, auto v) {
        using CI = decltype(ci);
        using V = decltype(v);
        hipLaunchKernelGGL((k_tile_entries<CI, V>), dim3(grid_for(t.n_ent, EN_BLOCK * EN_ITEMS, INT32_MAX)),
                           dim3(EN_BLOCK), 0, s, typed<CI, V>(A), heavy_rows, t.nh, r0, t.a_ptr, t.n_ent, k_to_slice,
                           t.es, t.eh, static_cast<V *>(t.ea), n_kept);
        GM_CHECK_LAUNCH();
    });
}

void tile_mark(const Csr &A, const Csr &B, const int64_t *heavy_rows, int64_t n_heavy, int64_t r0,
               const int64_t *a_heavy_ptr, int64_t total, uint8_t *cls, hipStream_t s) {
    fill<uint8_t>(cls, 1, A.n_cols, s);
    if (total <= 0) return;
    with_index_type(A.ci64, [&](auto ci) {
        using CI = decltype(ci);
        hipLaunchKernelGGL(k_tile_mark<CI>, dim3(grid_for((total + 7) / 8, 256, (int64_t)1 << 30)), dim3(256), 0, s,
                           typed<CI, NoV>(A), B.rp, heavy_rows, n_heavy, r0, a_heavy_ptr, total, cls);
        GM_CHECK_LAUNCH();
    });
}

void tile_slices(const Csr &B, const int64_t *perm, int64_t ns, int32_t *slice_k, int64_t *len, int32_t *k_to_slice,
                 hipStream_t s) {
    fill<int32_t>(k_to_slice, -1, B.n_rows, s);
    if (ns <= 0) return;
    hipLaunchKernelGGL(k_tile_slices, dim3(grid_for(ns, 256, 16384)), dim3(256), 0, s, B.rp, perm, ns, slice_k, len,
                       k_to_slice);
    GM_CHECK_LAUNCH();
}

void tile_regions(const TileHeavy &t, unsigned long long *size, uint8_t *cls, int64_t *n_seg, hipStream_t s) {
    const int64_t n = t.nh * t.ncp;
    fill<unsigned long long>(size, 0ull, n, s);
    const int ncb = (int)std::min<int64_t>(ceil_pow2(t.nc), TE_BLOCK);
    hipLaunchKernelGGL(k_tile_sizes, dim3((unsigned)((t.n_ent + TE_BLOCK - 1) / TE_BLOCK), (unsigned)((t.nc + ncb - 1) / ncb)),
                       dim3(TE_BLOCK), 0, s, t.es, t.eh, t.n_ent, t.cnt, t.nc, ncb, t.nh, t.slog, size);
    GM_CHECK_LAUNCH();
    auto classes = [&](auto S) {
        hipLaunchKernelGGL(k_tile_classes<decltype(S)::value>, dim3(grid_for(n / decltype(S)::value, 256, 65536)), dim3(256),
                           0, s, size, t.nh, n, cls, t.grp, t.seg_end);
        GM_CHECK_LAUNCH();
    };
    switch (t.slog) {
    case 0: classes(std::integral_constant<int, 1>()); break;
    case 1: classes(std::integral_constant<int, 2>()); break;
    case 2: classes(std::integral_constant<int, 4>()); break;
    case 3: classes(std::integral_constant<int, 8>()); break;
    default: classes(std::integral_constant<int, 16>()); break;
    }
    scan_u32(t.seg_end, n, t.scan, s);
    hipLaunchKernelGGL(k_tile_total, dim3(1), dim3(1), 0, s, t.seg_end + n, n_seg);
    GM_CHECK_LAUNCH();
}

void tile_segments(const TileHeavy &t, hipStream_t s) {
    auto launch = [&](auto kernel, int c) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((t.n_ent + GM_WAVE - 1) / GM_WAVE), (unsigned)((t.nc + c - 1) / c)),
                           dim3(TL_BLOCK), 0, s, t.es, t.eh, t.n_ent, t.cnt, t.part, t.nc, t.nh, t.slog, t.seg_end,
                           t.seg, t.seg_e);
    };
    if (t.nc <= 8)
        launch(k_tile_lists<8>, 8);
    else if (t.nc <= 16)
        launch(k_tile_lists<16>, 16);
    else if (t.nc <= 32)
        launch(k_tile_lists<32>, 32);
    else
        launch(k_tile_lists<64>, 64);
    GM_CHECK_LAUNCH();
}

void tile_tasks(const TileHeavy &t, hipStream_t s) {
    const int64_t n = tile_items(t);
    if (n <= 0) return;
    hipLaunchKernelGGL(k_tile_tasks_sym, dim3(grid_for(n, 256, 65536)), dim3(256), 0, s, t.items + t.bins[TILE_EMPTY + 1], n,
                       t.grp, t.seg_end, t.nh, t.ncp, t.slog, t.tasks);
    GM_CHECK_LAUNCH();
}

// (the tasks hold the bins after TILE_EMPTY)
void tile_symbolic(const TileHeavy &t, int bin, int64_t *slot, hipStream_t s) {
    const int64_t first = t.bins[TILE_EMPTY + 1];
    const TileArgs<float> a = tile_args<float>(t, t.tasks, t.bins[bin] - first, t.bins[bin + 1] - first);
    const int64_t n = a.n;
    if (n <= 0) return;
    switch (bin) {
    case TILE_T: launch_regions(k_tile_sym_small<64, TILE_T_MAX, 4>, 256, (n + 3) / 4, s, a, t.nnz, slot); break;
    case TILE_S: launch_regions(k_tile_sym_small<256, TILE_S_MAX, 1>, 256, n, s, a, t.nnz, slot); break;
    case TILE_L: launch_regions(k_tile_sym_small<512, TILE_MERGE, 1>, 512, n, s, a, t.nnz, slot); break;
    case TILE_M: launch_regions(k_tile_sym<256>, 256, n, s, a, t.nnz, slot); break;
    case TILE_D: launch_regions(k_tile_sym<512>, 512, n, s, a, t.nnz, slot); break;
    case TILE_D_BIG: launch_regions(k_tile_sym<1024>, 1024, n, s, a, t.nnz, slot); break;
    default: break;
    }
}

// Orders the regions of more than TILE_MERGE products by numeric bin:
// large_bins (device) gets the bounds of the dense, large, middle and small
// rank regions, which t.large_perm lists.
void tile_large_bins(const TileHeavy &t, uint8_t *cls, int64_t *scratch, int64_t *large_bins, hipStream_t s) {
    const int64_t n = tile_large(t);
    if (n > 0) {
        hipLaunchKernelGGL(k_tile_large_classes, dim3(grid_for(n, 256, 65536)), dim3(256), 0, s, t.tasks, n, t.nnz, cls);
        GM_CHECK_LAUNCH();
    }
    partition_u8(cls, n, 4, t.large_perm, nullptr, large_bins, scratch, s);
}

int64_t tile_items(const TileHeavy &t) { return t.bins[TILE_NBINS] - t.bins[TILE_EMPTY + 1]; }
int64_t tile_large(const TileHeavy &t) { return t.bins[TILE_M + 1] - t.bins[TILE_D_BIG]; }

int tile_numeric(const TileHeavy &t, const int64_t *large_bins, TileTask *tasks, const int64_t *heavy_rows,
                 const int64_t *c_row_ptr, const int64_t *slot, bool ci64, bool v32, void *c_col, void *c_val,
                 int32_t *err, hipStream_t s) {
    const int64_t n_all = tile_items(t);
    if (n_all <= 0) return 0;
    hipLaunchKernelGGL(k_tile_tasks_num, dim3(grid_for(n_all, 256, 65536)), dim3(256), 0, s, t.tasks, n_all, t.large_perm,
                       tile_large(t), t.nh, t.nnz, slot, heavy_rows, c_row_ptr, tasks);
    GM_CHECK_LAUNCH();
    int launches = 0;
    with_types(ci64, v32, [&](auto ci, auto v) {
        using CI = decltype(ci);
        using V = decltype(v);
        const TileOut<CI, V> o{static_cast<CI *>(c_col), static_cast<V *>(c_val), err};
        const int64_t first = t.bins[TILE_EMPTY + 1];
        auto bin = [&](int64_t b0, int64_t b1, int per_group, int block, auto kernel) {
            if (b1 <= b0) return;
            launch_regions(kernel, block, (b1 - b0 + per_group - 1) / per_group, s, tile_args<V>(t, tasks, b0, b1), o);
            ++launches;
        };
        bin(large_bins[0], large_bins[1], 1, 1024, k_tile_num_dense<1024, CI, V>);
        bin(large_bins[1], large_bins[2], 1, 1024, k_tile_num_rank<1024, TILE_RANK_MAX, CI, V>);
        auto rank_bin = [&](int64_t b0, int64_t b1, int block, auto kernel) {
            if (b1 - b0 <= RANK_FEW)
                bin(b0, b1, 1, 1024, k_tile_num_rank<1024, TILE_RANK_MAX, CI, V>);
            else
                bin(b0, b1, 1, block, kernel);
        };
        rank_bin(large_bins[2], large_bins[3], 512, k_tile_num_rank<512, TILE_RANK_MID, CI, V>);
        rank_bin(large_bins[3], large_bins[4], 256, k_tile_num_rank<256, TILE_RANK_MIN, CI, V>);
        bin(t.bins[TILE_L] - first, t.bins[TILE_L + 1] - first, 1, 512, k_tile_num_small<512, TILE_MERGE, 1, CI, V>);
        bin(t.bins[TILE_S] - first, t.bins[TILE_S + 1] - first, 1, 256, k_tile_num_small<256, TILE_S_MAX, 1, CI, V>);
        bin(t.bins[TILE_T] - first, t.bins[TILE_T + 1] - first, 4, 256, k_tile_num_small<64, TILE_T_MAX, 4, CI, V>);
    });
    return launches;
}

}  // namespace gm
