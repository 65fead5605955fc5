// Rank accumulation of a few hundred to a few thousand products in LDS by one
// wave or one work group: sorted distinct columns without sorting and without
// hashing (the accumulator of light rows and of the sparse regions of heavy
// rows).
//
// A column c is found through words of 32 bits: the words of the columns
// themselves (bit c & 31 of word c >> 5), above them a bitmap of the words
// that exist, above that a bitmap of those bitmaps' words, and so on until a
// dense top of at most TOPW words covers the column range. Only words that
// hold something exist below the top: a level is marked, a scan over its words
// numbers their set bits, and these numbers are the places of the next level's
// words. After the last level the number of a column's bit is its rank in the
// sorted output, where the products are summed. The work follows the products
// (each is read once and stays in registers); the column range only adds a
// level per factor of 32.
//
// What bounds it: LDS (about 12 accesses a product; 40 to 54 % of its cycles, a
// third to a half of these bank conflicts) and the latency of the chain row ->
// parts -> products; the vector units are 43 to 60 % busy, 61 to 78 % where
// columns are only counted. Sums of fp32 values keep the LDS at 77 to 79 %.
#pragma once

#include "common.hpp"

namespace gm {

// 32 bits of a level with the number of set bits before them.
struct RankWord {
    uint32_t bits, rank;
};
GM_DEV uint32_t rank_of(const RankWord &x, uint32_t bit) { return x.rank + (uint32_t)__popc(x.bits & ((1u << bit) - 1u)); }

template <int BLOCK>
GM_DEV void region_sync() {
    if (BLOCK == GM_WAVE)
        wave_lds_fence();
    else
        __syncthreads();
}

// Exclusive scan over the threads of a region (one wave, or the whole work
// group with one barrier: `sm` must not be the one of the previous scan).
template <int BLOCK>
GM_DEV uint32_t region_scan(uint32_t x, uint32_t *sm, uint32_t *total) {
    const uint32_t inc = wave_incl_scan<uint32_t>(x);
    if constexpr (BLOCK == GM_WAVE) {
        *total = (uint32_t)__builtin_amdgcn_readlane((int)inc, GM_WAVE - 1);
        return inc - x;
    } else {
        constexpr int NW = BLOCK / GM_WAVE;
        const int w = threadIdx.x / GM_WAVE;
        if ((threadIdx.x & (GM_WAVE - 1)) == GM_WAVE - 1) sm[w] = inc;
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const uint32_t v = sm[q];
            before += q < w ? v : 0u;
            all += v;
        }
        *total = all;
        return before + inc - x;
    }
}

template <int BLOCK, int CAP, bool NUM, typename V>
struct RankLds {
    // (one wave, 128 words instead of 64: a level less for 2^22 columns, no faster, and 54 products a row 10 % slower)
    static constexpr int TOPW = BLOCK == GM_WAVE ? 64 : 256;
    RankWord x[CAP];  // first the parts, then levels
    // first the parts' scales, then levels, then the sums
    union {
        V vals[NUM ? CAP : 1];
        RankWord y[CAP];
    };
    RankWord top[TOPW];
    RankWord ends[CAP / 32];  // last products of the parts; rank: parts that end before the word
    uint32_t scan[2][BLOCK / GM_WAVE];
};

// Sets a bit; true for the product that set it. (Tested first: atomics of
// several lanes on one word take turns.)
GM_DEV bool rank_mark(RankWord *w, uint32_t bit) {
    const uint32_t m = 1u << bit;
    if (lds_peek(&w->bits) & m) return false;
    return !(__hip_atomic_fetch_or(&w->bits, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & m);
}

// Numbers the set bits of words [0, n), at most PER a thread; returns their
// count to every thread. A wave takes consecutive words, 64 at a time (a thread
// taking consecutive words itself meets eight-way bank conflicts: with 256
// words a wave and three levels, two thirds of the LDS cycles).
template <int BLOCK, int PER>
GM_DEV uint32_t rank_number(RankWord *words, int n, uint32_t *sm, int tid) {
    const int per = (n + BLOCK - 1) / BLOCK;  // (uniform)
    if (BLOCK > GM_WAVE && per == 1) {
        const uint32_t b = tid < n ? words[tid].bits : 0u;
        uint32_t total;
        const uint32_t run = region_scan<BLOCK>((uint32_t)__popc(b), sm, &total);
        if (tid < n) words[tid].rank = run;
        return total;
    }
    const int w = BLOCK == GM_WAVE ? 0 : tid / GM_WAVE, i0 = w * per * GM_WAVE + (tid & (GM_WAVE - 1));
    uint32_t before[PER], carry = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (q >= per) break;
        const int i = i0 + q * GM_WAVE;
        const int32_t c = i < n ? __popc(words[i].bits) : 0;
        const int32_t inc = wave_incl_scan<int32_t>(c);
        before[q] = carry + (uint32_t)(inc - c);
        carry += (uint32_t)__builtin_amdgcn_readlane(inc, GM_WAVE - 1);
    }
    uint32_t base = 0, total = carry;
    if constexpr (BLOCK > GM_WAVE) {
        if ((tid & (GM_WAVE - 1)) == 0) sm[w] = carry;
        __syncthreads();
        total = 0;
#pragma unroll
        for (int q = 0; q < BLOCK / GM_WAVE; ++q) {
            const uint32_t v = sm[q];
            base += q < w ? v : 0u;
            total += v;
        }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (q >= per) break;
        const int i = i0 + q * GM_WAVE;
        if (i < n) words[i].rank = base + before[q];
    }
    return total;
}

// Accumulates the products of `src`, at most CAP of them in columns
// [0, width): returns the number of distinct columns; with NUM their sums are
// left in L.vals in order and put(rank, column) is called once per column. A
// thread (lane, when BLOCK is one wave) holds CAP / BLOCK products.
//
// src: np() parts, some of which may be empty; part(q, &st, &aux) gives part
// q's length, start and an offset for its columns; scale(q) its scale;
// RankWord pack(st, off, aux) / Pos at(pack, x) / col(at) / val(at): the
// place and column and value of product x of the region in a part whose first
// product is `off`.
template <int BLOCK, int CAP, bool NUM, typename V, class Src, class Put>
GM_DEV uint32_t rank_region(const Src &src, uint32_t width, RankLds<BLOCK, CAP, NUM, V> &L, int tid, Put &&put) {
    constexpr int EPT = CAP / BLOCK, NE = CAP / 32, TOPW = RankLds<BLOCK, CAP, NUM, V>::TOPW;
    for (int q = tid; q < NE; q += BLOCK) L.ends[q].bits = 0u;
    // levels below the top, and the top's words
    int depth = 1;
    while ((width - 1) >> (5 * depth + 5) >= (uint32_t)TOPW) ++depth;
    const int ntop = (int)((width - 1) >> (5 * depth + 5)) + 1;
    for (int q = tid; q < ntop; q += BLOCK) L.top[q].bits = 0u;
    region_sync<BLOCK>();
    const int64_t np = src.np();
    uint32_t n = 0, nparts = 0;  // products and non-empty parts so far
    int par = 0;
    for (int64_t j = 0; j < np; j += BLOCK) {
        const int64_t q = j + tid;
        uint32_t len = 0, aux = 0;
        int64_t st = 0;
        V scale = (V)0;
        if (q < np) {
            len = src.part(q, &st, &aux);
            if (NUM) scale = src.scale(q);  // (in flight with the part)
        }
        uint32_t tot;
        // products in the low, non-empty parts in the high 16 bits (at most CAP of each)
        const uint32_t ex = region_scan<BLOCK>(len ? (len | 0x10000u) : 0u, L.scan[par], &tot);
        par ^= 1;
        const uint32_t off = n + (ex & 0xffffu), p = nparts + (ex >> 16);
        if (len > 0 && off + len <= (uint32_t)CAP) {
            L.x[p] = src.pack(st, off, aux);
            if (NUM) L.vals[p] = scale;
            __hip_atomic_fetch_or(&L.ends[(off + len - 1) >> 5].bits, 1u << ((off + len - 1) & 31), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        n += tot & 0xffffu;
        nparts += tot >> 16;
        if (n > (uint32_t)CAP) break;  // (cannot happen: the bin holds regions of at most CAP products)
    }
    if (n > (uint32_t)CAP) n = 0;
    region_sync<BLOCK>();
    if (tid < GM_WAVE) {  // parts that end before each word of products
        constexpr int PER = (NE + GM_WAVE - 1) / GM_WAVE;
        uint32_t cnt = 0, b[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            b[q] = tid * PER + q < NE ? L.ends[tid * PER + q].bits : 0u;
            cnt += (uint32_t)__popc(b[q]);
        }
        uint32_t run = wave_incl_scan<uint32_t>(cnt) - cnt;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (tid * PER + q < NE) L.ends[tid * PER + q].rank = run;
            run += (uint32_t)__popc(b[q]);
        }
    }
    region_sync<BLOCK>();
    if (n == 0) return 0;
    uint32_t col[EPT], at[EPT];
    V val[EPT];
    {
        typename Src::Pos pos[EPT];
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const uint32_t x = (uint32_t)(tid + k * BLOCK) < n ? tid + k * BLOCK : n - 1;
            at[k] = rank_of(L.ends[x >> 5], x & 31);
            pos[k] = src.at(L.x[at[k]], x, &col[k]);
        }
        typename Src::Col lc[EPT];
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            lc[k] = src.col(pos[k]);
            if (NUM) val[k] = src.val(pos[k]);
        }
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            if (NUM) val[k] *= L.vals[at[k]];
            col[k] += src.local(lc[k]);
        }
    }
    // the top level
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
        at[k] = col[k] >> (5 * depth + 5);
        if ((uint32_t)(tid + k * BLOCK) < n) rank_mark(&L.top[at[k]], (col[k] >> (5 * depth)) & 31);
    }
    region_sync<BLOCK>();  // (the parts are read)
    uint32_t count = rank_number<BLOCK, (TOPW + BLOCK - 1) / BLOCK>(L.top, ntop, L.scan[par], tid);
    par ^= 1;
    RankWord *above = L.top;
    uint32_t fresh = 0;
    for (int d = depth; d >= 1; --d) {  // this level marks bits 5 (d - 1) .. 5 (d - 1) + 4 of the columns
        RankWord *cur = (d & 1) ? L.x : L.y;
        const int m = (int)count;
        for (int q = tid; q < m; q += BLOCK) cur[q].bits = 0u;
        region_sync<BLOCK>();
#pragma unroll
        for (int k = 0; k < EPT; ++k)
            if ((uint32_t)(tid + k * BLOCK) < n) {
                at[k] = rank_of(above[at[k]], (col[k] >> (5 * d)) & 31);
                const bool first = rank_mark(&cur[at[k]], (col[k] >> (5 * (d - 1))) & 31);
                if (d == 1 && first) fresh |= 1u << k;
            }
        if (!NUM && d == 1) {
            region_scan<BLOCK>((uint32_t)__popc(fresh), L.scan[par], &count);
            return count;
        }
        region_sync<BLOCK>();
        count = rank_number<BLOCK, EPT>(cur, m, L.scan[par], tid);
        par ^= 1;
        above = cur;
    }
    if constexpr (NUM) {
        for (uint32_t q = tid; q < count; q += BLOCK) L.vals[q] = (V)0;
        region_sync<BLOCK>();
#pragma unroll
        for (int k = 0; k < EPT; ++k)
            if ((uint32_t)(tid + k * BLOCK) < n) {
                const uint32_t rk = rank_of(L.x[at[k]], col[k] & 31);
                __hip_atomic_fetch_add(&L.vals[rk], val[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if ((fresh >> k) & 1u) put(rk, col[k]);
            }
        region_sync<BLOCK>();
    }
    return count;
}

}  // namespace gm
