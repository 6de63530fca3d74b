// Gram scan kernel for gfx950: filter, walks and emission of every output
// unit in one kernel, for images with a gram filter (every pattern of four
// bytes or more).
//
// The filter does not test every start position.  A pattern of S + 3 bytes or
// more that starts at p covers the four-byte gram at the next multiple t of S
// (t - p < S), so testing the grams at the multiples of S against the grams
// at offsets 0 .. S-1 of every pattern drops no match.  With S = 4 those
// grams are the text's aligned dwords, as the loads deliver them: 16 start
// positions a lane cost four tests of ten VALU instructions instead of
// sixteen of four and a second stage over many more survivors.
//
// Over four symbols (DNA) a gram of four bytes keeps 1 position in 256 or
// more; there a gram is up to 16 symbols, packed to two bits each by 8-bit dot
// products, the next 16 symbols taken from the next lane.  What bounds it are
// false positives: each reads its slots from L2 and takes 8 us of 1 GiB's time
// per KiB.  Patterns of 19 symbols or more hold four 16-symbol grams that start
// one after another, so there every position is tested against the grams at
// offsets 0 .. 3, one bit each, and four hits in a row are wanted: 1% for
// 100,000 patterns, where two bits a gram leave 11% of every second position or
// 29% of every fourth.  1 GiB, 100,000 patterns of 20 to 32: 333 us a call, of
// which VALU issue takes 280 (164 instructions a KiB; a hash per position and a
// second stage of walks 830, every second position 571, pairs of two-bit hits
// 343); 32 MiB, 500 patterns of 9 to 14, where the generic filter kept every
// 25th position: 26 us (90).
//
//   * a workgroup loads the bitmap (two hashed bits per gram, at most 128 KiB)
//     into LDS; each wave owns units of G consecutive 1 KiB chunks of test
//     positions and keeps a group of GC chunks of loads in flight;
//   * every test that hits queues its gram and position at once: reading the
//     gram again later would double the HBM traffic, since the text streams
//     through L2 faster than the queue fills;
//   * 64 queued grams at a time are checked against 16-bit slots in global
//     memory (L2);
//   * a slot's record gives the offset of the gram in its pattern, that is the
//     start, and the pattern, which is compared with the text in one go; a
//     gram that several patterns share at one trie node is walked from that
//     node, and one of several nodes has its possible starts walked from their
//     depth-K nodes;
//   * matches of a unit collect in LDS, past that in the unit's part of a
//     global buffer, and are staged in (pos, id) order.
// Unit u holds the starts from S - 1 before its first test position to S - 1
// before its end, so no start is seen by two units.
#include <hip/hip_runtime.h>

#include "trie.hpp"
#include "wave_common.hpp"

namespace pfac {

// A wave's lists in LDS: queued grams (6 bytes each), grams whose starts are
// to be looked at (6) and matches of the unit (8).  The short ones fit 16 waves
// beside a bitmap of 128 KiB; texts that hit often (words: 50 grams a KiB)
// want the long ones, so that a group never overflows the queue.  Either way a
// wave's area is a multiple of 16 bytes: emit_spilled reads 16 at a time from
// its start.
constexpr uint32_t kGqShort = 160, kGcShort = 84, kGmShort = 64;
constexpr uint32_t kGqLong = 444, kGcLong = 192, kGmLong = 160;
constexpr uint32_t kGqPad = 4;    // entries past the queue's end, the first written by grams that find it full
constexpr uint32_t kGqRoom = 57;  // the queue is emptied when a group leaves less room

typedef __attribute__((address_space(3))) const uint32_t lds_word_t;
typedef __attribute__((address_space(4))) const uint32_t scalar_u32_t;
typedef __attribute__((address_space(4))) const uint64_t scalar_u64_t;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const u32x2 lds_pair_t;
typedef __attribute__((address_space(3))) uint32_t lds_out32_t;
typedef __attribute__((address_space(3))) uint16_t lds_out16_t;

// The filter's hash of a gram: its 16-bit halves times two odd constants.
__device__ __forceinline__ uint32_t gram_hash(uint32_t x) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    union { uint32_t w; u16x2 h; } a, c;
    a.w = x;
    c.w = kGramC0 | kGramC1 << 16;
    return __builtin_amdgcn_udot2(a.h, c.h, 0u, false);
}

// at + the set bits of m below the lane
__device__ __forceinline__ uint32_t mbcnt_from(unsigned long long m, uint32_t at) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, at));
}

// the lesser of each 16-bit half
__device__ __forceinline__ uint32_t pk_min(uint32_t x, uint32_t y) {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    union { uint32_t w; u16x2 h; } a, b, r;
    a.w = x;
    b.w = y;
    r.h = __builtin_elementwise_min(a.h, b.h);
    return r.w;
}

// The kernel's arguments read again from the kernel argument segment: code
// that runs once per unit takes them from there, so that they do not occupy
// scalar registers (or spill) in the loop over the chunks.
__device__ __forceinline__ const ScanArgs &again(const ScanArgs &a) {
    auto *p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    (void)a;
    return *(const ScanArgs *)(const void *)p;
}

// Wait for all loads of the wave: at the end of code that runs once per unit,
// so that no load of it into a register that the chunk loop uses stays open
// (the compiler would set the loop's waits for that path).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }

// The texts of one unit's starts: the one text they all lie in (known), or
// the range [lo, hi) of texts and the lanes' first 64 starts of it.
struct UnitTexts {
    bool known = false;
    uint32_t tid = 0, lo = 0, hi = 0;
    uint64_t start = 0, end = 0;  // of the one text
    uint64_t at = 0;              // the lane's: start of text lo + lane (frame position)
};

// Texts of unit u, whose starts begin at frame position ubase.
__device__ __forceinline__ UnitTexts unit_texts(const ScanArgs &a, uint32_t u, uint64_t ubase) {
    UnitTexts t;
    if (!a.offsets) {
        t.known = true;
        t.start = a.shift;
        t.end = a.shift + a.total;
        return t;
    }
    // (scalar loads: they do not wait for the chunks in flight)
    const scalar_u32_t *first = (const scalar_u32_t *)(uintptr_t)a.tile_first_text;
    const scalar_u64_t *off = (const scalar_u64_t *)(uintptr_t)a.offsets;
    t.lo = first[u];
    t.hi = (u + 1 < (uint32_t)a.n_tiles ? first[u + 1] : a.n_texts - 1) + 1;
    if (t.hi - t.lo == 1) {
        t.tid = t.lo;
        t.start = off[t.lo] + a.shift;
        t.end = off[t.lo + 1] + a.shift;
        // (starts before the first text's are refused by their position)
        t.known = true;
    } else {
        t.at = a.offsets[min(t.lo + lane_id(), a.n_texts)] + a.shift;
    }
    return t;
}

// The text holding frame position p (of the unit's starts, inside the frame's
// valid range): its index, start and end.  Every lane of the wave calls it at
// once; a lane without such a position gets any text.
struct TextSpan {
    uint32_t tid;
    uint64_t start, end;
};

__device__ __forceinline__ TextSpan text_span(const ScanArgs &a, uint64_t p, const UnitTexts &t) {
    if (t.known) return TextSpan{t.tid, t.start, t.end};
    uint32_t i;
    if (t.hi - t.lo < 64) {
        // among the starts that the lanes hold (those past hi lie past p):
        // the largest r with start(lo + r) <= p
        uint32_t r = 0;
        for (uint32_t step = 32; step > 0; step >>= 1) {
            const uint64_t v = __shfl(t.at, (int)(r + step), 64);
            if (v <= p && r + step < t.hi - t.lo) r += step;
        }
        const uint64_t s0 = __shfl(t.at, (int)r, 64), s1 = __shfl(t.at, (int)(r + 1), 64);
        return TextSpan{t.lo + r, s0, s1};
    }
    i = text_of(a.offsets, t.lo, t.hi, a.shift, p);
    return TextSpan{i, a.offsets[i] + a.shift, a.offsets[i + 1] + a.shift};
}

// 20 text bytes at frame position p as five words, or false when their whole
// loads could pass the text's last 16-byte block (at blk_hi).
__device__ __forceinline__ bool text20(const uint8_t *base, uint64_t p, uint64_t blk_hi, uint32_t (&t)[5]) {
    const uint64_t p4 = p & ~3ull;
    if (p4 + 24 > blk_hi + 16) return false;
    const uint32_t *q = (const uint32_t *)(base + p4);
    uint32_t w[6];
#pragma unroll
    for (int k = 0; k < 6; k++) w[k] = q[k];
#pragma unroll
    for (int k = 0; k < 5; k++) t[k] = __builtin_amdgcn_alignbyte(w[k + 1], w[k], (uint32_t)(p & 3));
    return true;
}

// whether the first n (at most 20) of the text bytes t are those at pat
__device__ __forceinline__ bool equal20(const uint32_t (&t)[5], const uint8_t *pat, uint32_t n) {
    const uint32_t *c = (const uint32_t *)pat;
    uint32_t diff = 0;
#pragma unroll
    for (int k = 0; k < 5; k++) {
        const int32_t left = (int32_t)n - 4 * k;
        diff |= (t[k] ^ c[k]) & (left >= 4 ? 0xffffffffu : left <= 0 ? 0u : (1u << (8 * left)) - 1u);
    }
    return diff == 0;
}

// walk_g from node v at depth d with the first 16 text bytes in registers: a
// step down to there is one dependent load, the node.  (One body for both, with
// the byte from a functor, made 16 MiB of words 2% slower.)
__device__ __forceinline__ uint2 walk_from(const ImageView &im, const uint8_t *base, uint64_t p, uint32_t lim,
                                           uint32_t v, uint32_t d, uint64_t hi_valid, const uint4 t) {
    uint2 hit = make_uint2(0, 0);
    for (;;) {
        const uint4 r = im.node[v];
        if (r.z & kTermFlagD) hit = make_uint2(r.w, r.z >> kCountShiftD);
        const uint32_t nc = r.z & 0xffffu;
        if (nc == 0 || d >= lim) break;
        const bool skip = (r.z & kSkipFlagD) != 0;
        if (skip) {
            const uint32_t len = r.z >> kSkipShiftD;
            if (d + len > lim) break;
            if (p + d + len + 36 <= hi_valid) {
                const bool leaf = (r.z & kLeafEndD) != 0;
                if (!chain_equal_g(base, p + d, im.chain, leaf ? r.x & 0xffffffu : r.x, len)) break;
                if (leaf) {
                    hit = make_uint2(r.w, r.x >> 24);
                    break;
                }
                v = r.w;
                d += len;
                continue;
            }
        }
        uint32_t c;
        if (d < 16) {
            const uint32_t lo = d & 4 ? t.y : t.x, hi = d & 4 ? t.w : t.z;
            c = ((d & 8 ? hi : lo) >> (8 * (d & 3))) & 0xffu;
        } else {
            c = base[p + d];
        }
        uint32_t j;
        if (skip) {
            if (c != im.label[r.y - 1]) break;
            j = 0;
        } else if (nc <= 4) {
            const uint32_t x = r.x ^ (c * 0x01010101u);
            const uint32_t m = (x - 0x01010101u) & ~x & 0x80808080u;  // lowest flag = first zero byte
            if (m == 0) break;
            j = (uint32_t)__builtin_ctz(m) >> 3;
            if (j >= nc) break;
        } else {
            const uint8_t *lab = im.label + (r.y - 1);
            uint32_t lo = 0, hi = nc;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (lab[mid] < c) lo = mid + 1; else hi = mid;
            }
            if (lo == nc || lab[lo] != c) break;
            j = lo;
        }
        v = r.y + j;
        d++;
    }
    return hit;
}

// Walk for the start p whose text ends at `end` (end - p >= the shortest
// pattern), from the depth-K node of its first K (at most 12) symbols.
__device__ __forceinline__ uint2 walk_start(const ImageView &im, const uint8_t *base, uint64_t p,
                                            uint64_t end, uint64_t hi_valid) {
    const uint32_t K = im.K;
    const uint32_t lim = (uint32_t)umin64(end - p, 0xffffffffull);
    uint32_t v = 0;
    if (K) {
        uint32_t code = 0, bad = 0;
        for (uint32_t d = 0; d < K; d++) {
            const uint32_t byte = base[p + d];
            const uint32_t s = im.identity ? byte : (uint32_t)im.sym[byte];
            bad |= im.identity ? 0u : (uint32_t)(s == 0xffu);
            code = (code << im.b) | s;
        }
        if (bad) return make_uint2(0, 0);
        const uint2 lv = ((const uint2 *)im.lvl)[code >> 5];
        const uint32_t bit = code & 31u;
        if (!((lv.x >> bit) & 1u)) return make_uint2(0, 0);
        v = im.lvl_start + lv.y + (uint32_t)__builtin_popcount(lv.x & ((1u << bit) - 1u));
    }
    return walk_g(im, base, p, lim, v, K, hi_valid);
}

// A start's pattern list (0 ids: no match), for starts in any order; `in`:
// the lane has one.
__device__ __forceinline__ uint2 scan_start(const ScanArgs &a, bool in, uint64_t p, const UnitTexts &ut) {
    const TextSpan t = text_span(a, p, ut);
    // (a start before the text wraps around)
    if (!in || p - a.shift >= a.total || t.end - p < a.im.min_len) return make_uint2(0, 0);
    return walk_start(a.im, a.base, p, t.end, a.shift + a.total);
}

// 1 when the text at frame position p equals the `len` pattern bytes at pat
// (a multiple of four), 0 when not, -1 when its whole loads could pass the
// text's last 16-byte block (at blk_hi).  64 bytes a round, all in flight.
__device__ __forceinline__ int equal_pattern(const uint8_t *base, uint64_t p, const uint8_t *pat, uint32_t len,
                                             uint64_t blk_hi) {
    const uint64_t p4 = p & ~3ull;
    if (p4 + (len + 63u) / 64u * 64u + 4 > blk_hi + 16) return -1;
    const uint32_t sh = (uint32_t)(p & 3);
    uint32_t diff = 0;
    for (uint32_t i = 0; i < len; i += 64) {
        const uint32_t *t32 = (const uint32_t *)(base + p4 + i);
        const uint32_t *c32 = (const uint32_t *)(pat + i);
        uint32_t tw[17], cw[16];
#pragma unroll
        for (int k = 0; k < 17; k++) tw[k] = t32[k];
#pragma unroll
        for (int k = 0; k < 16; k++) cw[k] = c32[k];
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const int32_t left = (int32_t)(len - i) - 4 * k;
            const uint32_t mask = left >= 4 ? 0xffffffffu : (left <= 0 ? 0u : ((1u << (8 * left)) - 1u));
            diff |= (__builtin_amdgcn_alignbyte(tw[k + 1], tw[k], sh) ^ cw[k]) & mask;
        }
        if (diff) return 0;
    }
    return 1;
}

// Matches in the kernel's lists: x = unit position | stored list length << 16,
// y = the list's offset or kGramId | the id of a list of one.
__device__ __forceinline__ uint2 list_of(const ImageView &im, uint2 e) {
    const uint32_t n = e.x >> 16;
    return (e.y & kGramId) ? make_uint2(e.y, 1u) : hit_list(im, make_uint2(e.y, n));
}

// Write the records of a match at p (`ids` from list_of; none: no match) to
// dst[idx ..] below cap.
__device__ __forceinline__ void put(const ScanArgs &a, uint64_t p, uint2 ids, pfac_match *dst, uint64_t idx,
                                    uint64_t cap, const UnitTexts &ut) {
    const TextSpan t = text_span(a, p, ut);
    // four ids at a time, so that their loads do not wait for stores
    for (uint32_t k = 0; k < ids.y && idx < cap; k += 4, idx += 4) {
        uint32_t id[4];
#pragma unroll
        for (uint32_t q = 0; q < 4; q++)
            id[q] = (ids.x & kGramId) ? ids.x & ~kGramId : a.im.pout_ids[ids.x + min(k + q, ids.y - 1)];
#pragma unroll
        for (uint32_t q = 0; q < 4; q++) {
            pfac_match m;
            m.pos = p - t.start;
            m.pattern_id = id[q];
            m.text_id = t.tid + a.text_id0;
            if (k + q < ids.y && idx + q < cap) dst[idx + q] = m;
        }
    }
    if (a.counts && ids.y) a.counts[p - a.shift] = ids.y;
}

// Reserve `total` records of unit u: its inline slots, its part of the spill
// area where the unit's lists have not used that (spare), or the staging area.
// (One atomic per unit on the staging cursor takes 10 ns each: 33 of 69 us on
// 16 MiB of words with 10 matches a KiB.)
__device__ __forceinline__ void reserve_unit(const ScanArgs &a, uint64_t u, uint32_t total, bool spare,
                                             pfac_match *&dst, uint64_t &base, uint64_t &cap) {
    const uint32_t lane = lane_id();
    unsigned long long b = ~0ull;
    dst = a.inline_stage + u * a.inline_cap;
    cap = a.inline_cap;
    if (total > cap) {
        if (spare && total <= a.spill_cap) {
            b = kUnitSpill;
            dst = (pfac_match *)(a.spill + 2 * u * a.spill_cap);
            cap = a.spill_cap;
        } else {
            if (lane == 0) b = atomicAdd(a.stage_cursor, (unsigned long long)total);
            b = __shfl(b, 0, 64);
            dst = a.stage;
            cap = a.stage_cap;
        }
    }
    if (lane == 0) {
        a.unit_count[u] = total;
        a.unit_off[u] = b;
        if (a.blocksum && total) atomicAdd(&a.blocksum[u >> kSumShift], (unsigned long long)total);
    }
    base = b >= kUnitSpill ? 0 : b;
}

// Stage a unit of at most 64 matches, one a lane: each is ranked by its
// position against the others (scalar reads of their lanes).
__device__ __forceinline__ void emit_small(const ScanArgs &a, uint64_t u, uint64_t ubase, const uint2 *wm,
                                           uint32_t mn, uint2 *sorted, const UnitTexts &ut) {
    const uint32_t lane = lane_id();
    if (mn == 0) {
        if (lane == 0) a.unit_count[u] = 0;
        return;
    }
    const uint2 e = wm[lane];
    const uint32_t pos = e.x & 0xffffu;
    uint32_t rk = 0;
    for (uint32_t q = 0; q < mn; q++)
        rk += (uint32_t)__builtin_amdgcn_readlane((int)pos, (int)q) < pos ? 1u : 0u;
    if (lane < mn) sorted[rk] = e;
    wave_sync();
    const uint2 f = sorted[lane];
    const uint2 ids = lane < mn ? list_of(a.im, f) : make_uint2(0, 0);
    uint32_t total;
    const uint32_t before = wave_excl_scan(ids.y, total);
    pfac_match *dst;
    uint64_t base, cap;
    reserve_unit(a, u, total, true, dst, base, cap);
    put(a, ubase + (f.x & 0xffffu), ids, dst, base + before, cap, ut);
}

// Stage a unit of more matches that all lie in LDS, ranked likewise against
// LDS reads that every lane shares.
__device__ __forceinline__ void emit_lds(const ScanArgs &a, uint64_t u, uint64_t ubase, const uint2 *wm,
                                         uint32_t mn, uint2 *sorted, const UnitTexts &ut) {
    const uint32_t lane = lane_id();
    uint32_t total = 0;
    for (uint32_t r = 0; r < mn; r += 64) {
        const uint32_t i = r + lane;
        const uint2 e = wm[min(i, mn - 1)];
        const uint32_t pos = e.x & 0xffffu;
        uint32_t rk = 0;
#pragma unroll 8
        for (uint32_t q = 0; q < mn; q++) rk += (wm[q].x & 0xffffu) < pos ? 1u : 0u;
        if (i < mn) sorted[rk] = e;
        uint32_t t;
        wave_excl_scan(i < mn ? list_of(a.im, e).y : 0u, t);
        total += t;
    }
    wave_sync();
    pfac_match *dst;
    uint64_t base, cap;
    reserve_unit(a, u, total, true, dst, base, cap);
    for (uint32_t r = 0; r < mn; r += 64) {
        const uint32_t i = r + lane;
        const uint2 e = sorted[min(i, mn - 1)];
        const uint2 ids = i < mn ? list_of(a.im, e) : make_uint2(0, 0);
        uint32_t t;
        const uint32_t before = wave_excl_scan(ids.y, t);
        put(a, ubase + (e.x & 0xffffu), ids, dst, base + before, cap, ut);
        base += t;
    }
}

// Unit u again, 64 starts at a time in position order, when its matches
// overflow both lists: one pass counts, the next emits.
__device__ __forceinline__ void redo_unit(const ScanArgs &a, uint64_t u, uint64_t ubase, uint32_t n_starts,
                                          const UnitTexts &ut) {
    const uint32_t lane = lane_id();
    pfac_match *dst = nullptr;
    uint64_t base = 0, cap = 0;
    uint32_t total = 0;
    for (int pass = 0; pass < 2; pass++) {
        for (uint32_t r = 0; r < n_starts; r += 64) {
            const uint64_t p = ubase + r + lane;
            uint2 ids = make_uint2(0, 0);
            const uint2 h = scan_start(a, r + lane < n_starts, p, ut);
            if (h.y) ids = hit_list(a.im, h);
            uint32_t t;
            const uint32_t before = wave_excl_scan(ids.y, t);
            if (pass == 0) {
                total += t;
            } else {
                put(a, p, ids, dst, base + before, cap, ut);
                base += t;
            }
        }
        if (pass == 0) reserve_unit(a, u, total, true, dst, base, cap);
    }
}

// Stage a unit whose matches went past mcap: entry i is wm[i] or
// spill[i - mcap], in no order.  For each window of 8,192 positions the
// entries in it are ranked by a bit map of its positions (256 words and 64
// prefix words in LDS) and written in position order to `sorted` (global),
// which a last pass emits.
__device__ __forceinline__ void emit_spilled(const ScanArgs &a, uint64_t u, uint64_t ubase, const uint2 *wm,
                                             uint32_t mcap, const uint2 *spill, uint2 *sorted, uint32_t mn,
                                             uint32_t n_starts, uint32_t *map, uint32_t *pre, const UnitTexts &ut) {
    const uint32_t lane = lane_id();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    // (two loads, not one through a pointer to either memory)
    auto get = [&](uint32_t i) -> uint2 {
        const u32x2 m = ((lds_pair_t *)wm)[min(i, mcap - 1)];
        uint2 e = make_uint2(m.x, m.y);
        if (i >= mcap) e = spill[i - mcap];
        return e;
    };
    uint32_t done = 0, total = 0;
    for (uint32_t w0 = 0; w0 < n_starts && done < mn; w0 += 8192) {
        for (uint32_t i = lane; i < 256; i += 64) map[i] = 0;
        wave_sync();
        for (uint32_t r = 0; r < mn; r += 64) {
            const uint32_t i = r + lane;
            const uint32_t q = i < mn ? (get(i).x & 0xffffu) - w0 : ~0u;
            if (q < 8192) atomicOr(&map[q >> 5], 1u << (q & 31u));
        }
        wave_sync();
        const uint4 m4 = ((const uint4 *)map)[lane];
        uint32_t all;
        pre[lane] = wave_excl_scan((uint32_t)(__builtin_popcount(m4.x) + __builtin_popcount(m4.y) +
                                              __builtin_popcount(m4.z) + __builtin_popcount(m4.w)), all);
        wave_sync();
        for (uint32_t r = 0; r < mn; r += 64) {
            const uint32_t i = r + lane;
            uint32_t n = 0;
            if (i < mn) {
                const uint2 e = get(i);
                const uint32_t q = (e.x & 0xffffu) - w0, w = q >> 5;
                if (q < 8192) {
                    uint32_t rk = pre[w >> 2] + (uint32_t)__builtin_popcount(map[w] & ((1u << (q & 31u)) - 1u));
                    for (uint32_t k = w & ~3u; k < w; k++) rk += (uint32_t)__builtin_popcount(map[k]);
                    sorted[done + rk] = e;
                    n = list_of(a.im, e).y;
                }
            }
            uint32_t t;
            wave_excl_scan(n, t);
            total += t;
        }
        wave_sync();
        done += all;
    }
    pfac_match *dst;
    uint64_t base, cap;
    reserve_unit(a, u, total, false, dst, base, cap);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    for (uint32_t r = 0; r < mn; r += 64) {
        const uint32_t i = r + lane;
        uint2 e = make_uint2(0, 0), ids = make_uint2(0, 0);
        if (i < mn) {
            e = sorted[i];
            ids = list_of(a.im, e);
        }
        uint32_t t;
        const uint32_t before = wave_excl_scan(ids.y, t);
        put(a, ubase + (e.x & 0xffffu), ids, dst, base + before, cap, ut);
        base += t;
    }
}

// S: the distance of test positions (im.gram_s).  LT: the bitmap is copied to
// LDS; without it the tests read it from global memory.  SYM: a gram is
// im.gram_q symbols of two bits each; 2 (S = 1): 16 of them, and a position
// counts when the three after it hit too.
template <int S, bool LT, int SYM>
__global__ __launch_bounds__(1024) void scan_grams(const ScanArgs a) {
    extern __shared__ __align__(16) uint8_t lds[];
    constexpr uint32_t TL = 16 / S;            // tests per lane and chunk
    constexpr uint32_t GC = SYM ? 3 : S == 4 ? 4 : 2;  // chunks per group and in flight
    const ImageView &im = a.im;
    const uint32_t tid = threadIdx.x;
    const uint32_t waves = blockDim.x >> 6;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t lane = tid & 63;

    // the bitmap by direct global-to-LDS loads, at LDS address 0
    const uint32_t n_tab = LT ? (4u << im.gram_lw) / 16 : 0u;
    for (uint32_t b = wave * 64; b < n_tab; b += waves * 64)
        if (b + lane < n_tab)
            __builtin_amdgcn_global_load_lds((const void *)((const uint4 *)im.gram + b + lane),
                                             (__attribute__((address_space(3))) void *)(lds + 16 * b), 16, 0, 0);
    if (tid == 0) *(uint32_t *)(lds + a.off_wave + waves * a.wave_bytes) = waves;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    uint8_t *wbase = lds + a.off_wave + wave * a.wave_bytes;
    const uint32_t gq = a.gq;
    uint32_t *wq = (uint32_t *)wbase;                        // queue: gram ...
    uint16_t *wqp = (uint16_t *)(wbase + 4 * (gq + kGqPad + a.gc));  // ... and unit position
    uint32_t *wcr = wq + gq + kGqPad;                            // starts: record of the gram's slot ...
    uint16_t *wcp = wqp + gq + kGqPad;                            // ... and its unit position
    uint2 *wm = (uint2 *)(wbase + 6 * (gq + kGqPad + a.gc));          // matches

    const uint64_t hi_valid = a.shift + a.total;
    const uint32_t n_u = (uint32_t)a.n_tiles, n_ch = (uint32_t)a.n_plan, G = a.group;
    const uint32_t ustride = gridDim.x * waves;
    const uint64_t blk_hi = (hi_valid - 1) & ~15ull;
    const uint32_t lane16 = 16u * lane;
    uint32_t adr_mask = (4u << im.gram_lw) - 4u;
    const uint32_t lb = im.gfp_lb;

    // ---- loads: GC chunks of a unit from chunk g on; a slot past the unit's
    // last chunk repeats it, lanes past the text's last 16-byte block repeat
    // that, so every load is issued and every wait counts only later loads
    struct Slot {
        uint4 v;
        uint32_t h;  // the dword after the lane's 16 bytes (S < 4); SYM: dword lane % 4 of the 16 bytes after the chunk
    };
    struct Cur {
        uint32_t u, g, n;  // unit, first chunk of the group, chunks of the unit
    };
    auto start_at = [&](uint32_t u) -> Cur { return Cur{u, 0u, u < n_u ? min(G, n_ch - u * G) : 0u}; };
    // the workgroup's units are blockIdx.x * waves + (0 .. waves - 1), plus
    // multiples of the grid's waves; a wave's first one is its own, each next
    // one is the workgroup's next, so that a wave held up by a cluster of
    // matches or of small texts ends with fewer units
    uint32_t *wnext = (uint32_t *)(lds + a.off_wave + waves * a.wave_bytes);
    auto advance = [&](Cur &c) {
        c.g += GC;
        if (c.g < c.n) return;
        uint32_t i = 0;
        if (lane == 0) i = atomicAdd(wnext, 1u);
        i = (uint32_t)__builtin_amdgcn_readfirstlane((int)i);
        c = start_at(i / waves * ustride + blockIdx.x * waves + i % waves);
    };
    auto load = [&](const Cur &c, uint32_t i) -> Slot {
        uint64_t sb = ((uint64_t)c.u * G + c.g) * kChunk;
        sb = sb < blk_hi ? sb : blk_hi;
        const uint32_t lim = (uint32_t)umin64(blk_hi - sb, 0x7fffffffull);
        const uint32_t last = c.n > c.g ? c.n - c.g - 1 : 0u;
        const uint32_t o = lane16 + kChunk * min(i, last);
        Slot s;
        // (non-temporal: the text is read once, the tables of the walks stay in L2)
        const u32x4 v = __builtin_nontemporal_load((const u32x4 *)(a.base + sb + min(o, lim)));
        s.v = make_uint4(v.x, v.y, v.z, v.w);
        if (SYM)
            s.h = *(const uint32_t *)(a.base + sb + min(kChunk * (min(i, last) + 1), lim) + 4 * (lane & 3));
        else
            s.h = S == 4 ? 0u : *(const uint32_t *)(a.base + sb + min(o + 16u, lim));
        return s;
    };
    uint32_t qn = 0;  // grams queued (kept in scalar registers, as all counts)
    // the filter's word of gram x (one 16-bit dot product: two shifts, two
    // multiplies and an add fewer than 24-bit ones), and its bit 0 set if
    // both bits of x are
    auto lookup = [&](uint32_t x, uint32_t &h) -> uint32_t {
        h = gram_hash(x);
        const uint32_t at = (SYM == 2 ? h : h >> (kGramShift - 2)) & adr_mask;
        return LT ? *(lds_word_t *)(uintptr_t)at : *(const uint32_t *)((const uint8_t *)im.gram + at);
    };
    auto test = [&](uint32_t ent, uint32_t h, uint32_t x) -> uint32_t {
        return (SYM == 2 ? 1u : ent >> (h & 31u)) & (ent >> (x & 31u)) & 1u;
    };
    // queue the grams x that hit, at unit positions pos; past the queue's end
    // they are counted, and written to the entry there that nothing reads.
    // (The loop has more uniform values than scalar registers: those of every
    // test are in vector ones.)
    uint32_t q_at = a.off_wave + wave * a.wave_bytes, qp_at = q_at + 4 * (gq + kGqPad + a.gc), q_end = gq;
    asm volatile("" : "+v"(adr_mask), "+v"(q_at), "+v"(qp_at), "+v"(q_end));
    auto queue = [&](uint32_t hit, uint32_t x, uint32_t pos) {
        const unsigned long long mk = __ballot(hit != 0);
        if (mk == 0) return;
        const uint32_t at = qn;
        qn += (uint32_t)__popcll(mk);
        if (__builtin_amdgcn_inverse_ballot_w64(mk)) {  // the compare's mask as it is
            const uint32_t i = min(mbcnt_from(mk, at), q_end);
            *(lds_out32_t *)(uintptr_t)(q_at + 4 * i) = x;
            *(lds_out16_t *)(uintptr_t)(qp_at + 2 * i) = (uint16_t)pos;
        }
    };
    // four text bytes' symbols, two bits each from bit gram_sh of each byte, in
    // 8 bits from there on (first symbol lowest)
    const uint32_t sym_sh = im.gram_sh;
    uint32_t sym_bits = 0x03030303u << sym_sh;
    uint32_t sym_mask = SYM ? 0xffffffffu >> (32 - 2 * im.gram_q) : 0u;
    if (SYM) asm volatile("" : "+v"(sym_bits), "+v"(sym_mask));
    auto pack4 = [&](uint32_t w) -> uint32_t { return __builtin_amdgcn_udot4(w & sym_bits, 0x40100401u, 0u, false); };
    // Queue a lane's grams that hit (bit j of m: at unit position pos + j * S),
    // one of every lane at a time: symbols, whose grams are one shift away.  (32
    // MiB against 500 motifs: 26 us, 30 with a ballot per test.  Bytes, whose
    // gram is chosen among five registers: 2.1 GB of packets and files 718, 515
    // with a ballot per test.)
    auto queue_bits = [&](uint32_t m, uint32_t p0, uint32_t p1, uint32_t pos) {
        for (;;) {
            const unsigned long long mk = __ballot(m != 0);
            if (mk == 0) return;
            const uint32_t at = qn;
            qn += (uint32_t)__popcll(mk);
            if (__builtin_amdgcn_inverse_ballot_w64(mk)) {
                const uint32_t i = min(mbcnt_from(mk, at), q_end), b = S * (uint32_t)__builtin_ctz(m);
                *(lds_out32_t *)(uintptr_t)(q_at + 4 * i) =
                    __builtin_amdgcn_alignbit(p1, p0, 2 * b) & (SYM == 2 ? ~0u : sym_mask);
                *(lds_out16_t *)(uintptr_t)(qp_at + 2 * i) = (uint16_t)(pos + b);
                m &= m - 1;
            }
        }
    };
    // bytes: the last gram seen that starts nothing behind the dword pass_y
    uint32_t pass_x = im.gram_alph, pass_y = pass_x;
    if (!SYM && S > 1) asm volatile("" : "+v"(pass_x), "+v"(pass_y));
    // the TL tests of a lane's 16 positions from unit position pos on
    auto tests = [&](const Slot &s, uint32_t pos) {
        const uint32_t w[5] = {s.v.x, s.v.y, s.v.z, s.v.w, s.h};
        uint32_t x[TL], h[TL], ent[TL];
        uint32_t p0 = 0, p1 = 0;
        if (SYM) {
            // the lane's 16 symbols and, from the next lane, those after them;
            // lane 63 takes them from the 16 bytes after the chunk
            p0 = (pack4(w[0]) + (pack4(w[1]) << 8)) >> sym_sh | (pack4(w[2]) + (pack4(w[3]) << 8)) << (16 - sym_sh);
            uint32_t e = pack4(w[4]) >> sym_sh << (8 * (lane & 3));
            e |= (uint32_t)__builtin_amdgcn_mov_dpp((int)e, 0xB1, 0xf, 0xf, true);  // of lane ^ 1
            e |= (uint32_t)__builtin_amdgcn_mov_dpp((int)e, 0x4E, 0xf, 0xf, true);  // of lane ^ 2
            p1 = (uint32_t)__builtin_amdgcn_update_dpp((int)e, (int)p0, 0x130, 0xf, 0xf, false);  // of lane + 1
        }
#pragma unroll
        for (uint32_t j = 0; j < TL; j++) {
            const uint32_t b = j * S;
            if (SYM)
                x[j] = (b == 0 ? p0 : __builtin_amdgcn_alignbit(p1, p0, 2 * b)) & (SYM == 2 ? ~0u : sym_mask);
            else
                x[j] = (b & 3) == 0 ? w[b >> 2] : __builtin_amdgcn_alignbyte(w[(b >> 2) + 1], w[b >> 2], b & 3);
            ent[j] = lookup(x[j], h[j]);
        }
        if (SYM) {
            uint32_t m = 0;  // the tests that hit, shifted in from the upper end
#pragma unroll
            for (uint32_t j = 0; j < TL; j++)
                m = __builtin_amdgcn_alignbit((SYM == 2 ? ~0u : ent[j] >> (h[j] & 31u)) & (ent[j] >> (x[j] & 31u)), m, 1);
            if (SYM == 2) {
                // those of the next lane behind them (after lane 63 taken as hits)
                m = __builtin_amdgcn_alignbit((uint32_t)__builtin_amdgcn_update_dpp(-1, (int)m, 0x130, 0xf, 0xf, false) >> 16, m, 16);
                m &= m >> 1;
                m &= (m >> 2) & 0xffffu;
            } else {
                m >>= 32 - TL;
            }
            // a lane whose tests all hit: a run of one symbol, or of a byte
            // outside the alphabet that looks like one (N in place of G); there
            // only the tests at bytes of the alphabet are left (128 MiB, a tenth of
            // it N, 20,000 patterns and G x 20: 1,429 us without this, 45 with; the
            // 16-symbol filter 108)
            constexpr uint32_t kAll = (1u << TL) - 1u;
            if (__builtin_expect(__ballot((m & kAll) == kAll) != 0, 0)) {
                const uint32_t alph = again(a).im.gram_alph;
                uint32_t other = 0;
#pragma unroll
                for (uint32_t q = 0; q < 4; q++) {
                    const uint32_t d = w[q] ^ __builtin_amdgcn_perm(alph, alph, (w[q] >> sym_sh) & 0x03030303u);
                    const uint32_t nz = ((d & 0x7f7f7f7fu) + 0x7f7f7f7fu) | d;  // upper bit of each byte of d that is not zero
#pragma unroll
                    for (uint32_t b = 0; b < 4; b += S) other |= ((nz >> (8 * b + 7)) & 1u) << ((4 * q + b) / S);
                }
                m &= ~other;
            }
            queue_bits(m, p0, p1, pos);
            return;
        }
        // Where a text repeats up to eight bytes (padding, blanks, tables), a gram
        // of theirs hits in every lane, though at offset 1 .. S-1 of a pattern
        // that may start nowhere in it.  In chunks that do (one compare) the hits
        // count only if a pattern begins with the four bytes from one of the S
        // starts on: asked once for a pair of dwords, those of one lane that
        // repeats itself.  (64 MiB with 64 KiB runs of zeros for a tenth of it, one
        // pattern in a hundred with four zeros past its first byte: 210 us without
        // this, 30 with; the prefix filter of the split kernels 51.)
        if (S > 1 && __builtin_expect(__ballot(w[0] == w[2]) != 0, 0)) {
            // the dword before the lane's 16 bytes: of lane - 1; lane 0, which has
            // none, keeps its tests there
            const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[3], 0x138, 0xf, 0xf, false);
            const ScanArgs &r = again(a);
            const scalar_u32_t *first = (const scalar_u32_t *)(uintptr_t)r.im.gper;
            constexpr uint32_t P = 4 / S;  // tests a dword
#pragma unroll
            for (uint32_t k = 0; k < 2 * P; k++) {
                const unsigned long long hits = __ballot(w[0] == w[2] && w[1] == w[3] && test(ent[P + k], h[P + k], x[P + k]) != 0 &&
                                                         (x[P + k] != pass_x || x[k] != pass_y));
                if (hits) {
                    const int l = (int)__builtin_ctzll(hits);
                    const uint32_t x0 = (uint32_t)__builtin_amdgcn_readlane((int)x[P + k], l);
                    const uint32_t y0 = (uint32_t)__builtin_amdgcn_readlane((int)x[k], l);
                    uint32_t any = 0;
#pragma unroll
                    for (uint32_t o = 0; o < S; o++) {
                        const uint32_t f = o == 0 ? x0 : __builtin_amdgcn_alignbyte(x0, y0, 4 - o), g = f * kPfx4Mul;
                        const uint32_t e = first[g >> (32 - r.im.gper_lw)];
                        any |= (e >> ((g >> 5) & 31)) & (e >> (f >> 27)) & 1;
                    }
                    if (!any) {
                        pass_x = x0;
                        pass_y = y0;
                    }
                }
#pragma unroll
                for (uint32_t j = k; j < TL; j += 2 * P) {
                    const uint32_t y = j >= P ? x[j - P] : k == 0 ? before : __builtin_amdgcn_alignbyte(w[0], before, k * S);
                    ent[j] = x[j] == pass_x && y == pass_y && (j >= P || lane != 0) ? 0u : ent[j];
                }
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < TL; j++) queue(test(ent[j], h[j], x[j]), x[j], pos + j * S);
    };

    // ---- the unit being scanned
    uint32_t cn = 0, mn = 0;  // grams with starts, matches
    // The check of 64 queued grams is spread over two groups, so that its
    // loads are not waited for: their slots are loaded after one group's tests
    // and read after the next's.  (All loads of a wave return in order, so a
    // load waited for at once also waits for the chunks in flight.)
    uint32_t nb = 0, tb = 0, gb = 0;
    uint4 fb0 = make_uint4(0, 0, 0, 0), fb1 = fb0;

    // One step of the check.  It is inlined twice: after a group's tests,
    // where the loads it waits for are older than the chunks in flight, and in
    // the loop that empties the queue.
    auto check = [&](uint32_t at_least) __attribute__((always_inline)) {
        if (nb) {
            // the slot with the gram's fingerprint
            const uint32_t want = gb >> (20u - lb) << 4 & 0xfff0u, w2 = want << 16 | want;
            uint32_t m = pk_min(fb0.x ^ w2, fb0.y ^ w2);
            m = pk_min(m, pk_min(fb0.z ^ w2, fb0.w ^ w2));
            m = pk_min(m, pk_min(fb1.x ^ w2, fb1.y ^ w2));
            m = pk_min(m, fb1.z ^ w2);
            m = min(m & 0xffffu, m >> 16);
            const bool pass = lane < nb && m < 14u;
            const unsigned long long mk = __ballot(pass);
            if (pass) {
                const uint32_t i = cn + mbcnt(mk);
                wcr[i] = fb1.w + m;
                wcp[i] = (uint16_t)tb;
            }
            cn += (uint32_t)__popcll(mk);
            nb = 0;
        }
        if (qn >= at_least) {
            // the last (up to) 64 grams of the queue
            nb = min(qn, 64u);
            qn -= nb;
            const uint32_t i = min(qn + lane, gq - 1);
            tb = wqp[i];
            gb = wq[i] * im.pfx4_mul;
            const uint4 *bk = im.gfp + (gb >> (32u - lb) << 1);
            fb0 = bk[0];
            fb1 = bk[1];
        }
    };

    Cur cc = start_at(blockIdx.x * waves + wave);
    Slot slot[GC];
#pragma unroll
    for (uint32_t i = 0; i < GC; i++) {
        // in the order of use, as in the loop: the waits there are set for
        // the path with the fewest later loads
        slot[i] = load(cc, i);
        __builtin_amdgcn_sched_barrier(0);
    }
    while (cc.n) {
        Cur pc = cc;
        advance(pc);
        const uint64_t ulo = (uint64_t)cc.u * G * kChunk;  // frame position of the unit's first chunk
        const uint64_t ubase = ulo - (S - 1);              // start of its range of starts
        const uint32_t rem = cc.n - cc.g;
        const bool last = rem <= GC;
        const uint32_t gpos = cc.g * kChunk + lane16;
        // a chunk that overflows the queue is tested again below, one test at a
        // time
        uint32_t redo = 0;
#pragma unroll
        for (uint32_t i = 0; i < GC; i++) {
            const uint32_t q0 = qn;
            if (i == 0 || i < rem) tests(slot[i], gpos + i * kChunk);
            if (qn > gq) {
                qn = q0;
                redo |= 1u << i;
            }
            // (SYM images may queue 60 grams a chunk)
            if (SYM) {
                wave_sync();
                if (qn >= 64 && cn <= a.gc - 64) check(64);
            }
            slot[i] = load(pc, i);
        }
        if (!SYM) {
            wave_sync();
            check(64);
        }
        uint32_t ra = 0;  // next test of the chunk that is tested again

        if (last || redo || qn + kGqRoom > gq || cn > a.gc - 64) {
            // ---- empty the queue as far as the next group needs it, and wholly
            // after the unit's last group
            const ScanArgs &r = again(a);
            UnitTexts ut = unit_texts(r, cc.u, ubase);
            for (;;) {
                if (redo && qn + 64 <= gq) {
                    const uint32_t pos = gpos + (uint32_t)__builtin_ctz(redo) * kChunk + ra;
                    const uint8_t *ub = a.base + ulo;
                    const uint32_t last4 = (uint32_t)umin64(blk_hi + 12 - ulo, 0x7fffffffull);
                    const uint32_t t4 = min(pos & ~3u, last4);
                    uint32_t x = *(const uint32_t *)(ub + t4), h;
                    if (SYM) {
                        uint64_t k = pack4(x);
                        for (uint32_t i = 1; i < 5; i++)
                            k += (uint64_t)pack4(*(const uint32_t *)(ub + min(t4 + 4 * i, last4))) << (8 * i);
                        x = (uint32_t)(k >> sym_sh >> (2 * (pos & 3u))) & sym_mask;
                    } else if (S < 4) {
                        x = __builtin_amdgcn_alignbyte(*(const uint32_t *)(ub + min(t4 + 4u, last4)), x, pos & 3u);
                    }
                    const uint32_t ent = lookup(x, h);
                    queue(test(ent, h, x), x, pos);
                    wave_sync();
                    ra += S;
                    if (ra == 16) {
                        ra = 0;
                        redo &= redo - 1;
                    }
                }
                const bool done = redo == 0 && (last ? (nb | qn) == 0 : qn < 64);
                if (cn > r.gc - 64 || (last && done)) {
                    // ---- compare or walk the starts; matches go to LDS, past
                    // gm to global memory
                    wave_sync();
                    for (uint32_t c0 = 0; c0 < cn; c0 += 64) {
                        const uint32_t ci = min(c0 + lane, r.gc - 1);
                        const uint32_t t = wcp[ci];
                        uint4 rec = make_uint4(kNone, 0u, 0u, 0u);
                        if (c0 + lane < cn) rec = r.im.grec[wcr[ci]];
                        uint32_t om = 0;
                        uint2 h = make_uint2(0, 0);
                        const uint32_t len = rec.y & 0xffffu;
                        uint32_t pr = t + (uint32_t)(S - 1) - (rec.x == kGramNode ? rec.y & 3u : rec.y >> 16 & 3u);
                        const TextSpan ts = text_span(r, ubase + pr, ut);
                        if (c0 + lane < cn) {
                            om = rec.x == kNone ? rec.y : 0u;
                            if (rec.x == kGramNode && ubase + pr - r.shift < r.total &&
                                ts.end - (ubase + pr) >= r.im.min_len) {
                                const uint32_t o = rec.y & 3u, d = rec.y >> 8;
                                uint32_t tw[5];
                                if (!text20(r.base, ubase + pr, blk_hi, tw))
                                    om = 1u << o;
                                else if (equal20(tw, r.im.gpat + rec.z, d))
                                    h = walk_from(r.im, r.base, ubase + pr,
                                                  (uint32_t)umin64(ts.end - (ubase + pr), 0xffffffffull), rec.w, d,
                                                  hi_valid, make_uint4(tw[0], tw[1], tw[2], tw[3]));
                            } else if (rec.x < kGramNode && ubase + pr - r.shift < r.total &&
                                       ts.end - (ubase + pr) >= len) {
                                const int eq = equal_pattern(r.base, ubase + pr, r.im.gpat + rec.x, len, blk_hi);
                                if (eq < 0)  // too near the text's end for whole loads
                                    om = 1u << (rec.y >> 16 & 3u);
                                else if (eq)
                                    h = make_uint2(rec.z, rec.y >> 18);
                            }
                        }
                        // Of the starts that a record of several nodes leaves,
                        // only those whose first four bytes are a pattern's:
                        // two loads instead of a walk for each (blanks and the
                        // like: one in 200 patterns with four of them past its
                        // first byte, runs of 40 bytes for a tenth of 64 MiB, 45
                        // us, 58 with the walks).
                        if (SYM == 0 && S > 1 && om && rec.x == kNone) {
                            // (the gram's dword and the one before; three where
                            // it need not be aligned)
                            const uint64_t q = ubase + t + (S - 1), q4 = q & ~3ull;
                            if (q4 >= 4 && q4 + (S == 4 ? 4 : 8) <= blk_hi + 16) {
                                const uint32_t *tw = (const uint32_t *)(r.base + q4);
                                const uint32_t w0 = tw[-1], w1 = tw[0], w2 = S == 4 ? 0u : tw[1];
                                const uint32_t at = S == 4 ? 0u : (uint32_t)q & 3u;
                                uint32_t no = 0;
#pragma unroll
                                for (uint32_t o = 0; o < S; o++) {
                                    const uint32_t x = at >= o ? __builtin_amdgcn_alignbyte(w2, w1, at - o) : __builtin_amdgcn_alignbyte(w1, w0, 4 + at - o);
                                    const uint32_t g = x * kPfx4Mul, w = r.im.gper[g >> (32 - r.im.gper_lw)];
                                    no |= (~((w >> ((g >> 5) & 31)) & (w >> (x >> 27))) & 1u) << o;
                                }
                                om &= ~no;
                            }
                        }
                        for (;;) {
                            const bool got = h.y != 0;
                            const unsigned long long mk = __ballot(got);
                            if (got) {
                                const uint32_t s = mn + mbcnt(mk);
                                const uint2 e = make_uint2(pr | (h.y << 16), h.x);
                                if (s < r.gm) wm[s] = e;
                                else if (s - r.gm < r.spill_cap) r.spill[2ull * cc.u * r.spill_cap + s - r.gm] = e;
                            }
                            mn += (uint32_t)__popcll(mk);
                            if (__ballot(om != 0) == 0) break;
                            const bool in = om != 0;
                            if (in) pr = t + (uint32_t)(S - 1) - (uint32_t)__builtin_ctz(om);
                            om &= om - 1;
                            h = scan_start(r, in, ubase + pr, ut);
                        }
                    }
                    cn = 0;
                    wave_sync();
                }
                if (done) break;
                // (the loop ends: with tests left, either the queue takes one
                // above or this takes grams from it; then it only shrinks)
                check(redo ? gq - 63 : last ? 1 : 64);
            }

            // ---- the unit's last group: its matches in (pos, id) order
            wait_loads();
            if (last) {
                uint2 *spill = r.spill + 2ull * cc.u * r.spill_cap;
                if (mn <= 64)
                    emit_small(r, cc.u, ubase, wm, mn, (uint2 *)wbase, ut);
                else if (mn <= r.gm)
                    emit_lds(r, cc.u, ubase, wm, mn, (uint2 *)wbase, ut);
                else if (mn <= r.spill_cap)
                    emit_spilled(r, cc.u, ubase, wm, r.gm, spill, spill + r.spill_cap, mn, cc.n * kChunk, (uint32_t *)wbase,
                                 (uint32_t *)(wbase + 1024), ut);
                else
                    redo_unit(r, cc.u, ubase, cc.n * kChunk, ut);
                mn = 0;
                wave_sync();
            }
        }
        cc = pc;
    }
}

// ------------------------------------------------------------------ launchers

template <bool LT>
static const void *gram_fn(uint32_t s, uint32_t sym) {
    if (sym == 2) return (const void *)scan_grams<1, LT, 2>;
    if (sym == 1)
        return s == 4 ? (const void *)scan_grams<4, LT, 1>
             : s == 2 ? (const void *)scan_grams<2, LT, 1> : (const void *)scan_grams<1, LT, 1>;
    return s == 4 ? (const void *)scan_grams<4, LT, 0>
         : s == 2 ? (const void *)scan_grams<2, LT, 0> : (const void *)scan_grams<1, LT, 0>;
}

static uint32_t gram_sym(const ImageView &im) { return !im.gram_q ? 0u : im.gram_run ? 2u : 1u; }

int gram_fn_id(const ImageView &im) { return (int)(im.gram_s + 8 * gram_sym(im)); }

void gram_lds_layout(ScanArgs &a, uint32_t waves, bool lds_table, uint32_t lds_limit) {
    a.off_wave = lds_table ? 4u << a.im.gram_lw : 0u;
    auto lists = [&](uint32_t gq, uint32_t gc, uint32_t gm) {
        a.gq = gq;
        a.gc = gc;
        a.gm = gm;
        a.wave_bytes = 6 * (gq + kGqPad + gc) + 8 * gm;
        a.lds_total = a.off_wave + waves * a.wave_bytes + 16;
    };
    // the queue's and the starts' place is also where a unit's matches are
    // sorted (at most gm entries, or 256 + 64 words)
    static_assert(4 * (256 + 64) <= 6 * (kGqShort + kGqPad + kGcShort) && 8 * kGmLong <= 6 * (kGqLong + kGqPad + kGcLong), "sort area");
    static_assert(6 * (kGqShort + kGqPad + kGcShort) % 16 == 0 && 8 * kGmShort % 16 == 0 &&
                      6 * (kGqLong + kGqPad + kGcLong) % 16 == 0 && 8 * kGmLong % 16 == 0,
                  "lists and matches at multiples of 16");
    static_assert(kGqShort >= 64 + kGqRoom - 1 && kGcShort >= 64 && kGmShort >= 64, "a round fits");
    lists(kGqLong, kGcLong, kGmLong);
    if (!lds_table || a.lds_total > lds_limit) lists(kGqShort, kGcShort, kGmShort);
}

hipError_t prepare_gram_kernel(int fn_id, uint32_t lds_bytes) {
    // the bitmap is addressed at LDS address 0: no static LDS in front of it
    const void *fn = gram_fn<true>((uint32_t)fn_id & 7u, (uint32_t)fn_id >> 3);
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, fn);
    if (e != hipSuccess) return e;
    if (attr.sharedSizeBytes != 0) return hipErrorInvalidKernelFile;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
}

hipError_t launch_scan_grams(const ScanArgs &a, uint32_t waves, bool lds_table, uint32_t grid, hipStream_t s) {
    ScanArgs arg = a;
    void *args[] = {(void *)&arg};
    const uint32_t sym = gram_sym(a.im);
    const void *fn = lds_table ? gram_fn<true>(a.im.gram_s, sym) : gram_fn<false>(a.im.gram_s, sym);
    const hipError_t e = hipLaunchKernel(fn, dim3(grid), dim3(64 * waves), args, a.lds_total, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

}  // namespace pfac
