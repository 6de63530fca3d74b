// Device helpers shared by the wave kernels (scan_wave.hip, scan_gram.hip):
// wave scans and fences, the walk in global memory and the emission of a
// unit's matches.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.hpp"

namespace pfac {

constexpr uint32_t kChunk = 1024;   // start positions per chunk (16 per lane)

__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t x, uint32_t &total) {
    const uint32_t incl = wave_incl_scan(x);
    total = wave_last(incl);
    return incl - x;
}

__device__ __forceinline__ uint64_t umin64(uint64_t x, uint64_t y) { return x < y ? x : y; }

// The lane index, tied to a value that changes from chunk to chunk: a
// comparison of it inside the chunk loop stays there (one compare) instead
// of being hoisted into a lane mask that occupies two scalar registers for
// the whole kernel.
__device__ __forceinline__ uint32_t lane_at(uint32_t salt) {
    uint32_t l;
    asm("; lane %1" : "=v"(l) : "s"(salt), "0"(threadIdx.x & 63u));
    return l;
}

__device__ __forceinline__ uint32_t mbcnt(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// True when text[g .. g+len) (global) equals chain[o .. o+len); the caller
// guarantees g + len + 36 <= the end of the valid text.
__device__ __forceinline__ bool chain_equal_g(const uint8_t *base, uint64_t g, const uint8_t *chain,
                                              uint32_t o, uint32_t len) {
    const uint32_t *c32 = (const uint32_t *)chain;
    uint32_t diff = 0;
    for (uint32_t i = 0; i < len; i += 32) {
        uint32_t cw[9], tw[9];
        const uint32_t cb = (o + i) >> 2;
        const uint32_t *t32 = (const uint32_t *)(base + ((g + i) & ~3ull));
#pragma unroll
        for (int k = 0; k < 9; k++) cw[k] = c32[cb + k];
#pragma unroll
        for (int k = 0; k < 9; k++) tw[k] = t32[k];
        const uint32_t cs = (o + i) & 3, ts = (uint32_t)((g + i) & 3);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int32_t r = (int32_t)(len - i) - 4 * k;
            const uint32_t mask = r >= 4 ? 0xffffffffu : (r <= 0 ? 0u : ((1u << (8 * r)) - 1u));
            const uint32_t c = __builtin_amdgcn_alignbyte(cw[k + 1], cw[k], cs);
            const uint32_t t = __builtin_amdgcn_alignbyte(tw[k + 1], tw[k], ts);
            diff |= (c ^ t) & mask;
        }
    }
    return diff == 0;
}

// Walk for the start position at frame position p from node v at depth d,
// reading the text from global memory; the text ends lim bytes after p.
// Returns the pattern list of the deepest terminal node passed.
__device__ __forceinline__ uint2 walk_g(const ImageView &im, const uint8_t *base, uint64_t p,
                                        uint32_t lim, uint32_t v, uint32_t d, uint64_t hi_valid) {
    uint2 hit = make_uint2(0, 0);
    for (;;) {
        const uint4 r = im.node[v];
        if (r.z & kTermFlagD) hit = make_uint2(r.w, r.z >> kCountShiftD);
        const uint32_t nc = r.z & 0xffffu;
        if (nc == 0 || d >= lim) break;
        const bool skip = (r.z & kSkipFlagD) != 0;
        if (skip) {
            // no pattern ends inside a single-child run: it matches whole or
            // the walk ends with nothing more to report
            const uint32_t len = r.z >> kSkipShiftD;
            if (d + len > lim) break;
            if (p + d + len + 36 <= hi_valid) {
                const bool leaf = (r.z & kLeafEndD) != 0;
                if (!chain_equal_g(base, p + d, im.chain, leaf ? r.x & 0xffffffu : r.x, len)) break;
                if (leaf) {
                    // the run ends at a leaf: its pattern list is in the record
                    hit = make_uint2(r.w, r.x >> 24);
                    break;
                }
                v = r.w;
                d += len;
                continue;
            }
        }
        const uint32_t c = base[p + d];
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

// Stage the matches of unit u in (pos, id) order.  wm[i] = (unit position |
// stored list length << 16, list offset).  At most inline_cap records go to
// the unit's inline slots; more reserve staging space with one atomic.
__device__ __forceinline__ void emit_unit(const ScanArgs &a, uint64_t u, uint64_t unit_lo,
                                          const uint2 *wm, uint32_t mn, uint2 *sorted,
                                          const UnitText &ut = UnitText{}) {
    const ImageView &im = a.im;
    const uint32_t lane = lane_id();
    if (mn == 0) {
        if (lane == 0) a.unit_count[u] = 0;
        return;
    }
    for (uint32_t i = lane; i < mn; i += 64) {
        const uint2 e = wm[i];
        uint32_t rk = 0;
        for (uint32_t q = 0; q < mn; q++) rk += (wm[q].x & 0xffffu) < (e.x & 0xffffu);
        sorted[rk] = e;
    }
    wave_sync();
    uint32_t total = 0;
    for (uint32_t r0 = 0; r0 < mn; r0 += 64) {
        const uint32_t i = r0 + lane;
        const uint32_t n = i < mn ? hit_list(im, make_uint2(sorted[i].y, sorted[i].x >> 16)).y : 0u;
        uint32_t t;
        wave_excl_scan(n, t);
        total += t;
    }
    pfac_match *dst;
    uint64_t base = 0, cap;
    if (total <= a.inline_cap) {
        dst = a.inline_stage + u * a.inline_cap;
        cap = a.inline_cap;
        if (lane == 0) {
            a.unit_count[u] = total;
            a.unit_off[u] = ~0ull;
            if (a.blocksum) atomicAdd(&a.blocksum[u >> kSumShift], (unsigned long long)total);
        }
    } else {
        unsigned long long b = 0;
        if (lane == 0) {
            b = atomicAdd(a.stage_cursor, (unsigned long long)total);
            a.unit_count[u] = total;
            a.unit_off[u] = b;
            if (a.blocksum) atomicAdd(&a.blocksum[u >> kSumShift], (unsigned long long)total);
        }
        base = __shfl(b, 0, 64);
        dst = a.stage;
        cap = a.stage_cap;
    }
    for (uint32_t r0 = 0; r0 < mn; r0 += 64) {
        const uint32_t i = r0 + lane;
        uint2 ids = make_uint2(0, 0);
        if (i < mn) ids = hit_list(im, make_uint2(sorted[i].y, sorted[i].x >> 16));
        uint32_t t;
        const uint32_t before = wave_excl_scan(ids.y, t);
        if (i < mn) emit(a, unit_lo + (sorted[i].x & 0xffffu), ids, dst, base + before, cap, ut);
        base += t;
    }
}

}  // namespace pfac
