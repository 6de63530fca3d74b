// The gram filter of seeded pattern sets under AddressSanitizer /
// UndefinedBehaviorSanitizer: byte alphabets, words, alphabets of two to four
// symbols, shortest patterns of 4 to 24 bytes, duplicates, patterns that begin
// with others, runs of one to four bytes at every phase.  Every gram at offsets
// 0 .. S-1 of every pattern has its bits in the bitmap, a slot in its bucket and
// a record that leads back to the pattern; the first bytes of every pattern are
// marked.  Exits non-zero where not.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "../../paper_1702_03657_amd/csrc/trie.hpp"

using namespace pfac;

static int fail(const char *what, int seed, size_t pattern, uint32_t o) {
    std::fprintf(stderr, "invariant failed: %s (seed %d, pattern %zu, offset %u)\n", what, seed, pattern, o);
    return 1;
}

int main() {
    const std::string alphabets[] = {"", "abcdefghijklmnopqrstuvwxyz", "ACGT", "01", "ACT", std::string("\0\xff \x20""A", 5)};
    uint32_t with = 0, by_s[5] = {}, runs = 0;
    for (int seed = 0; seed < 240; seed++) {
        std::mt19937 rng(77 + seed);
        const std::string &al = alphabets[seed % 6];
        const bool few = al.size() && al.size() <= 4;
        const bool large = few && seed % 60 == 2;  // where runs of four one-bit hits pay
        const uint32_t k = large ? 40000 : 1 + rng() % (seed % 10 == 0 ? 6000 : 400);
        const uint32_t lo = large ? 20 : few ? 6 + rng() % 19 : 4 + rng() % 6, hi = lo + rng() % 30;
        std::vector<std::string> pats;
        for (uint32_t j = 0; j < k; j++) {
            std::string p;
            const uint32_t len = lo + rng() % (hi - lo + 1);
            if (j > 0 && rng() % 12 == 0) p = pats[rng() % j].substr(0, lo + rng() % 4);
            const uint32_t head = rng() % 6, period = 1 + rng() % 4;
            const bool run = rng() % 5 == 0;
            while (p.size() < len) {
                if (run && p.size() >= head + period && p.size() < head + 12)
                    p += p[p.size() - period];
                else
                    p += al.empty() ? (char)(rng() & 0xff) : al[rng() % al.size()];
            }
            pats.push_back(p);
        }
        std::vector<uint8_t> data;
        std::vector<uint64_t> off(1, 0);
        for (auto &p : pats) {
            data.insert(data.end(), p.begin(), p.end());
            off.push_back(data.size());
        }
        CrsTrie T;
        std::string err;
        if (!build_crs(data.data(), off.data(), k, T, err)) return fail("build", seed, 0, 0);
        DeviceImageHost I;
        pack_image(T, 16, 16, 0, 0, I);
        if (!I.gram_s) continue;
        with++;
        by_s[I.gram_s]++;
        runs += I.gram_run;
        const uint32_t S = I.gram_s, Q = I.gram_q ? I.gram_q : 4;
        if (I.gram.size() != 1u << I.gram_lw || I.gfp.size() != (size_t)16 << I.gfp_lb) return fail("sizes", seed, 0, 0);
        if (S + Q - 1 > T.min_len || (I.gram_run && (S != 1 || Q != 16 || T.min_len < 19))) return fail("step", seed, 0, 0);
        for (size_t j = 0; j < pats.size(); j++) {
            const std::string &p = pats[j];
            for (uint32_t o = 0; o < (I.gram_run ? 4 : S); o++) {
                uint32_t x = 0;
                if (I.gram_q)
                    for (uint32_t i = 0; i < Q; i++) x |= (uint32_t)(((uint8_t)p[o + i] >> I.gram_sh) & 3) << (2 * i);
                else
                    std::memcpy(&x, p.data() + o, 4);
                const uint32_t h = (x & 0xffff) * kGramC0 + (x >> 16) * kGramC1;
                const uint32_t w = I.gram[(h >> (I.gram_run ? 2 : kGramShift)) & ((1u << I.gram_lw) - 1)];
                if (!((w >> (x & 31)) & 1) || (!I.gram_run && !((w >> (h & 31)) & 1))) return fail("bitmap", seed, j, o);
                if (o >= S) continue;
                const uint32_t g = x * kPfx4Mul;
                const uint16_t *bk = &I.gfp[16 * (size_t)(g >> (32 - I.gfp_lb))];
                const uint32_t fp = (g >> (20 - I.gfp_lb)) & 0xfff;
                uint32_t slot = 14;
                for (uint32_t i = 0; i < 14; i++)
                    if (bk[i] == (fp << 4 | i)) slot = i;
                if (slot == 14) return fail("slot", seed, j, o);
                const size_t at = 4 * ((size_t)(bk[14] | (uint32_t)bk[15] << 16) + slot);
                if (at + 4 > I.grec.size()) return fail("record number", seed, j, o);
                const uint32_t *rec = &I.grec[at];
                if (rec[0] == kNone) {
                    if (!(rec[1] >> o & 1)) return fail("offsets", seed, j, o);
                } else if (rec[0] == kGramNode) {
                    // the node's prefix is the pattern's (another pattern may
                    // have the gram at another offset only with a record of its own)
                    const uint32_t ro = rec[1] & 3, d = rec[1] >> 8;
                    if (ro != o || d != o + Q || rec[2] + 20 > I.gpat.size()) return fail("node", seed, j, o);
                    if (std::memcmp(&I.gpat[rec[2]], p.data(), d)) return fail("node's prefix", seed, j, o);
                    if (rec[3] < T.level_start[d] || rec[3] >= T.level_start[d + 1]) return fail("node's depth", seed, j, o);
                } else {
                    const uint32_t len = rec[1] & 0xffff;
                    if ((rec[1] >> 16 & 3) != o || len != p.size()) return fail("string", seed, j, o);
                    if (rec[0] + (size_t)(len + 63) / 64 * 64 > I.gpat.size()) return fail("string's end", seed, j, o);
                    if (std::memcmp(&I.gpat[rec[0]], p.data(), len)) return fail("string's bytes", seed, j, o);
                    if (!(rec[1] >> 18)) return fail("ids", seed, j, o);
                    if ((rec[2] & kGramId) && pats[rec[2] & ~kGramId] != p) return fail("id", seed, j, o);
                }
                if (I.gram_q) continue;
                auto begins = [&](uint32_t y) {
                    const uint32_t e = I.gper[y * kPfx4Mul >> (32 - I.gper_lw)];
                    return (e >> ((y * kPfx4Mul >> 5) & 31)) & (e >> (y >> 27)) & 1;
                };
                uint32_t first;
                std::memcpy(&first, p.data(), 4);
                if (!begins(first)) return fail("first bytes", seed, j, o);
                for (uint32_t q = 0, z = I.gram_alph; q < 4; q++, z = z << 8 | z >> 24)
                    if (begins(z)) return fail("dword that begins nothing", seed, j, o);
            }
        }
        if (I.gram_q)
            for (const char c : data)
                if ((uint8_t)(I.gram_alph >> (8 * (((uint8_t)c >> I.gram_sh) & 3))) != (uint8_t)c)
                    return fail("alphabet", seed, 0, 0);
    }
    std::printf("gram sanitizer run: ok, %u sets (%u, %u and %u with S 1, 2 and 4, %u with runs)\n", with, by_s[1], by_s[2],
                by_s[4], runs);
    return with > 120 && by_s[1] && by_s[2] && by_s[4] && runs ? 0 : 1;
}
