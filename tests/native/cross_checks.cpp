// Host-only checks of the words by which the tiles of a cluster meet, and of the
// two-orientation plans' maps at every size; built and run by tests/test_cross_host.py.
#include "qw_kernels.h"

#include <cstdio>
#include <cstdlib>

namespace qw {
void set_error(const std::string &) {}
}  // namespace qw

using namespace qw;

#define CHECK(cond, ...)               \
    do {                               \
        if (!(cond)) {                 \
            std::printf("FAIL %s: ", #cond); \
            std::printf(__VA_ARGS__);  \
            std::printf("\n");         \
            std::exit(1);              \
        }                              \
    } while (0)

static void words()
{
    for (int round : {1, 2, 3, 1000, 131072})
        for (int xcd = 0; xcd < 8; ++xcd) {
            const int word = round * 16 + xcd;
            CHECK(cross_state(word, word) == CROSS_MET, "word %d", word);
            CHECK(cross_state(0, word) == CROSS_NOT_YET, "cleared, word %d", word);
            for (int other = 0; other < 8; ++other) {
                CHECK(cross_state((round - 1) * 16 + other, word) == CROSS_NOT_YET, "the round before, word %d", word);
                if (other != xcd) CHECK(cross_state(round * 16 + other, word) == CROSS_NEVER, "word %d, %d", word, other);
            }
        }
}

template <int XH> static uint64_t tile_of(uint32_t b, uint32_t nb, int shift) { return cross_tile<XH>(b, nb, shift); }

// Index maps are disjoint unions of bit fields, so bases and elements are checked
// apart: bases distinct and free of the element bits, elements a bijection of the rest.
template <typename R> static void maps(int n, bool tables, int K)
{
    const std::vector<OrientSpec> S = pair_plan<R>(n, tables, K);
    uint64_t covered = 0;
    for (const OrientSpec &o : S) {
        const PassPlan &p = o.pl;
        const int tb = p.L + p.h;
        CHECK(tb == o.fused.tb && tb == o.add.tb, "n %d: tile", n);
        const uint32_t ntiles = 1u << (n - tb);
        uint64_t elements = 0;
        for (uint32_t e = 0; e < (1u << tb); ++e) {
            const uint64_t i = tile_index(0, e, p.L, p.g0);
            CHECK(e == 0 || (i ^ tile_index(0, e & (e - 1), p.L, p.g0)) == tile_index(0, e & -e, p.L, p.g0), "n %d element %u", n, e);
            elements |= i;
        }
        CHECK(__builtin_popcountll(elements) == tb, "n %d: element bits", n);
        std::vector<uint8_t> seen(ntiles, 0);
        std::vector<uint32_t> block(ntiles);
        for (uint32_t b = 0; b < ntiles; ++b) {
            const int shift = p.g0 - p.L;
            const uint64_t t = o.xh == 0 ? (o.xcd ? xcd_tile(b, ntiles) : b)
                             : o.xh == 1 ? tile_of<1>(b, ntiles, shift) : o.xh == 2 ? tile_of<2>(b, ntiles, shift)
                             : o.xh == 3 ? tile_of<3>(b, ntiles, shift) : tile_of<4>(b, ntiles, shift);
            CHECK(t < ntiles && !seen[t], "n %d block %u", n, b);
            seen[t] = 1;
            block[t] = b;
            const uint64_t base = tile_base(t, p.L, p.g0, p.h);
            CHECK((base & elements) == 0 && base < (uint64_t(1) << n), "n %d tile %llu", n, (unsigned long long)t);
            for (int j = 0; j < o.xh; ++j)   // a partner's base differs in one cross bit
                CHECK((tile_base(t ^ (uint64_t(1) << (shift + j)), p.L, p.g0, p.h) ^ base) == uint64_t(1) << (p.g0 + p.h + j),
                      "n %d tile %llu", n, (unsigned long long)t);
        }
        // a cluster is the run of 2^xh neighbours in the launch order of one XCD
        for (uint32_t t = 0; t < ntiles && o.xh > 0; ++t)
            for (int j = 0; j < o.xh; ++j) {
                const uint32_t a = block[t], c = block[t ^ (1u << (p.g0 - p.L + j))];
                CHECK(a % 8 == c % 8 && (a / 8) >> o.xh == (c / 8) >> o.xh, "n %d tiles of blocks %u, %u", n, a, c);
            }
        for (int j = 0; j < p.h + o.xh; ++j) covered ^= uint64_t(1) << (p.g0 + j);
    }
    CHECK(S.empty() || covered == (uint64_t(1) << n) - 1, "n %d: bits", n);
    // four cross bits keep at most 15 CUs of an XCD's 32 waiting
    for (const OrientSpec &o : S) CHECK(o.xh <= 4, "n %d", n);
}

int main()
{
    words();
    for (int n = 1; n <= 32; ++n)
        for (bool tables : {false, true})
            for (int K : {1, 2, 100}) {
                maps<float>(n, tables, K);
                maps<double>(n, tables, K);
            }
    std::printf("CROSS OK\n");
    return 0;
}
