// Host-only checks of the words by which the tiles of a cluster meet; built and run
// by tests/test_cross_host.py.
#include "qw_kernels.h"

#include <cstdio>

namespace qw {
void set_error(const std::string &) {}
}  // namespace qw

using namespace qw;

int main()
{
    int bad = 0;
    auto expect = [&](int seen, int word, int want) {
        if (cross_state(seen, word) != want) {
            std::printf("seen %d word %d: %d\n", seen, word, cross_state(seen, word));
            ++bad;
        }
    };
    for (int round : {1, 2, 3, 1000, 131072})
        for (int xcd = 0; xcd < 8; ++xcd) {
            const int word = round * 16 + xcd;
            expect(word, word, CROSS_MET);
            expect(0, word, CROSS_NOT_YET);                      // cleared
            for (int other = 0; other < 8; ++other) {
                expect((round - 1) * 16 + other, word, CROSS_NOT_YET);   // the round before
                if (other != xcd) expect(round * 16 + other, word, CROSS_NEVER);
            }
        }
    std::printf(bad ? "FAIL\n" : "CROSS OK\n");
    return bad != 0;
}
