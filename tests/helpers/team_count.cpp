// Checks the launch-relative counts of a team's control words (team_count,
// team_counted) on the host: exit status 0, or a line per failure.
#include <cstdio>

#include "sca_internal.hpp"

using sca::team_count;
using sca::team_counted;

int main()
{
    int bad = 0;
    const auto expect = [&](uint64_t word, uint64_t epoch, uint32_t want) {
        const uint32_t got = team_counted(word, epoch);
        if (got == want) return;
        std::printf("word %016llx in launch %llx: %u, not %u\n", (unsigned long long)word, (unsigned long long)epoch, got, want);
        ++bad;
    };
    const uint32_t most = (1u << sca::kTeamCountBits) - 1u;
    // launches around every power of two, and what 2^30 and more MCS in launches
    // of their own, two half-steps each, bring them to
    for (int b = 0; b < 40; ++b)
        for (int64_t d = -1; d <= 1; ++d) {
            const uint64_t e = (uint64_t)(((int64_t)1 << b) + d);
            if (e == 0) continue;
            for (uint32_t n : {0u, 1u, 2u, 511u, 1u << 20, most}) {
                expect(team_count(e, n), e, n);
                expect(team_count(e, n), e + 1, 0);  // an earlier launch's count is none
                for (int s = 0; s < 40; ++s)         // however many launches lie between
                    if (e + ((uint64_t)1 << s) < (uint64_t)1 << 40) expect(team_count(e, n), e + ((uint64_t)1 << s), 0);
            }
            expect(0, e, 0);  // as sca_init leaves the word
        }
    return bad != 0;
}
