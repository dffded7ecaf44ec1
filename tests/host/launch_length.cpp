// How long a launch of a team keeps its units: iterations times what an iteration measured (us), by rows of a member.
#include <cstdio>

#include "team_host.hpp"

using namespace shell;

int main() {
    const struct {
        int rows;
        bool membrane;
        double us;
    } measured[] = {{256, false, 7.6}, {512, false, 11.5}, {1536, false, 23.1}, {2048, false, 26.9}, {3136, false, 34.0},
                    {4096, false, 42.0}, {256, true, 15.6}, {2048, true, 64.0}, {4096, true, 122.0}};
    for (const auto& m : measured)
        for (bool shared : {false, true}) {
            const double ms = 1e-3 * m.us * team_launch_iterations(m.rows, m.membrane, shared), want = shared ? 10 : 50;
            if (ms > 0.6 * want && ms < 1.3 * want) continue;
            std::printf("%d rows: %g ms\n", m.rows, ms);
            return 1;
        }
    TeamSlots s(256);
    if (s.shared()) return 1;
    {
        TeamLease one(s, 1), two;
        if (!s.shared()) return 1;
    }
    if (s.shared()) return 1;
    std::puts("ok");
}
