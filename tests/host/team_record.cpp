// How long a handle's solves keep to the chain after teams that gave up.
#include <cstdio>

#include "team_host.hpp"

using namespace shell;

static int chain_solves(TeamRecord& r) {
    int n = 0;
    while (r.rests()) ++n;
    return n;
}

int main() {
    TeamRecord r;
    if (chain_solves(r) != 0) return 1;
    for (int want : {16, 32, 64, 128, 256, 512, 1024, 1024}) {
        r.gave_up();
        const int n = chain_solves(r);
        if (n == want) continue;
        std::printf("%d solves of the chain, not %d\n", n, want);
        return 1;
    }
    r.met();
    if (chain_solves(r) != 0) return 1;
    r.gave_up();
    if (chain_solves(r) != 16) return 1;
    std::puts("ok");
}
