// The members of a team never outnumber the compute units, whatever the mesh and the device.
#include <cstdio>

#include "team_host.hpp"

using namespace shell;

int main() {
    for (int cus : {1, 4, 8, 32, 33, 38, 64, 80, 128, 256, 304})
        for (int64_t nv = 1; nv < 2000000; nv += nv < 20000 ? 1 : 997)
            for (int64_t rows : {team_rows(nv, cus), team_rows_membrane(nv, cus)}) {
                const int64_t members = (nv + rows - 1) / rows;
                if (rows % 64 == 0 && members <= cus) continue;
                std::printf("%ld rows, %d units: %ld members of %ld rows\n", long(nv), cus, long(members), long(rows));
                return 1;
            }
    // a whole device keeps the measured deal
    if (team_rows(4225, 256) != 256 || team_rows(16384, 256) != 256 || team_rows(16385, 256) != 512 ||
        team_rows(1024, 256) != 1024 || team_rows(1048576, 256) != 4096 || team_rows_membrane(4096, 256) != 256)
        return 1;
    std::puts("ok");
}
