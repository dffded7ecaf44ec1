// How teams (team.hpp) are dealt out on a device.  Plain host code, which any compiler takes.
#pragma once

#include <algorithm>
#include <cstdint>

namespace shell {

// Rows per member by the mesh's rows and the device's compute units: one member up to `alone` rows, then at least
// `least` rows each, and never more members than units, since all of them have to be resident together.
inline int64_t team_rows_spread(int64_t nv, int cus, int64_t alone, int64_t least) {
    auto whole = [](int64_t n) { return (n + 63) / 64 * 64; };
    return nv <= alone ? whole(nv) : std::max(least, whole((nv + cus - 1) / cus));
}

// Rows per member of a bending simulation on its own.  One member up to 1024 rows (no meetings: 6.8 us per iteration
// against 7.5 with two members of 512); then few rows each, since an iteration's product is a chain of
// latencies that grows with a member's rows: 256 while one wave can read all members' sums (4225 rows: 7.6 us
// against 8.5 with 512 and 10.5 with 1024), 512 up to as many members as compute units (32761 rows: 9.5 us
// against 10.4 with 256), beyond that whatever keeps one member per unit.
inline int64_t team_rows(int64_t nv, int cus) {
    const int64_t wave = std::min<int64_t>(64, cus);
    if (nv > 1024 && nv <= wave * 256) return 256;
    return team_rows_spread(nv, cus, 1024, 512);
}

// Rows per member with the membrane: one member up to 512, then as many members as compute units, of at least 256 rows
// (an iteration reads four times the matrix of the bending solve, so the rows are dealt out sooner: 65536 rows 15.6
// us with 256, 16.2 with 512; 128 rows gain 8% at 1089 and lose 10% at 16384).
inline int64_t team_rows_membrane(int64_t nv, int cus) { return team_rows_spread(nv, cus, 512, 256); }

}  // namespace shell
