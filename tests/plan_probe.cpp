// Prints, for every line "kind rows d r V" of standard input (kind: low or full), what csrc/plan.hpp plans for one
// launch of that many rows.  Host arithmetic only; linked with the library for the rules it keeps in its sources.
#define __host__
#define __device__
#include "../paper_2605_10453_amd/csrc/plan.hpp"
#include <cstdio>
#include <cstring>

using namespace slimspec;

int main()
{
    char kind_name[16];
    int rows, d, r, V;
    while (std::scanf("%15s %d %d %d %d", kind_name, &rows, &d, &r, &V) == 5) {
        const HeadKind kind = std::strcmp(kind_name, "full") == 0 ? HeadKind::Full : HeadKind::LowRank;
        const MfmaPlan p = make_mfma_plan(kind, rows, d, r, V);
        std::printf("resident=%d rows_per_block=%d gw=%d nsr=%d\n", p.resident ? 1 : 0, p.rt, p.gw, p.nsr);
    }
    return 0;
}
