// The host-only rules of the library (tiles, plans) behind a C interface, for
// the tests that need no GPU.
#include "../paper_2109_07710_amd/csrc/plan.hpp"

extern "C" {

int probe_compact_list_cap() { return kCompactListCap; }

// blocks, share, begin, end, first, last
void probe_compact_share(int total, int nsplit, int z, int32_t* out)
{
    const CompactShare s = compact_share(total, nsplit, z);
    out[0] = s.blocks; out[1] = s.share; out[2] = s.begin; out[3] = s.end; out[4] = s.first; out[5] = s.last;
}

}  // extern "C"
