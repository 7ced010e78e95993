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

// tile channels, tile rows, groups, ptiles, ptaps, split, then the partial region's bytes
int probe_data_plan(const cbw_conv_desc* d, int masked, int64_t* out)
{
    cbw::DataPlan p;
    const int st = cbw::plan_data(d, masked != 0, &p);
    const int64_t v[] = {p.bm, p.brows, p.groups, p.ptiles, p.ptaps, p.split, (int64_t)p.partial.bytes};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
    return st;
}

// workgroups a split, chunks, splits
int probe_f32_weight_plan(const cbw_conv_desc* d, int64_t* out)
{
    cbw::WeightPlan p;
    const int st = cbw::plan_weight(d, &p, true);
    out[0] = (int64_t)p.tgroups * p.ctiles * p.ktiles * p.subc * p.subk;
    out[1] = p.nchunks;
    out[2] = p.nsplit;
    return st;
}

// fills the splits of `n` cases of (workgroups, chunks, limit)
void probe_f32_weight_splits(const cbw_conv_desc* d, int n, const int64_t* cases, int32_t* splits)
{
    for (int i = 0; i < n; ++i)
        splits[i] = cbw::f32_weight_splits(d, cases[3 * i], (int)cases[3 * i + 1], (int)cases[3 * i + 2]);
}

}  // extern "C"
