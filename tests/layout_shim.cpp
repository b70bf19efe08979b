// Host build of the item-sizing rules in csrc/vp_layout.h, for the CPU tests of the host logic
// (the same inline functions run in the planning kernels and in the host API).
#define __host__
#define __device__
#include "vp_layout.h"

extern "C" int shim_tiles_per_wave(long long total_tiles, int target_items, int min_items)
{
    return vp_tiles_per_wave(total_tiles, target_items, min_items);
}

extern "C" int shim_tiles_per_wave_units(long long total_tiles, int units, int target_items, int min_items)
{
    return vp_tiles_per_wave_units(total_tiles, units, target_items, min_items);
}

extern "C" int shim_raw_tiles(void) { return VP_RAW_TILES; }
extern "C" int shim_partial_floats(int k) { return vp_partial_floats(k); }

extern "C" int shim_item_of_workgroup(int wg, int total_items, int swz_rgs, int swz_chunks)
{
    return vp_item_of_workgroup(wg, total_items, swz_rgs, swz_chunks);
}
extern "C" int shim_xcd_block_items(void) { return VP_XCD_BLOCK_ITEMS; }
extern "C" int shim_rounds_item_count(int rgs, int slots, int vtiles) { return vp_rounds_item_count(rgs, slots, vtiles); }
extern "C" int shim_item_of_workgroup_even(int wg, int total_items) { return vp_item_of_workgroup_even(wg, total_items); }
extern "C" int shim_swept_item_count(int rgs, int slots, int vtiles, int kt, int max_items)
{
    return vp_swept_item_count(rgs, slots, vtiles, kt, max_items);
}
extern "C" int shim_sums_begin_anew(uint32_t events, int64_t n) { return vp_sums_begin_anew(events, n); }
extern "C" int shim_km_exact_entries(void) { return VP_KM_EXACT_ENTRIES; }
extern "C" long long shim_set_bounds_at(int N) { return vp_set_bounds_at(N); }
extern "C" long long shim_rows_head_bytes(int N) { return vp_rows_head_bytes(N); }
extern "C" int shim_floors_at(void) { return VP_FLOORS_AT; }
extern "C" int shim_bound_sets(void) { return VP_BOUND_SETS; }
extern "C" int shim_step_groups(int kt, int k, int shared, int ntiles, int trades) { return vp_step_groups(kt, k, shared != 0, ntiles, trades != 0); }
extern "C" int shim_trades_sets(int kt, int k, int N, int slots, int ntiles, int ncand) { return vp_trades_sets(kt, k, N, slots, ntiles, ncand); }
