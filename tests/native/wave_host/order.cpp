// The order in which the host model takes waves and workgroups, and what a
// call launches.
#include <hip/hip_runtime.h>

extern "C" void wave_host_order(int waves_descend, int groups_descend) {
  wave_host::waves_descend = waves_descend;
  wave_host::groups_descend = groups_descend;
}

// Launches counted but not run (nothing else than the dispatch), or run again.
extern "C" void wave_host_dry(int dry) {
  wave_host::max_groups = dry ? 0u : ~0u;
  wave_host::launches = wave_host::groups_launched = 0;
}
extern "C" uint32_t wave_host_launches() { return wave_host::launches; }
extern "C" uint32_t wave_host_groups() { return wave_host::groups_launched; }
extern "C" void *wave_host_last_kernel() { return wave_host::last_kernel; }
