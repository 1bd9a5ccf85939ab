// The order in which the host model takes waves and workgroups.
#include <hip/hip_runtime.h>

extern "C" void wave_host_order(int waves_descend, int groups_descend) {
  wave_host::waves_descend = waves_descend;
  wave_host::groups_descend = groups_descend;
}
