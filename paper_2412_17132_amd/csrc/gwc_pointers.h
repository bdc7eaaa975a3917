// Which of a caller's arrays kernels may read and write where they are.
#pragma once

namespace gwc {

// What the runtime reports of a pointer.
struct PointerKind {
  bool device = false;   // device memory (hipMemoryTypeDevice)
  bool managed = false;  // may move between the host and the devices
  int owner = -1;        // the device that holds it
};

// Only memory of the device that the call runs on: another device's memory may
// have no peer mapping (a kernel that touches it then faults, a copy does not),
// and managed memory would be migrated or read over the bus at every access.
// Anything else is copied.
inline bool kernels_may_use(const PointerKind &k, int current_device) {
  return k.device && !k.managed && k.owner == current_device;
}

}  // namespace gwc
