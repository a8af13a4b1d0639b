// Where a caller's coefficient rows may be used in place (host code, no GPU types).
#pragma once
#include <cstdint>

namespace stern {

// Kernels load and store rows where they are only in memory of the system's own device, at addresses that
// 16-byte loads may use. Rows anywhere else (another device's memory, which this one need not be able to
// reach; pinned, managed or plain host memory given as device memory) go through a copy by the runtime, as
// does memory whose place the runtime does not know (device_memory false).
inline bool rows_in_place(bool device_memory, int mem_device, int sys_device, std::uintptr_t p) {
  return device_memory && mem_device == sys_device && (p & 15) == 0;
}

}  // namespace stern
