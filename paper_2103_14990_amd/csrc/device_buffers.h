// Device memory of an engine, and the building of its optional forms.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <new>
#include <string>
#include <vector>

#include "dlmpc.h"

namespace dlmpc {

// Device buffers freed together.
class DeviceBuffers {
 public:
  DeviceBuffers() = default;
  DeviceBuffers(const DeviceBuffers &) = delete;
  DeviceBuffers &operator=(const DeviceBuffers &) = delete;
  ~DeviceBuffers() { give_back(); }

  template <typename U>
  int alloc(U **dst, size_t n, std::string &err) {
    const size_t bytes = std::max<size_t>(n, 1) * sizeof(U);
    p_.push_back(nullptr);
    if (hipMalloc(&p_.back(), bytes) != hipSuccess) {
      p_.pop_back();
      err = "hipMalloc of " + std::to_string(bytes) + " bytes failed";
      return DLMPC_ENOMEM;
    }
    *dst = static_cast<U *>(p_.back());
    return DLMPC_OK;
  }

  void give_back() {
    for (void *p : p_) (void)hipFree(p);
    p_.clear();
  }

 private:
  std::vector<void *> p_;
};

// Builds an optional form of an engine, whose device buffers are all in `mem`. Without device or host
// memory for it the form is left out (*have = false), and whatever it had taken is given back, so that
// the allocations after it meet the memory they would have met without the attempt. Other failures
// are returned.
template <class F>
int build_optional(DeviceBuffers &mem, F build, bool *have, std::string &err) {
  int rc;
  try {
    rc = build();
  } catch (const std::bad_alloc &) {
    rc = DLMPC_ENOMEM;
  }
  *have = rc == DLMPC_OK;
  if (rc) mem.give_back();
  if (rc == DLMPC_ENOMEM) {
    (void)hipGetLastError();
    err.clear();
    rc = DLMPC_OK;
  }
  return rc;
}

}  // namespace dlmpc
