// Helpers of the C-ABI layer shared by its source files: error reporting
// and parameter validation (defined in ebsd_api.hip).
#pragma once

#include "../../include/ebsd_tm.h"
#include "ebsd_internal.hpp"

#include <hip/hip_runtime.h>

#include <string>
#include <vector>

namespace ebsd {
namespace api {

extern thread_local std::string g_last_error;
int fail(int code, const char* msg);
int fail_hip(hipError_t e, const char* where);
int resolve_params(const ebsd_params* in, int n, ebsd_params* out);
FilterParams filter_of(const ebsd_params& p, int n);
int check_master(const ebsd_master* mp);
int check_geometry(const ebsd_geometry* geo);
int64_t spec_complex(int n);
int f32_images_only(const ebsd_params& p);

// Where an entry point's device scratch comes from.
class ScratchSource {
 public:
  virtual ~ScratchSource() = default;
  virtual void* raw(size_t bytes, hipError_t* err) = 0;
  template <class T>
  T* get(size_t count, hipError_t* err) {
    return static_cast<T*>(raw((count ? count : 1) * sizeof(T), err));
  }
};

// Scratch allocated in stream order on the caller's stream and released in
// stream order when the call returns; the device memory pool keeps it for
// the next call, so repeated calls do not reach the kernel-mode allocator
// (after a synchronisation, which gives free memory back, a block is mapped
// again: 25 us for 16 MB, 60 for 256 MB).
// Small buffers share blocks of 1 MiB: a call on a few patterns takes one to
// three allocations instead of eight to thirteen (an allocation and its
// release cost the host about 5 us together, as much as a launch).
class Scratch : public ScratchSource {
 public:
  explicit Scratch(hipStream_t s) : stream_(s) {}
  Scratch(const Scratch&) = delete;
  Scratch& operator=(const Scratch&) = delete;
  ~Scratch() override {
    for (void* p : ptrs_) (void)hipFreeAsync(p, stream_);
  }
  void* raw(size_t bytes, hipError_t* err) override {
    *err = hipSuccess;
    const size_t need = (bytes + 255) & ~size_t(255);
    if (need < bytes) {
      *err = hipErrorOutOfMemory;
      return nullptr;
    }
    if (need <= left_) {
      void* p = at_;
      at_ += need;
      left_ -= need;
      return p;
    }
    const size_t block = need < kBlock ? kBlock : need;
    void* p = nullptr;
    *err = hipMallocAsync(&p, block, stream_);
    if (*err != hipSuccess) return nullptr;
    ptrs_.push_back(p);
    if (block - need > left_) {
      at_ = static_cast<char*>(p) + need;
      left_ = block - need;
    }
    return p;
  }

 private:
  static constexpr size_t kBlock = size_t(1) << 20;
  hipStream_t stream_;
  char* at_ = nullptr;
  size_t left_ = 0;
  std::vector<void*> ptrs_;
};

}  // namespace api
}  // namespace ebsd
