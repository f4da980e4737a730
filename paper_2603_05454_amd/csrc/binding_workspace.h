// Workspace of one attention call made through the binding.
#pragma once
#include <ATen/core/Tensor.h>
#include <c10/core/Allocator.h>
#include <c10/util/Exception.h>

// The caller's, where it will do (contiguous, of so many bytes, aligned to 16).  Otherwise one of the call's own, memory of the current
// stream: the allocator hands it out again only behind the launch, so that calls on several streams and threads cannot meet in it.
// Neither where memory has run out: the call goes without.
struct Workspace {
  c10::DataPtr own;
  void *at = nullptr;
  size_t bytes = 0;
  Workspace(size_t need, const at::Tensor *given) {
    if (need == 0) return;
    if (given && given->is_contiguous() && given->nbytes() >= need) {
      void *p = given->mutable_data_ptr();
      if (reinterpret_cast<uintptr_t>(p) % 16 == 0) {
        at = p;
        bytes = need;
        return;
      }
    }
    try {
      own = c10::GetAllocator(c10::DeviceType::CUDA)->allocate(need);
      at = own.get();
      bytes = need;
    } catch (const c10::OutOfMemoryError &) {
    }
  }
};
