// Workspaces that the library keeps between calls, one per (device, stream or other owner).  Host code only; the caller locks.
#pragma once
#include <cstddef>
#include <map>
#include <utility>
#include <vector>

namespace prism {

// Grow-only.  A block that has become too small is kept until everything is released: work enqueued earlier, and HIP graphs captured
// from earlier calls, still hold its address.
struct WorkspaceCache {
  struct Block {
    void* ptr = nullptr;
    size_t bytes = 0;
    size_t refused = 0;            // least size that could not be had for a call that can do with less (0: none)
    std::vector<void*> retired;
  };
  std::map<std::pair<int, const void*>, Block> blocks;

  // Null if there is no block of that size and alloc(bytes) has none either.  optional: the caller asks again for less.  A size that such a call did not
  // get is not asked for again, so that the same call, repeated or captured into a graph, finds what it settled for and allocates nothing.
  template <typename Alloc>
  void* get(int device, const void* owner, size_t bytes, bool optional, Alloc&& alloc) {
    Block& b = blocks[std::make_pair(device, owner)];
    if (b.bytes < bytes) {
      if (optional && b.refused && bytes >= b.refused) return nullptr;
      void* fresh = alloc(bytes);
      if (!fresh) {
        if (optional) b.refused = bytes;
        return nullptr;
      }
      if (b.ptr) b.retired.push_back(b.ptr);
      b.ptr = fresh;
      b.bytes = bytes;
    }
    return b.ptr;
  }
};

}  // namespace prism
