// The pinned buffers of host transfers (daic_stage.h).
#include "daic_stage.h"

#include <mutex>

namespace daic {

namespace {
struct Blocks {  // those not in use
  char* block[kStageKept];
  uint32_t count = 0;
};
std::mutex g_lock;
uint32_t g_users = 0;
Blocks g_blocks[3];  // of each size
}  // namespace

StageUser::StageUser() {
  std::lock_guard<std::mutex> l(g_lock);
  ++g_users;
}

// (Transfers are made with a handle, so every block is back.)
StageUser::~StageUser() {
  std::lock_guard<std::mutex> l(g_lock);
  if (--g_users) return;
  for (Blocks& b : g_blocks)
    while (b.count) (void)hipHostFree(b.block[--b.count]);
}

char* stage_take(uint32_t size) {
  {
    std::lock_guard<std::mutex> l(g_lock);
    Blocks& b = g_blocks[size];
    if (b.count) return b.block[--b.count];
  }
  void* p = nullptr;
  if (hipHostMalloc(&p, kStageChunk * kStageBlocks[size], hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return static_cast<char*>(p);
}

void stage_give(char* block, uint32_t size) {
  {
    std::lock_guard<std::mutex> l(g_lock);
    Blocks& b = g_blocks[size];
    if (b.count < kStageKept) {
      b.block[b.count++] = block;
      return;
    }
  }
  (void)hipHostFree(block);
}

}  // namespace daic
