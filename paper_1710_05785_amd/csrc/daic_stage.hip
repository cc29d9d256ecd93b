// The pinned buffers of host transfers (daic_stage.h).
#include "daic_stage.h"

#include <mutex>

namespace daic {

namespace {
std::mutex g_life;      // users and the allocations
std::mutex g_transfer;  // held during a transfer
uint32_t g_users = 0;
char* g_one = nullptr;  // one chunk
char* g_all = nullptr;  // kStageThreads x kStageBuffers chunks
}  // namespace

StageUser::StageUser() {
  std::lock_guard<std::mutex> l(g_life);
  ++g_users;
}

StageUser::~StageUser() {
  std::lock_guard<std::mutex> l(g_life);
  if (--g_users) return;
  if (g_one) (void)hipHostFree(g_one);
  if (g_all) (void)hipHostFree(g_all);
  g_one = g_all = nullptr;
}

// The caller holds a handle, so the buffers stay until it is done.
char* stage_lock(uint64_t chunks) {
  g_transfer.lock();
  char** p = chunks > 1 ? &g_all : &g_one;
  {
    std::lock_guard<std::mutex> l(g_life);
    const size_t bytes = kStageChunk * (chunks > 1 ? kStageThreads * kStageBuffers : 1);
    if (!*p && hipHostMalloc((void**)p, bytes, hipHostMallocPortable) != hipSuccess) {
      (void)hipGetLastError();
      *p = nullptr;
    }
  }
  if (!*p) g_transfer.unlock();
  return *p;
}

void stage_unlock() { g_transfer.unlock(); }

}  // namespace daic
