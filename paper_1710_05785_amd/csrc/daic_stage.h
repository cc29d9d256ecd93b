// Transfers between host arrays and device state through pinned memory.
//
// The state of a problem and the arrays of a caller have different element
// types and layouts (FP32 v minus its compensation against doubles, 64-wide
// rows against rows of the right-hand sides in use), and the caller's arrays
// are pageable and often fresh. A kernel converts between the state and a
// pinned chunk, which it reads or writes over the bus, and host threads copy
// between their chunks and the caller's array, two chunks in turn each, so
// that bus, copies and page faults overlap. (Copies to pageable memory with a
// conversion loop on one core before: the ranks of RMAT-24, 134 MB of doubles,
// read in 42 ms, a batch of 120,000 x 64 set in 8.8 and read in 11.6 ms; now
// 3.6, 5.1 and 4.5 ms. 1,000 distances: 35 us, now 16.)
// A transfer of one chunk stays on the calling thread.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <thread>
#include <vector>

#include "daic_internal.h"

namespace daic {

constexpr size_t kStageChunk = 1u << 20;   // bytes of a chunk
constexpr uint32_t kStageThreads = 8;      // host threads of a transfer at most
constexpr uint32_t kStageBuffers = 2;      // chunks of each in turn
// Arrays of these sizes that need no conversion are written by a plain copy:
// each of v and dv with 64 KiB of doubles 12 us, 16 through the chunks; 1 MiB
// 42 and 52; 8 MiB 240 and 285; 16 MiB 515 and 515; 32 MiB 1,050 and 910. 4 KiB
// take 14 us either way, but the first kernel after such a copy 9 more. (Reads
// are faster through the chunks: 4 KiB 15 us against 30, 4 MiB 190 against 260.)
constexpr size_t kStageSmallWrite = 16u << 10, kStageLargeWrite = 12u << 20;

// The process's pinned buffers, in blocks: one chunk, and kStageBuffers for
// each of two or of kStageThreads threads (16 MiB; 30 us to allocate, 0.1 ms to
// free; as sixteen of 1 MiB 0.5 and 2 ms). They exist while problems or batches
// do (their StageUser); kStageKept of each size are kept between transfers. A
// transfer holds a block of its own and waits for no other (a lock held during
// transfers had a read of 8 KB take 5.3 ms beside reads of 268 MB that took
// 6.3); beyond those kept, it allocates and frees one.
// stage_take returns null when pinned memory is not to be had.
constexpr uint32_t kStageKept = 2;
constexpr uint32_t kStageBlocks[3] = {1, 2 * kStageBuffers, kStageThreads * kStageBuffers};  // chunks
char* stage_take(uint32_t size);
void stage_give(char* block, uint32_t size);

// One thread's share of a transfer: chunks t, t + T, ...
template <bool OUT, typename Enqueue>
hipError_t stage_share(char* buf, char* host, uint64_t count, size_t elem, uint64_t per, uint32_t t, uint32_t T,
                       hipStream_t s, const Enqueue& enqueue) {
  const uint64_t chunks = (count + per - 1) / per;
  hipEvent_t ev[kStageBuffers] = {};
  hipError_t e = hipSuccess;
  for (uint32_t k = 0; k < kStageBuffers && e == hipSuccess; ++k)
    e = hipEventCreateWithFlags(&ev[k], hipEventDisableTiming);
  auto at = [&](uint64_t c) { return std::min(count, c * per); };
  auto run = [&](uint64_t c, uint32_t k) {
    enqueue(buf + k * kStageChunk, at(c), at(c + 1) - at(c));
    hipError_t x = hipGetLastError();
    return x == hipSuccess ? hipEventRecord(ev[k], s) : x;
  };
  auto copy = [&](uint64_t c, uint32_t k) {
    char* h = host + at(c) * elem;
    const size_t bytes = (at(c + 1) - at(c)) * elem;
    if (OUT) std::memcpy(h, buf + k * kStageChunk, bytes);
    else std::memcpy(buf + k * kStageChunk, h, bytes);
  };
  uint32_t k = 0;
  if (OUT) {
    if (e == hipSuccess && t < chunks) e = run(t, 0);
    for (uint64_t c = t; c < chunks && e == hipSuccess; c += T, k ^= 1) {
      if (c + T < chunks) e = run(c + T, k ^ 1);
      if (e == hipSuccess) e = hipEventSynchronize(ev[k]);
      if (e == hipSuccess) copy(c, k);
    }
  } else {
    for (uint64_t c = t; c < chunks && e == hipSuccess; c += T, k ^= 1) {
      if (c >= t + 2 * (uint64_t)T) e = hipEventSynchronize(ev[k]);  // the buffer's last chunk was read
      if (e == hipSuccess) {
        copy(c, k);
        e = run(c, k);
      }
    }
  }
  for (uint32_t i = 0; i < kStageBuffers; ++i) {  // nothing of this thread's is in flight after it
    if (ev[i] && e == hipSuccess) e = hipEventSynchronize(ev[i]);
    if (ev[i]) (void)hipEventDestroy(ev[i]);
  }
  if (e != hipSuccess) (void)hipStreamSynchronize(s);
  return e;
}

// count elements of `elem` bytes between a host array and the device:
// enqueue(chunk, first, n) launches the kernel that writes (OUT) or reads n
// elements of the chunk, for the array's elements [first, first + n), on s.
// Returns when the transfer is complete.
template <bool OUT, typename Enqueue>
daic_status stage_move(void* host, uint64_t count, size_t elem, hipStream_t s, const Enqueue& enqueue) {
  if (count == 0) return DAIC_OK;
  char* h = static_cast<char*>(host);
  const uint64_t per = kStageChunk / elem, chunks = (count + per - 1) / per;
  const uint32_t size = chunks == 1 ? 0 : chunks / 2 <= 2 ? 1 : 2;
  char* buf = stage_take(size);
  hipError_t e = hipSuccess;
  if (!buf) {  // no pinned memory: a device chunk and plain copies
    void* d = nullptr;
    e = hipMalloc(&d, kStageChunk);
    for (uint64_t i = 0; i < count && e == hipSuccess; i += per) {
      const uint64_t n = std::min(per, count - i);
      if (!OUT) e = hipMemcpy(d, h + i * elem, n * elem, hipMemcpyHostToDevice);
      if (e == hipSuccess) enqueue(d, i, n);
      if (e == hipSuccess) e = hipGetLastError();
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      if (OUT && e == hipSuccess) e = hipMemcpy(h + i * elem, d, n * elem, hipMemcpyDeviceToHost);
    }
    if (d) (void)hipFree(d);
  } else if (chunks == 1) {
    if (!OUT) std::memcpy(buf, h, count * elem);
    enqueue(buf, 0, count);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (OUT && e == hipSuccess) std::memcpy(h, buf, count * elem);
  } else {
    const uint32_t T = (uint32_t)std::min<uint64_t>(
        {kStageThreads, std::max(1u, std::thread::hardware_concurrency()), chunks / 2});
    int device = 0;
    e = hipGetDevice(&device);
    hipError_t got[kStageThreads] = {};
    auto share = [&](uint32_t t) {
      got[t] = t ? hipSetDevice(device) : hipSuccess;
      if (got[t] == hipSuccess)
        got[t] = stage_share<OUT>(buf + (size_t)t * kStageBuffers * kStageChunk, h, count, elem, per, t, T, s, enqueue);
    };
    std::thread pool[kStageThreads];
    bool mine[kStageThreads] = {true};
    for (uint32_t t = 1; t < T && e == hipSuccess; ++t) {
      try {
        pool[t] = std::thread(share, t);
      } catch (...) {
        mine[t] = true;  // no thread to be had: its share after this thread's own
      }
    }
    for (uint32_t t = 0; t < T && e == hipSuccess; ++t)
      if (mine[t]) share(t);
    for (uint32_t t = 1; t < T; ++t)
      if (pool[t].joinable()) pool[t].join();
    for (uint32_t t = 0; t < T && e == hipSuccess; ++t) e = got[t];
  }
  if (buf) stage_give(buf, size);
  if (e != hipSuccess)
    return fail(e == hipErrorOutOfMemory ? DAIC_E_OOM : DAIC_E_DEVICE, "host transfer: %s", hipGetErrorString(e));
  return DAIC_OK;
}

// ---- kernels: state <-> chunk -------------------------------------------------
inline dim3 stage_grid(uint64_t n) {
  return dim3((uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((n + 255) / 256, 1024)));
}

// out[i] = a[first + i] (minus c[first + i] when given), converted.
template <typename From, typename To>
__global__ void k_stage_out(const From* a, const From* c, uint64_t first, uint64_t n, To* out) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    To x = (To)a[first + i];
    if (c) x -= (To)c[first + i];
    out[i] = x;
  }
}

// a[first + i] = in[i], converted; c (when given) takes the rounding of it.
template <typename From, typename To>
__global__ void k_stage_in(const From* in, uint64_t first, uint64_t n, To* a, To* c) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    const From x = in[i];
    const To y = (To)x;
    a[first + i] = y;
    if (c) c[first + i] = (To)((From)y - x);
  }
}

}  // namespace daic
