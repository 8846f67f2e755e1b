#include "common.h"
#include "wavealign.h"

#include <mutex>

// Scheduler state of the attention entry point that allocates nothing: a static device array of the
// library, one per GPU, held until the process ends. In a source of its own, since the runtime loads a source's device
// code, with its arrays, at its first use: beside the kernels, the 36 MiB were held by every process that
// called any of them. Host code never uses an array's name as an address: its device address is looked up once per
// device (with that device current) and cached.
static constexpr size_t kNoAllocInts = WA_NOALLOC_SCRATCH_BYTES / 4;
static __device__ __align__(256) int32_t scratch[kNoAllocInts];
// Its split rows (tasks, arrival counters and partial tiles) have an array of their own.
static constexpr size_t kNoAllocSplitInts = wa::kPartBytes / 4 + 65536;
static __device__ __align__(256) int32_t split_scratch[kNoAllocSplitInts];
static std::mutex g_scratch_mu;
static int32_t* g_scratch_ptr[64];
static int32_t* g_split_ptr[64];

hipError_t wa_noalloc_scratch(int32_t** ptr, size_t* bytes, int32_t** split, size_t* split_bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    void* sp = nullptr;
    e = hipGetSymbolAddress(&sp, HIP_SYMBOL(split_scratch));
    if (e != hipSuccess) return e;
    if (!sp) return hipErrorInvalidSymbol;
    g_split_ptr[dev] = (int32_t*)sp;
    g_scratch_ptr[dev] = (int32_t*)p;
  }
  *ptr = g_scratch_ptr[dev];
  *bytes = kNoAllocInts * 4;
  *split = g_split_ptr[dev];
  *split_bytes = kNoAllocSplitInts * 4;
  return hipSuccess;
}
