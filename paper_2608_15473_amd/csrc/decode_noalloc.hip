// Fixed device scratch for the allocation-free decode (qf_attn_decode_noalloc).
//
// The decode keeps the partial states of every (shard, chunk) slot in device memory beyond its inputs
// and outputs.  For callers that cannot allocate (graph capture, serving loops, harnesses that forbid
// hipMalloc) that memory is this file-scope array: every GPU the library runs on holds its own copy
// for the life of the process.  Host code never passes the array's name to a kernel (on the host it is
// only a stand-in for the symbol); the device address of each GPU's copy is looked up once per device
// with hipGetSymbolAddress and kept, and only that address is used.
//
// The decode here is the sweep's launch and the merge's.  One launch whose last workgroup of a
// (request, KV head) merges needs arrival counters, which this array cannot be trusted to hold at zero
// (calls may have raced on it), so a kernel cleared them first: two launches as well, of which the
// fused one waits for every workgroup's stores and counts them.  Measured in a HIP graph, 4 ragged
// requests of up to 5,987 positions at G = 4: 19.6 -> 17.2 us a layer.
#include <atomic>
#include <mutex>

#include "qf_internal.h"
#include "qfattn.h"

static_assert(QF_NOALLOC_STATE_BYTES == qf::kNoallocStateBytes &&
                  QF_NOALLOC_STATE_BYTES <= QF_NOALLOC_SCRATCH_BYTES,
              "state bytes of the header");
static_assert(QF_NOALLOC_MAX_GROUPS == qf::kNoallocMaxGroups, "groups of the header");

static __device__ __align__(256) unsigned char scratch[qf::kNoallocStateBytes];

namespace qf {
namespace {

constexpr int kMaxDevices = 64;
std::atomic<unsigned char*> g_scratch[kMaxDevices];
std::mutex g_setup;

}  // namespace

hipError_t noalloc_states(void** states) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  unsigned char* base = g_scratch[dev].load(std::memory_order_acquire);
  if (!base) {
    // Set-up, once per device, with that device current: its copy's address.
    std::lock_guard<std::mutex> lock(g_setup);
    base = g_scratch[dev].load(std::memory_order_relaxed);
    if (!base) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return e;
      if (!p) return hipErrorInvalidSymbol;
      base = static_cast<unsigned char*>(p);
      g_scratch[dev].store(base, std::memory_order_release);
    }
  }
  *states = base;
  return hipSuccess;
}

}  // namespace qf
