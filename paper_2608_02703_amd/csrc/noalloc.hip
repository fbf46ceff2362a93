// archead_logits_noalloc: archead_logits for callers that cannot allocate
// device memory (code under HIP graph capture, tight serving loops,
// harnesses that forbid allocation).  The call's workspace is a fixed
// device array of this library, so the call itself allocates nothing.
//
// The arrays are file-scope __device__ objects: in host code their names are
// host-side stand-ins, not device addresses.  Their device addresses are taken
// once per device with hipGetSymbolAddress, with that device current, when
// the first handle that may need them is created on it (archead_create calls
// scratch_setup), and only those addresses are passed to kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "archead.h"
#include "internal.h"

namespace {

constexpr int kMaxDevices = 64;

// The static workspaces of a device, held until the process ends.  Which calls
// are taken is decided by noalloc_bytes against ARCHEAD_NOALLOC_SCRATCH_BYTES;
// it leaves out the tiled kernel's scaled copy of x and its group sums.  The
// small array has room for those of a few hundred tokens beside it, the large
// one for those of every call taken on heads with groups of up to 128 (x's
// copy is at most 64 times the slot biases: 256 MiB); calls of larger groups
// that need more run in chunks of tokens (bit-identical: the split of stage 1
// along d is the whole call's).  The large one, which costs its memory and
// about 0.1 s when a process first creates such a handle, is there for heads
// small enough that their tables leave room for such calls.  In chunks that
// the small array holds, V = 2000, d = 8192, M = 5888 took 2005 us, 276 in one.
constexpr size_t kScratchBytes = size_t(ARCHEAD_NOALLOC_SCRATCH_BYTES) + (4u << 20);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_mu;
void* g_scratch[kMaxDevices];   // device address of `scratch` per device, or null
void* g_large[kMaxDevices];     // and of the large array

}  // namespace

namespace archead {

archead_status scratch_setup(const archead_handle* h) {
  const int device = h->device;
  if (device < 0 || device >= kMaxDevices)
    return fail(ARCHEAD_E_UNSUPPORTED, "device index %d out of range", device);
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_scratch[device]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(ARCHEAD_E_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    g_scratch[device] = p;
  }
  if (!g_large[device] && noalloc_wants(h, kScratchBytes)) {
    // (no memory for it is no reason to refuse the head: its calls then run in
    // chunks that the small array holds)
    void* p = nullptr;
    if (scratch_large(&p) == ARCHEAD_OK) g_large[device] = p;
    else (void)hipGetLastError();
  }
  return ARCHEAD_OK;
}

}  // namespace archead

using namespace archead;

extern "C" {

archead_status archead_logits_noalloc(const archead_handle* h, const void* x, int64_t M,
                                      int64_t ldx, void* out, archead_dtype out_dtype,
                                      int64_t ldo, void* stream) {
  clear_error();
  if (!h) return fail(ARCHEAD_E_INVALID_ARG, "handle is NULL");
  if (M < 0) return fail(ARCHEAD_E_INVALID_ARG, "M = %lld < 0", (long long)M);
  if (M == 0) return ARCHEAD_OK;
  const size_t need = noalloc_bytes(h, M);
  if (need > size_t(ARCHEAD_NOALLOC_SCRATCH_BYTES))
    return fail(ARCHEAD_E_WORKSPACE,
                "M = %lld needs %zu bytes of workspace; the static workspace holds %zu "
                "(use archead_logits with a caller workspace)",
                (long long)M, need, size_t(ARCHEAD_NOALLOC_SCRATCH_BYTES));
  void* ws = nullptr;
  size_t ws_bytes = kScratchBytes;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (h->device >= 0 && h->device < kMaxDevices) {
      ws = g_scratch[h->device];
      if (g_large[h->device] && noalloc_call_bytes(h, M) > kScratchBytes) {
        ws = g_large[h->device];
        ws_bytes = kScratchLargeBytes;
      }
    }
  }
  if (!ws) return fail(ARCHEAD_E_HIP, "static workspace of device %d is not set up", h->device);
  return logits_in_chunks(h, x, M, ldx, out, out_dtype, ldo, ws, ws_bytes, stream);
}

}  // extern "C"
