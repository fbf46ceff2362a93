// The large static workspace of archead_logits_noalloc: its own code object,
// which the runtime loads (and gives its memory) when the address is first
// taken.
#include <hip/hip_runtime.h>

#include "archead.h"
#include "internal.h"

static __device__ __align__(256) unsigned char scratch_l[archead::kScratchLargeBytes];

namespace archead {

archead_status scratch_large(void** p) {
  *p = nullptr;
  const hipError_t e = hipGetSymbolAddress(p, HIP_SYMBOL(scratch_l));
  return e == hipSuccess && *p ? ARCHEAD_OK : ARCHEAD_E_HIP;
}

}  // namespace archead
