// Logit fidelity of the packed head against a dense bf16 head inside the
// head's V-tile pass (Section 4, "Logit Fidelity", Table 8): the tiled
// kernel's fidelity and rank variants and the per-token merge of the fidelity pass's tile statistics.
#include "dev_mfma.cuh"
#include "kernels.h"

namespace {

// One workgroup per token: the tiles' statistics, each thread its tiles in
// order, then a fixed tree (fp64 sums rescaled to the row maxima), giving
// KL(p_dense || p_packed), the summed squared logit error, the dense head's
// first argmax and the packed logit there; the rank is cleared for the rank
// pass, and the tiles marked that hold a packed logit ranked ahead of the one
// at the dense head's top-1 (their maximum is larger, or equal at a smaller
// index): only those does the rank pass compute again.  With one lane per
// token the 594 tiles of a 151936-row head took 397 us at 1024 tokens.
__global__ __launch_bounds__(kBlock) void k_fidh_merge(const FidTilePart* part, int64_t n_vt, int64_t M,
                                                       float* kl, float* sq, int64_t* ref_idx,
                                                       float* bref, int64_t* rank, int* need) {
  __shared__ float sma[kBlock], smb[kBlock], sbat[kBlock];
  __shared__ int64_t sia[kBlock];
  __shared__ double sd[4][kBlock];
  const int64_t m = blockIdx.x;
  const int tid = threadIdx.x;
  const FidTilePart* p = part + m * n_vt;
  constexpr int64_t kNone = int64_t(1) << 62;
  float ma = -INFINITY, mb = -INFINITY, bat = 0.f;
  int64_t ia = kNone;
  auto take = [&](float oma, int64_t oia, float obat, float omb) {
    if (oma > ma || (oma == ma && oia < ia)) {
      ma = oma;
      ia = oia;
      bat = obat;
    }
    mb = fmaxf(mb, omb);
  };
  for (int64_t c = tid; c < n_vt; c += kBlock) {
    const int col = p[c].iab & 0xffff;
    take(p[c].ma, col == kNoCol ? kNone : c * kTN + col, p[c].bat, p[c].mb);
  }
  sma[tid] = ma;
  smb[tid] = mb;
  sbat[tid] = bat;
  sia[tid] = ia;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (tid < s) {
      take(sma[tid + s], sia[tid + s], sbat[tid + s], smb[tid + s]);
      sma[tid] = ma;
      smb[tid] = mb;
      sbat[tid] = bat;
      sia[tid] = ia;
    }
    __syncthreads();
  }
  ma = sma[0];
  mb = smb[0];
  bat = sbat[0];
  ia = sia[0] == kNone ? 0 : sia[0];
  double sa = 0.0, sb = 0.0, t = 0.0, s2 = 0.0;
  int* const nd = need + m / 64 * n_vt;
  for (int64_t c = tid; c < n_vt; c += kBlock) {
    // a tile's sums were taken relative to its own maxima
    const FidTilePart q = p[c];
    const double fa = exp(double(q.ma) - double(ma));
    const double fb = exp(double(q.mb) - double(mb));
    sa += double(q.sa) * fa;
    t += double(q.t) * fa;
    sb += double(q.sb) * fb;
    s2 += double(q.sq);
    // (every token of the tile that needs it writes the same word)
    const int bcol = q.iab >> 16;   // kNoCol: every logit -inf (or NaN)
    if (q.mb > bat || (q.mb == bat && c * kTN + (bcol == kNoCol ? 0 : bcol) < ia)) nd[c] = 1;
  }
  sd[0][tid] = sa;
  sd[1][tid] = sb;
  sd[2][tid] = t;
  sd[3][tid] = s2;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (tid < s) {
#pragma unroll
      for (int k = 0; k < 4; ++k) sd[k][tid] += sd[k][tid + s];
    }
    __syncthreads();
  }
  if (tid) return;
  sa = sd[0][0];
  sb = sd[1][0];
  t = sd[2][0];
  // sum_v p (log p - log q) with log p = a - ma - ln sa and
  // log q = b - mb - ln sb: E_p[a - b] + (mb - ma) + ln(sb / sa)
  kl[m] = float(t / sa + (double(mb) - double(ma)) + (log(sb) - log(sa)));
  sq[m] = float(sd[3][0]);
  ref_idx[m] = ia;
  bref[m] = bat;
  rank[m] = 0;
}

}  // namespace

namespace archead {
namespace kern {

const void* mfma_fid(int tm) {
  return tm == 128 ? reinterpret_cast<const void*>(k_mfma<false, 128, 8, 1>)
                   : reinterpret_cast<const void*>(k_mfma<false, 64, 4, 1>);
}
const void* mfma_rank() { return reinterpret_cast<const void*>(k_mfma<false, 64, 4, 2>); }
const void* fid_head_merge() { return reinterpret_cast<const void*>(k_fidh_merge); }

}  // namespace kern
}  // namespace archead
