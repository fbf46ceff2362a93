// Top-k selection: the single-token decode GEMV with the fused top-k
// epilogue and the merge of its per-partial lists, and the top-k of rows of
// fp32 logits.  Every list is in the order of the first-index argmax (larger value
// first, equal values by smaller index), so the merged result is the first k
// entries of the stable descending sort of the token's logits.
#include "dev_gemv.cuh"
#include "kernels.h"

namespace {

using GemvFn = void (*)(GemvArgs);

template <bool SC8, int GEN>
GemvFn gemv_topk_by_lpr(int lpr) {
  if constexpr (GEN > 0) {
    switch (lpr) {
      case 8: return k_gemv<1, 8, false, SC8, GEN, true>;
      case 16: return k_gemv<1, 16, false, SC8, GEN, true>;
      default: return nullptr;
    }
  } else {
    switch (lpr) {
      case 1: return k_gemv<1, 1, false, SC8, GEN, true>;
      case 2: return k_gemv<1, 2, false, SC8, GEN, true>;
      case 4: return k_gemv<1, 4, false, SC8, GEN, true>;
      case 8: return k_gemv<1, 8, false, SC8, GEN, true>;
      case 16: return k_gemv<1, 16, false, SC8, GEN, true>;
      case 32: return k_gemv<1, 32, false, SC8, GEN, true>;
      default: return k_gemv<1, 64, false, SC8, GEN, true>;
    }
  }
}

template <int GEN>
const void* gemv_topk_fn(int lpr, bool sc8) {
  GemvFn fn = sc8 ? gemv_topk_by_lpr<true, GEN>(lpr) : gemv_topk_by_lpr<false, GEN>(lpr);
  return reinterpret_cast<const void*>(fn);
}

__device__ __forceinline__ void tk_pick(float& bv, int& bi, float ov, int oi) {
  const bool t = tk_better(ov, oi, bv, bi);
  bv = t ? ov : bv;
  bi = t ? oi : bi;
}
template <int CTRL>
__device__ __forceinline__ void tk_pick_dpp(float& v, int& i) {
  const float ov = dpp_swap<CTRL>(v);
  const int oi = __builtin_amdgcn_update_dpp(0, i, CTRL, 0xF, 0xF, false);
  tk_pick(v, i, ov, oi);
}
// the best pair of each row of 16 lanes, in every lane of the row
__device__ __forceinline__ void tk_row16_best(float& v, int& i) {
  tk_pick_dpp<0xB1>(v, i);
  tk_pick_dpp<0x4E>(v, i);
  tk_pick_dpp<0x141>(v, i);
  tk_pick_dpp<0x140>(v, i);
}

// ------------------------------------------------ top-k of rows of logits
// Two launches.  k_topk_max writes the largest logit of every chunk of a row
// (as an order key); the k-th largest of a row's chunk maxima is a floor for
// its k-th largest logit, so k_topk_select reads again only the chunks whose
// maximum reaches the floor (k of them, but for ties) and ranks the few logits
// at or above it.  Of chunks whose maxima are equal it reads no more than can be
// wanted, and a row with many logits at or above the floor (few chunks, equal or
// sorted logits) is reduced to its k best by counting first, so no values make
// it slow.  What bounds it: the first launch reads the logits once, from
// the caches for the usual sizes; the second is a chain of short steps of one
// workgroup per token.  24 tokens of 128256 logits, k = 50: 5.5 + 9.3 us
// (sorted lists per slice and a merge in k rounds: 61 + 52 us).  24 tokens of
// 151936 logits, k = 10 / 50, both: random 16 / 19 us, around 1000 18 / 21, all
// equal 26 / 39, ascending 22 / 33.
//
// Order key of a logit: larger for larger values, equal for equal ones (0 and
// -0), 0 for NaN (which is never selected).
__device__ __forceinline__ uint32_t tk_key(float v) {
  const uint32_t u = __float_as_uint(v + 0.f);   // -0 becomes 0
  return v != v ? 0u : (u & 0x80000000u ? ~u : u | 0x80000000u);
}

constexpr int kChunkUnit = 64;           // logits a wave takes per load
constexpr int kSelBlock = 1024, kSelWaves = kSelBlock / 64;
constexpr int kSelCand = 128;            // candidates ranked one against all; more are reduced to k first
constexpr int kRedFew = 4, kRedMany = 16;   // units a wave of that reduction holds
static_assert(kSelCand >= kTopKMax, "room for the k best");
constexpr int kWaveUnits = 16;           // units a wave of k_topk_max takes at a time
constexpr int kSelUnits = 8;             // units a wave of k_topk_select has in flight
static_assert(archead::kTopKChunks == kSelBlock && archead::kTopKChunkUnit == kChunkUnit &&
              archead::kTopKWave == kChunkUnit * kWaveUnits, "host and kernels agree on the chunks");

// keys[m][c] = the largest key of logits [c cs, (c + 1) cs) of row m.  UPC:
// units per chunk, or kWaveUnits for chunks of any multiple of them; a wave
// takes kWaveUnits / UPC chunks.
template <int UPC>
__global__ __launch_bounds__(kBlock) void k_topk_max(const float* logits, int64_t ldl, int64_t V, int cs,
                                                     int n_chunk, uint32_t* keys) {
  constexpr int kCpw = kWaveUnits / UPC;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int64_t m = blockIdx.y;
  const float* row = logits + m * ldl;
  const int c0 = (int(blockIdx.x) * kWaves + wid) * kCpw;
  const int span = UPC < kWaveUnits ? kWaveUnits * kChunkUnit : cs;
  uint32_t best[kCpw] = {};
  for (int o = 0; o < span; o += kWaveUnits * kChunkUnit) {
    float v[kWaveUnits];
#pragma unroll
    for (int u = 0; u < kWaveUnits; ++u) {
      const int64_t j = int64_t(c0) * cs + o + u * kChunkUnit + lane;
      v[u] = j < V ? row[j] : NAN;
    }
#pragma unroll
    for (int u = 0; u < kWaveUnits; ++u) best[u / UPC] = max(best[u / UPC], tk_key(v[u]));
  }
#pragma unroll
  for (int c = 0; c < kCpw; ++c) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) best[c] = max(best[c], uint32_t(__shfl_xor(int(best[c]), off, 64)));
    if (lane == 0 && c0 + c < n_chunk) keys[m * n_chunk + c0 + c] = best[c];
  }
}

// Grid tokens: the k best of row m in order, out to vals[m * ldk + j] (may be
// null) and idx[m * ldk + j], j < k; a slot no value reached (fewer than k
// non-NaN logits) gets (-inf, -1).  n_chunk <= kSelBlock.
__global__ __launch_bounds__(kSelBlock) void k_topk_select(const float* logits, int64_t ldl, int64_t V, int cs,
                                                           int n_chunk, const uint32_t* keys, int k,
                                                           float* vals, int64_t* idx, int64_t ldk) {
  __shared__ uint32_t skey[kSelBlock];
  __shared__ int slist[kSelBlock];
  __shared__ float cval[kSelCand];
  __shared__ int cidx[kSelCand];
  __shared__ int sties[kSelWaves];   // chunks at the floor before each wave's
  __shared__ int scount[2][64];
  __shared__ uint32_t sfloor;
  __shared__ int smost, nlist, ncand;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m = blockIdx.x;
  const float* row = logits + m * ldl;
  const uint32_t mine = tid < n_chunk ? keys[m * n_chunk + tid] : 0u;
  skey[tid] = mine;
  if (tid == 0) {
    nlist = 0;
    ncand = 0;
  }
  __syncthreads();
  if (wid == 0) {
    // the largest key prefix that at least k chunk maxima reach: of 20 bits,
    // and where clearly more than k reach that one (a large common offset,
    // ties) of up to 32, the k-th largest maximum itself
    uint32_t kk[kSelWaves];
#pragma unroll
    for (int i = 0; i < kSelWaves; ++i) kk[i] = skey[64 * i + lane];
    const int enough = k + k / 4 + 3;   // (reading a few chunks more is cheaper than 12 steps more)
    uint32_t f = 0;
    int reach = n_chunk;   // maxima that reach f
    auto step = [&](int bit) {
      const uint32_t t = f | (1u << bit);
      int n = 0;
#pragma unroll
      for (int i = 0; i < kSelWaves; ++i) n += __popcll(__ballot(kk[i] >= t));
      f = n >= k ? t : f;
      reach = n >= k ? n : reach;
    };
#pragma unroll
    for (int bit = 31; bit >= 12; --bit) step(bit);
#pragma unroll 1
    for (int bit = 11; bit >= 0 && reach > enough; --bit) step(bit);
    int most = kSelBlock;
    if (__builtin_expect(f && reach > enough, 0)) {
      // Many maxima equal to f: the first k - (maxima above f) of their chunks
      // hold as many of the logits equal to f as can be wanted, those of the
      // smallest indices among them; no other chunk of f's is read.
      int before = 0;
      most = k;
#pragma unroll
      for (int i = 0; i < kSelWaves; ++i) {
        if (lane == 0) sties[i] = before;
        before += __popcll(__ballot(kk[i] == f));
        most -= __popcll(__ballot(kk[i] > f));
      }
    }
    if (lane == 0) {
      sfloor = f ? f : 1u;   // 1: every logit but NaN
      smost = most;
    }
  }
  __syncthreads();
  const uint32_t fl = sfloor;
  const uint64_t lower = (uint64_t(1) << lane) - 1;
  bool listed = mine >= fl;
  if (__builtin_expect(smost < kSelBlock, 0)) {
    const uint64_t tie = __ballot(mine == fl);
    listed = mine > fl || (mine == fl && sties[wid] + __popcll(tie & lower) < smost);
  }
  if (listed) slist[atomicAdd(&nlist, 1)] = tid;
  __syncthreads();
  const int lu = __builtin_ctz(cs / kChunkUnit), units = nlist << lu;   // (a power of two)
  // this lane's logit of unit u of the listed chunks: its index (V: none)
  auto index_of = [&](int u) {
    const int64_t j = u < units ? int64_t(slist[u >> lu]) * cs + (u & ((1 << lu) - 1)) * kChunkUnit + lane : V;
    return int(j < V ? j : V);
  };
  for (int u0 = wid; u0 < units; u0 += kSelUnits * kSelWaves) {
    float v[kSelUnits];
    int j[kSelUnits];
#pragma unroll
    for (int b = 0; b < kSelUnits; ++b) {
      j[b] = index_of(u0 + b * kSelWaves);
      v[b] = j[b] < V ? row[j[b]] : NAN;
    }
#pragma unroll
    for (int b = 0; b < kSelUnits; ++b) {
      const bool hit = tk_key(v[b]) >= fl;
      const uint64_t mask = __ballot(hit);
      if (!mask) continue;
      int at = 0;
      if (lane == 0) at = atomicAdd(&ncand, __popcll(mask));
      at = __builtin_amdgcn_readfirstlane(at) + __popcll(mask & lower);
      if (hit && at < kSelCand) {
        cval[at] = v[b];
        cidx[at] = j[b];
      }
    }
  }
  __syncthreads();
  int nc = ncand;
  if (__builtin_expect(nc > kSelCand, 0)) {
    // More than are ranked one against all: the k best of them, some units
    // a wave at a time together with the k best so far, by a search for the
    // k-th largest key and among its equals for the largest index taken; the
    // whole workgroup counts.  Its cost depends on the number of logits alone.
    uint32_t top = mine;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) top = max(top, uint32_t(__shfl_xor(int(top), off, 64)));
    const uint64_t lm = __ballot(listed);
    if (lane == 0) {   // (skey's words were read above)
      skey[wid] = top;
      skey[kSelWaves + wid] = lm ? 64 * wid + __builtin_ctzll(lm) : kSelBlock;
      skey[2 * kSelWaves + wid] = lm ? 64 * wid + 63 - __builtin_clzll(lm) : 0;
    }
    __syncthreads();
    uint32_t c_lo = kSelBlock, c_hi = 0;   // first and last chunk listed
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
      top = max(top, skey[w]);
      c_lo = min(c_lo, skey[kSelWaves + w]);
      c_hi = max(c_hi, skey[2 * kSelWaves + w]);
    }
    const int high = top == fl ? -1 : 31 - __builtin_clz(top ^ fl);   // the keys agree above it
    // and the indices above this one (cs > 1: they differ somewhere)
    const uint32_t j_lo = c_lo * uint32_t(cs), j_hi = c_hi * uint32_t(cs) + uint32_t(cs - 1);
    const int j_high = 31 - __builtin_clz(j_lo ^ j_hi);
    int have = 0, end = int(V);
    uint32_t f = fl;
    auto reduce = [&](auto units_per_wave) {
      constexpr int kRedUnits = decltype(units_per_wave)::value;
      for (int r0 = 0; r0 < units; r0 += kRedUnits * kSelWaves) {
        // element 0: one of the k best so far; then those read now that may join them
        uint32_t key[kRedUnits + 1];
        int j[kRedUnits + 1];
        j[0] = tid < have ? cidx[tid] : int(V);
        key[0] = tid < have ? tk_key(cval[tid]) : 0u;
#pragma unroll
        for (int b = 1; b <= kRedUnits; ++b) {
          j[b] = index_of(r0 + wid + (b - 1) * kSelWaves);
          key[b] = j[b] < V ? tk_key(row[j[b]]) : 0u;
          if (!(key[b] > f || (key[b] == f && j[b] < end))) key[b] = 0u;
        }
        __syncthreads();   // every thread has read ncand, the counts and the k best so far
        if (tid < 64) scount[0][tid] = scount[1][tid] = 0;
        if (tid == 0) ncand = 0;
        __syncthreads();
        // Logits of the workgroup that satisfy `hit`; each word of scount once.
        auto count = [&](int* word, auto hit) {
          int n = 0;
#pragma unroll
          for (int b = 0; b <= kRedUnits; ++b) n += __popcll(__ballot(hit(key[b], j[b])));
          if (lane == 0 && n) atomicAdd(word, n);
          __syncthreads();
          return *word;
        };
        const int n_in = count(&scount[0][32], [&](uint32_t kb, int) { return kb > 0; });
        if (n_in == have) continue;
        end = int(V);   // equals of f from this index on are left out
        if (n_in > k) {
          f = high == 31 ? 0u : fl >> (high + 1) << (high + 1);
          int reach = n_in;
          for (int bit = high; bit >= 0 && reach != k; --bit) {
            const uint32_t t = f | (1u << bit);
            const int n = count(&scount[0][bit], [&](uint32_t kb, int) { return kb >= t; });
            if (n >= k) {
              f = t;
              reach = n;
            }
          }
          if (reach != k) {
            const int want = k - count(&scount[0][33], [&](uint32_t kb, int) { return kb > f; });
            int n = -1;
            end = int(j_lo >> j_high >> 1 << 1 << j_high);
            for (int bit = j_high; bit >= 0 && n != want; --bit) {
              const int t = end | (1 << bit);
              n = count(&scount[1][bit], [&](uint32_t kb, int jb) { return kb == f && jb < t; });
              if (n <= want) end = t;
            }
          }
        }
#pragma unroll
        for (int b = 0; b <= kRedUnits; ++b) {
          if (key[b] > f || (key[b] == f && j[b] < end)) {
            const int at = atomicAdd(&ncand, 1);
            cval[at] = row[j[b]];
            cidx[at] = j[b];
          }
        }
        __syncthreads();
        have = ncand;
      }
    };
    if (units <= kRedFew * kSelWaves) reduce(std::integral_constant<int, kRedFew>{});
    else reduce(std::integral_constant<int, kRedMany>{});
    nc = have;
  }
  // rank each candidate among all (distinct indices: distinct ranks)
  for (int t = tid; t < nc; t += kSelBlock) {
    const float v = cval[t];
    const int i = cidx[t];
    int rank = 0;
    for (int o = 0; o < nc; ++o) rank += tk_better(cval[o], cidx[o], v, i);
    if (rank < k) {
      if (vals) vals[m * ldk + rank] = v;
      idx[m * ldk + rank] = int64_t(i);
    }
  }
  if (tid >= nc && tid < k) {
    if (vals) vals[m * ldk + tid] = -INFINITY;
    idx[m * ldk + tid] = -1;
  }
}

// Per token m (grid M, workgroups of kMergeBlock): the k best of its n_part
// partial lists of k pairs, at most kMergeBlock * kMergeC candidates in all, out
// to vals[m * ldk + j] (may be null) and idx[m * ldk + j], j < k; a slot no
// value reached (fewer than k non-NaN logits) gets (-inf, -1).  It takes k
// rounds.  Each thread holds up to
// kMergeC candidates and its best one; a round finds the best of the
// workgroup (DPP within rows of 16 lanes, then the four rows of the wave,
// then the waves through LDS), writes it out, and its owner (indices are
// distinct across the partial lists) drops it and takes its next best.  The
// cost is k rounds, whatever the values.
constexpr int kMergeC = 8;
static_assert(archead::kTopKMergeBlock == 1024 && kMergeC == archead::kTopKMergeC,
              "host and kernel agree on the merge workgroup");

template <int kMergeBlock>
__global__ __launch_bounds__(kMergeBlock) void k_topk_merge(const float* pv, const int* pi,
                                                            int64_t n_part, int k, float* vals,
                                                            int64_t* idx, int64_t ldk) {
  constexpr int kMergeWaves = kMergeBlock / 64;
  __shared__ float wv[2][kMergeWaves];
  __shared__ int wi[2][kMergeWaves];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m = blockIdx.x;
  const int64_t n = n_part * k;
  const float* v = pv + m * n;
  const int* ix = pi + m * n;
  float cv[kMergeC];
  int ci[kMergeC];
#pragma unroll
  for (int u = 0; u < kMergeC; ++u) {
    const int64_t j = int64_t(u) * kMergeBlock + tid;
    cv[u] = j < n ? v[j] : -INFINITY;
    ci[u] = j < n ? ix[j] : kNoIdx;
  }
  float tv = -INFINITY;
  int ti = kNoIdx;
#pragma unroll
  for (int u = 0; u < kMergeC; ++u) tk_pick(tv, ti, cv[u], ci[u]);
  for (int r = 0; r < k; ++r) {
    float bv = tv;
    int bi = ti;
    tk_row16_best(bv, bi);
    float gv = rlane_f(bv, 0);
    int gi = __builtin_amdgcn_readlane(bi, 0);
#pragma unroll
    for (int row = 1; row < 4; ++row)
      tk_pick(gv, gi, rlane_f(bv, 16 * row), __builtin_amdgcn_readlane(bi, 16 * row));
    if (lane == 0) {
      wv[r & 1][wid] = gv;
      wi[r & 1][wid] = gi;
    }
    __syncthreads();
    gv = lane < kMergeWaves ? wv[r & 1][lane] : -INFINITY;
    gi = lane < kMergeWaves ? wi[r & 1][lane] : kNoIdx;
    tk_row16_best(gv, gi);
    gv = rlane_f(gv, 0);
    gi = __builtin_amdgcn_readlane(gi, 0);
    if (tid == 0) {
      if (vals) vals[m * ldk + r] = gv;
      idx[m * ldk + r] = gi == kNoIdx ? int64_t(-1) : int64_t(gi);
    }
    if (gi != kNoIdx && ti == gi) {
#pragma unroll
      for (int u = 0; u < kMergeC; ++u) {
        const bool hit = ci[u] == gi;
        cv[u] = hit ? -INFINITY : cv[u];
        ci[u] = hit ? kNoIdx : ci[u];
      }
      tv = -INFINITY;
      ti = kNoIdx;
#pragma unroll
      for (int u = 0; u < kMergeC; ++u) tk_pick(tv, ti, cv[u], ci[u]);
    }
  }
}

}  // namespace

namespace archead {
namespace kern {

const void* gemv_topk(int lpr, bool sc8, int gen) {
  if (gen == 2) return gemv_topk_fn<2>(lpr, sc8);
  if (gen == 1) return gemv_topk_fn<1>(lpr, sc8);
  return gemv_topk_fn<0>(lpr, sc8);
}

const void* topk_max(int cs) {
  return cs == kChunkUnit       ? reinterpret_cast<const void*>(k_topk_max<1>)
         : cs == 4 * kChunkUnit ? reinterpret_cast<const void*>(k_topk_max<4>)
                                : reinterpret_cast<const void*>(k_topk_max<kWaveUnits>);
}
const void* topk_select() { return reinterpret_cast<const void*>(k_topk_select); }
const void* topk_merge(int block) {
  return block == 256 ? reinterpret_cast<const void*>(k_topk_merge<256>)
                      : reinterpret_cast<const void*>(k_topk_merge<1024>);
}

}  // namespace kern
}  // namespace archead
