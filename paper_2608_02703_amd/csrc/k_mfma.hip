// The tiled many-token kernel's instantiations and its prologue kernels
// (head-derived tables, stage 1 on MFMA and its split-d sum).
#include "dev_mfma.cuh"
#include "kernels.h"

namespace {

// The head-derived tables, by thread t0 of nthr.  What bounds it: latency;
// so a column's scales are read eight at a time, ahead of the stores (one at a
// time 50 us for the 151936-row head).
__device__ __forceinline__ void prep_tables(const PrepArgs& a, int64_t t0, int64_t nthr) {
  // (a) one thread per (vocabulary tile, column): walk the slots of the row
  // (lanes write consecutive columns)
  for (int64_t e = t0; e < a.n_vt * kTN; e += nthr) {
    const int64_t vt = e / kTN, c = e % kTN;
    const int64_t v = vt * kTN + c < a.V ? vt * kTN + c : a.V - 1;
    const uint16_t* src = a.rs + v * a.ngrp;
    const uint8_t* src8 = reinterpret_cast<const uint8_t*>(a.rs) + v * a.ngrp;
    const float rsv = a.rrs ? f16_to_f32(a.rrs[v]) : 0.f;
    const float su = a.rc ? nz_scale(a.su[v]) : 0.f, sa = a.rr ? nz_scale(a.sa[v]) : 0.f;
    float* dst = a.ratio + vt * int64_t(a.nslot) * kTN + c;
    float prev = 0.f;
    int k = 0;
    constexpr int kAhead = 8;
    for (int k0 = 0; k0 < a.ngrp; k0 += kAhead) {
      float s[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int j = k0 + u < a.ngrp ? k0 + u : a.ngrp - 1;
        if (a.rrs) {   // rs * q, exact in fp32
          s[u] = rsv * float(src8[j]);
          s[u] = s[u] == 0.f ? kZeroScale : s[u];
        } else {
          s[u] = nz_scale(src[j]);
        }
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (k0 + u >= a.ngrp) break;
        dst[int64_t(k) * kTN] = k ? prev / s[u] : 0.f;
        prev = s[u];
        ++k;
      }
    }
    if (a.rc) {
      dst[int64_t(k++) * kTN] = prev / su;
      prev = su;
    }
    if (a.rr) {
      dst[int64_t(k++) * kTN] = prev / sa;
      prev = sa;
    }
    a.fin[vt * kTN + c] = prev * ldexpf(1.f, -(kXExp + kCodeExp));
  }
  // (b) 16 dimensions per thread, stored twice (row-major, so lanes write
  // consecutive chunks)
  const int nch = a.urow / 32;
  for (int64_t e = t0; e < a.V * nch; e += nthr) {
    const int64_t v = e / nch;
    const int j0 = int(e % nch) * kExpDims;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      const int j = j0 + jj;
      int8_t c = 0;
      if (j < a.rc_pad) {
        if (j < a.rc)
          c = int8_t(fcode1(reinterpret_cast<const uint8_t*>(a.cu) + v * a.cu_row, j, a.u5 != 0));
      } else if (j - a.rc_pad < a.rr) {
        c = a.ca[v * a.rr + (j - a.rc_pad)];
      }
      w[jj / 4] |= uint32_t(uint8_t(c)) << (8 * (jj % 4));
    }
    uint4* dst = reinterpret_cast<uint4*>(a.ucodes + e * 32);
    dst[0] = dst[1] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

__global__ __launch_bounds__(kBlock) void k_prep(PrepArgs a) {
  prep_tables(a, int64_t(blockIdx.x) * kBlock + threadIdx.x, int64_t(gridDim.x) * kBlock);
}

// One token's scaled x (a workgroup).
__device__ __forceinline__ void scale_row(const Stage1MArgs& a, int64_t m, int* smax) {
  const uint16_t* x = a.x + m * a.ldx;
  int mx = 0;
  for (int i = 8 * int(threadIdx.x); i < a.d; i += 8 * kS1MBlock) {
    const u32x4_t v = *reinterpret_cast<const u32x4_t*>(x + i);
#pragma unroll
    for (int j = 0; j < 4; ++j) mx = max(mx, max(int(v[j] & 0x7fffu), int((v[j] >> 16) & 0x7fffu)));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = max(mx, __shfl_xor(mx, off, 64));
  if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kS1MWaves; ++w) mx = max(mx, smax[w]);
  int e = (mx >> 7) - 127;   // zero and subnormal rows: -126; inf and NaN stay themselves
  e = e < -126 ? -126 : (e > 127 ? 127 : e);
  for (int i = 8 * int(threadIdx.x); i < a.d; i += 8 * kS1MBlock) {
    u32x4_t v = *reinterpret_cast<const u32x4_t*>(x + i);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = a.even ? kXExpFid - e : kXExp - e - (j & 1 ? 4 : 0);
      const uint32_t lo = __float_as_uint(ldexpf(bf16_lo(v[j]), k));
      const uint32_t hi = __float_as_uint(ldexpf(bf16_hi(v[j]), k));
      v[j] = (lo >> 16) | (hi & 0xffff0000u);
    }
    *reinterpret_cast<u32x4_t*>(a.xs + m * a.ldxs + i) = v;
  }
  if (threadIdx.x == 0) a.rowexp[m] = ldexpf(1.f, e);
}

// The first p.blocks workgroups build the head-derived tables (a head used
// without prepared ones): the two are independent and each too short to fill
// the chip.
__global__ __launch_bounds__(kS1MBlock) void k_stage1m(Stage1MArgs a, PrepArgs p) {
  __shared__ float red[kS1MWaves][kS1MTok][kS1MCols + 1];
  const int64_t blk = stage1_block();
  if (blk < p.blocks) {
    prep_tables(p, blk * kS1MBlock + threadIdx.x, int64_t(p.blocks) * kS1MBlock);
    return;
  }
  const int wg = int(blk - p.blocks);
  const int64_t n_s1 = int64_t(a.mblocks) * a.rblocks * a.ksplit;
  if (wg >= n_s1) {
    if (wg - n_s1 < a.M) scale_row(a, wg - n_s1, reinterpret_cast<int*>(&red[0][0][0]));
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, q = lane >> 4;
  const int R = a.rc + a.rr;
  const int bx = wg % a.mblocks, byz = wg / a.mblocks;
  const int by = byz % a.rblocks;
  const int64_t tok0 = int64_t(bx) * kS1MTok;
  const int kb = by * kS1MCols;           // first factor row of this workgroup
  const int ngrp = a.d / a.g, cpg = a.g / 32;
  // this workgroup's residual groups (split ks of ksplit equal parts), dealt
  // to its waves
  const int ks = byz / a.rblocks, gps = ngrp / a.ksplit, g0 = ks * gps;
  const int c0 = (g0 + wid * gps / kS1MWaves) * cpg, c1 = (g0 + (wid + 1) * gps / kS1MWaves) * cpg;
  const int64_t mrow = tok0 + lr < a.M ? tok0 + lr : a.M - 1;
  const uint16_t* xrow = a.x + mrow * a.ldx + 8 * q;
  const bool do_sum = by == 0;
  constexpr int NB = kS1MCols / 16;
  const int nblk = R - kb >= kS1MCols ? NB : (R - kb + 15) / 16;

  // this lane's factor row in each 16-column block (clamped; masked on store)
  const int8_t* wrow[NB];
  const uint16_t* srow[NB];
  int sgrp[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    int k = kb + 16 * nb + lr;
    k = k < R ? k : (R > 0 ? R - 1 : 0);
    const bool core = k < a.rc;
    wrow[nb] = (core ? a.cv + int64_t(k) * a.d : a.cb + int64_t(k - a.rc) * a.d) + 8 * q;
    sgrp[nb] = core ? a.gv : a.gb;
    srow[nb] = core ? a.sv + int64_t(k) * (a.d / a.gv) : a.sb + int64_t(k - a.rc) * (a.d / a.gb);
  }
  const bf16x8_t ones = {(__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f,
                         (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f};
  f32x4_t acc[NB], gs = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  bf16x8_t A, An;
  u32x2_t B[NB], Bn[NB];   // int8 codes
  float s[NB], sn[NB];
  auto load = [&](int c, bf16x8_t& A_, u32x2_t* B_, float* s_) {
    const int k0 = 32 * c;
    A_ = *reinterpret_cast<const bf16x8_t*>(xrow + k0);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if (nb < nblk) {
        B_[nb] = *reinterpret_cast<const u32x2_t*>(wrow[nb] + k0);
        s_[nb] = f16_to_f32(srow[nb][k0 / sgrp[nb]]);
      }
    }
  };
  if (c0 < c1) load(c0, A, B, s);
  for (int c = c0; c < c1; ++c) {
    if (c + 1 < c1) load(c + 1, An, Bn, sn);
    if (do_sum) gs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, ones, gs, 0, 0, 0);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if (nb < nblk) {
        const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
        acc[nb] += s[nb] * __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, int8x8_to_bf16(B[nb].x, B[nb].y), z, 0, 0, 0);
      }
    }
    if (do_sum && (c + 1) % cpg == 0) {
      const int j = c / cpg;
      if (lr == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t m = tok0 + 4 * q + i;
          if (m < a.M) a.gsum[j * a.M + m] = gs[i];
        }
      }
      gs = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    A = An;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) B[nb] = Bn[nb], s[nb] = sn[nb];
  }
  if (R == 0) return;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wid][4 * q + i][16 * nb + lr] = acc[nb][i];
  __syncthreads();
  for (int e = threadIdx.x; e < kS1MTok * kS1MCols; e += kS1MBlock) {
    const int tt = e / kS1MCols, c = e % kS1MCols;
    const int64_t m = tok0 + tt;
    const int k = kb + c;
    if (m < a.M && k < R) {
      float v = red[0][tt][c];
#pragma unroll
      for (int w = 1; w < kS1MWaves; ++w) v += red[w][tt][c];
      a.tpart[(int64_t(ks) * a.M + m) * R + k] = v;
    }
  }
}

// One thread per (token, rank dimension padded to blocks of 16), then one per
// (residual group, token of the padded count, tokens fastest).
__global__ __launch_bounds__(kBlock) void k_stage1m_fin(Stage1MArgs a) {
  const int R = a.rc + a.rr, ngrp = a.d / a.g, dims = a.nch * kExpDims;
  int64_t t = stage1_block() * kBlock + threadIdx.x;
  const int scale_exp = (a.even ? kXExpFid : kXExp) + kCodeExp;
  auto exponent = [&](int64_t m) { return int(__float_as_uint(a.rowexp[m]) >> 23) - 127; };
  if (t < a.M * dims) {
    const int64_t m = t / dims;
    const int c = int(t % dims) / kExpDims, i = int(t % kExpDims);
    const int dim = (c < a.nch_u ? c : c - a.nch_u) * kExpDims + i;
    __bf16 hi = (__bf16)0.f, md = hi, lo = hi;
    if (dim < (c < a.nch_u ? a.rc : a.rr)) {
      const int k = c < a.nch_u ? dim : a.rc + dim;
      float v = a.tpart[m * R + k];
      for (int ks = 1; ks < a.ksplit; ++ks) v += a.tpart[(int64_t(ks) * a.M + m) * R + k];
      v = ldexpf(v, scale_exp - exponent(m));
      hi = (__bf16)v;
      const float r1 = v - float(hi);
      md = (__bf16)r1;
      lo = (__bf16)(r1 - float(md));
    }
    uint16_t* dst = a.tsplit + m * a.ldxs + c * 64 + i;
    dst[0] = __builtin_bit_cast(uint16_t, hi);
    dst[16] = __builtin_bit_cast(uint16_t, md);
    dst[32] = __builtin_bit_cast(uint16_t, lo);
    dst[48] = 0;
    return;
  }
  t -= a.M * dims;
  const int64_t mp = (a.M + kTM - 1) / kTM * kTM;
  const int64_t m = t % mp, j = t / mp;
  if (j >= ngrp) return;
  a.gbias[((m / kTM) * ngrp + j) * kTM + m % kTM] =
      m < a.M ? -8.f * ldexpf(a.gsum[j * a.M + m], scale_exp - exponent(m)) : 0.f;
}

}  // namespace

namespace archead {
namespace kern {

const void* mfma(bool ce, int tm, int nw) {
  if (tm == 64 && nw == 4)
    return ce ? reinterpret_cast<const void*>(k_mfma<true, 64, 4>)
              : reinterpret_cast<const void*>(k_mfma<false, 64, 4>);
  if (tm == 128 && nw == 4)
    return ce ? reinterpret_cast<const void*>(k_mfma<true, 128, 4>)
              : reinterpret_cast<const void*>(k_mfma<false, 128, 4>);
  if (tm == 128)
    return ce ? reinterpret_cast<const void*>(k_mfma<true, 128, 8>)
              : reinterpret_cast<const void*>(k_mfma<false, 128, 8>);
  return ce ? reinterpret_cast<const void*>(k_mfma<true, kTM, 8>)
            : reinterpret_cast<const void*>(k_mfma<false, kTM, 8>);
}
const void* prep() { return reinterpret_cast<const void*>(k_prep); }
const void* stage1m() { return reinterpret_cast<const void*>(k_stage1m); }
const void* stage1m_fin() { return reinterpret_cast<const void*>(k_stage1m_fin); }

}  // namespace kern
}  // namespace archead
