// The tiled many-token MFMA kernel template (k_mfma) and the argument blocks
// of its prologue kernels.
#pragma once

#include "dev_common.cuh"

namespace {

// ------------------------------------------------------------ many tokens: MFMA
// Tiled bf16 MFMA path for many tokens (needs g % 64 == 0).  A workgroup owns
// a TM x kTN tile (tokens x vocabulary rows), its waves blocks of WM x 64, each
// a grid of 32x32 MFMA tiles (v_mfma_f32_32x32x16_bf16: lane l holds row l%32
// of an operand and 8 k-slots of half l/32; D lane l holds column l%32, rows
// 8 (i/4) + 4 (l/32) + i%4).  The K loop runs in stages of kKS elements that
// direct global-to-LDS buffer loads bring, with no register staging: x into a
// ring of kRing stages, the codes of two stages into one place, which every
// wave empties into registers before the stage that uses them.  Within a
// stage half-wave h takes the row's code dwords 4h .. 4h + 3 (one 16-byte
// read) and the x units of the same indices.  Token rows and vocabulary rows
// are XOR-swizzled in 16-byte units so fragment reads are bank-conflict free.
//
// Codes are unpacked per wave to bf16 u 2^-133, u = c + 8 (exact,
// unpack8_sub), against x scaled per token by a power of two (kXExp; in the
// fidelity and rank passes kXExpFid) and, at the elements of the odd code
// pairs, by 1 / 16.  The accumulator is kept in units of the current scale
// slot's scale: at the start of slot k it becomes
// acc * (s'_{k-1} / s'_k) + bias_k, after which the MFMAs add the slot's
// terms, so at the end s'_last * acc is the scaled logit.  Slots are the
// residual groups (bias -8 * (sum of x over the group), the MFMAs adding
// sum u x), then the rank-r expansion's core part (scale s_U) and correction
// part (s_A).  s' is the scale with zero replaced by kZeroScale, which pushes
// a zero-scale slot's contribution below fp32 resolution of the result.  The
// expansion parts run as extra stages with the same geometry, 16 rank
// dimensions per stage: the "x" rows hold t split into three bf16 parts (hi =
// bf16(t), mid = bf16(t - hi), lo = bf16(t - hi - mid); their sum is t to
// fp32 precision) as [hi | mid | lo | 0], the "code" rows the int8 factor
// codes (exact in bf16) twice, [c | c]; one K-step per part.
//
// What bounds it.  Many tokens: the matrix unit and the VALU share the SIMD's
// time (a 32-cycle MFMA hides about four VALU operations of either resident
// wave; more lengthen it), and the chip runs at its power limit (about 1.65-1.75
// GHz under this load, falling as the matrix unit gets busier), so the loop is
// built for few VALU operations per MFMA: 1.25 for the unpack and 2 for the
// rescale (one FMA per element and group of 128).  The codes are the MFMA's
// first operand, so a lane holds the logits of one token: the biases are one
// LDS word per token block, and the softmax epilogues reduce within the lane.
// Against 16x16x32 MFMAs with lanes along the vocabulary, magic-number codes
// and the barrier between stages (us per call): Qwen CE M = 4096 4943 -> 4603,
// 128k head M = 512 1052 -> 1015; matrix unit busy 54 / 59% -> 62 / 63%.
// Few tokens: the stream of codes, and in it the size of the pieces: 64 bytes
// of a row at a time instead of 32 took the Qwen head at M = 64 from 142 to
// 128.5 us per call (117 us in this kernel, 2.9 TB/s), M = 512 from 619 to 603.
struct MfmaArgs {
  const uint8_t* codes;
  const uint16_t* x;       // [M][ldx] bf16, scaled (Stage1MArgs::xs)
  int64_t ldx;
  const uint16_t* tsplit;  // [M] rows of ldx: [nch][4][16] bf16, t hi, mid, lo, 0 per 16 rank dimensions
  const int8_t* ucodes;    // [V][nch][2][16] int8: U_c then A_w codes (each padded), twice
  const float* gbias;      // [n_mt][d / g][kTM] slot biases of the residual groups
  const float* rowexp;     // [n_mt][kTM] 2^e of each token
  const float* ratio;      // [n_vt][nslot][kTN]: s'_{k-1} / s'_k (0 for k = 0)
  const float* fin;        // [n_vt][kTN]: s' of the last slot * 2^-(kXExp + kCodeExp)
  int64_t M, V;
  int d, g, nslot, nch, nch_u;
  int64_t n_mt, n_vt, n_tiles, tiles_per_xcd;
  void* out;
  int64_t ldo;
  int out_bf16;
  const void* tgt;
  int tgt64;
  float2* part;            // [M, n_vt]
  int* part_idx;           // [M, n_vt] argmax partials, or null
  float* tgt_logit;        // [M]
  // logit fidelity against a dense bf16 head (XE = 1) and the rank pass (XE = 2)
  const uint16_t* dense;   // [V][ldw] bf16
  int64_t ldw;
  void* fid_part;          // [M][n_vt] FidTilePart
  int* fid_need;           // [ceil(M / 64)][n_vt] tiles the rank pass has to count
  const float* bref;       // [M] packed logit at the reference's top-1
  const int64_t* ref_idx;  // [M] the reference's top-1
  int64_t* rank;           // [M]
};

// One vocabulary tile's statistics of one token for the fidelity pass: the
// maxima of the dense (a) and packed (b) logits, b at the first maximum of a,
// and relative to the maxima sum e^(a - ma), sum e^(b - mb), sum e^(a - ma)
// (a - b) and sum (a - b)^2; and the first tile columns of both maxima.
struct FidTilePart {
  float ma, mb, bat, sa, sb, t, sq;
  int iab;                 // a's column | b's << 16 (kNoCol: no finite or infinite maximum)
};
constexpr int kNoCol = 0x7fff;
static_assert(sizeof(FidTilePart) == 32, "the workspace holds 32 bytes per tile and token");

// f(LO) + .. + f(LO + N - 1) as a tree (f takes an integral_constant): log2 N
// roundings in a lane's sums over a tile, where one after the other makes N.
template <int LO, int N, typename F>
__device__ __forceinline__ auto tree_sum(F f) {
  if constexpr (N == 1) return f(std::integral_constant<int, LO>{});
  else return tree_sum<LO, N / 2>(f) + tree_sum<LO + N / 2, N / 2>(f);
}

// XE: 0 logits or CE (CE), 1 the fidelity pass (the dense head's rows are
// loaded straight into the waves' registers, one stage ahead, and accumulated
// beside the packed logits; per-tile FidTilePart out), 2 the rank pass (per
// token, packed logits ranked ahead of bref / ref_idx counted into rank, over
// the tiles that hold any).
// (waves per SIMD: 2 with 8-wave workgroups and with 128-row tiles of 4
// waves, two workgroups per CU; 3 with 64-row tiles, three per CU)
template <bool CE, int TM, int NW, int XE = 0>
__global__ __launch_bounds__(NW * 64)
__attribute__((amdgpu_waves_per_eu(XE != 1 && MGeomT<TM, NW>::WGS * NW / 4 > 2
                                       ? MGeomT<TM, NW>::WGS * NW / 4 : 2)))
void k_mfma(MfmaArgs a) {
  using G = MGeomT<TM, NW>;
  constexpr int MI = G::MI;        // row blocks per wave
  constexpr int WM = G::WM;        // token rows per wave
  constexpr int NI = G::NI;        // 32-column blocks per wave
  extern __shared__ __align__(16) uint8_t mfma_lds[];
  lds_u8* const L = (lds_u8*)mfma_lds;

  // tile: workgroups are dealt to the 8 XCDs round-robin, so XCD x runs
  // blocks x, x+8, ...; it gets the contiguous run [x T, (x+1) T) of the tile
  // order, which walks groups of kRasterGM token tiles across the vocabulary
  // (token tile fastest): the tiles one XCD runs at once share a few token
  // tiles and a few vocabulary tiles in its L2
  const int64_t b = blockIdx.x;
  const int64_t lin = (b & 7) * a.tiles_per_xcd + (b >> 3);
  if (lin >= a.n_tiles) return;
  const int64_t gsz = int64_t(kRasterGM) * a.n_vt;
  const int64_t rg = lin / gsz, first = rg * kRasterGM;
  const int64_t gm = a.n_mt - first < kRasterGM ? a.n_mt - first : kRasterGM;
  const int64_t within = lin - rg * gsz;
  const int64_t mt = first + within % gm, vt = within / gm;
  const int64_t m0 = mt * TM, v0 = vt * kTN;
  if constexpr (XE == 2) {
    static_assert(XE != 2 || TM == 64, "fid_need has one word per 64 tokens and tile");
    if (!a.fid_need[mt * a.n_vt + vt]) return;
  }
  const int rows = int(a.M - m0 < TM ? a.M - m0 : TM);
  const int cols = int(a.V - v0 < kTN ? a.V - v0 : kTN);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = NW == 8 ? wid >> 2 : 0, wn = wid & 3;
  const int lr = lane & 31, h = lane >> 5;
  const int ngrp = a.d / a.g;
  const uint32_t rowbytes = uint32_t(a.d) / 2;
  const uint32_t ldx2 = uint32_t(a.ldx) * 2;
  const uint32_t urow = uint32_t(a.nch) * 32;

  // buffer resources over exactly the bytes this tile may touch (loads past
  // them return zero instead of reading other memory)
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(a.x + m0 * a.ldx), 0, int((rows - 1) * ldx2 + uint32_t(a.d) * 2),
      kBufferWord3);
  const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a.codes + v0 * int64_t(rowbytes)), 0, int(uint32_t(cols) * rowbytes),
      kBufferWord3);
  const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(a.tsplit + m0 * a.ldx), 0,
      int(uint32_t(rows - 1) * ldx2 + uint32_t(a.nch) * 128), kBufferWord3);
  const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int8_t*>(a.ucodes + v0 * int64_t(urow)), 0, int(uint32_t(cols) * urow),
      kBufferWord3);
  // dense rows of the tile (fidelity pass)
  const uint32_t dstride = uint32_t(a.ldw) * 2;
  const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(XE == 1 ? a.dense + v0 * a.ldw : a.x), 0,
      XE == 1 ? int((cols - 1) * dstride + uint32_t(a.d) * 2) : 0, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rrat = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(a.ratio + vt * a.nslot * kTN), 0, a.nslot * kTN * 4, kBufferWord3);
  // (the biases are laid out per 256 tokens, [group][256]; a tile of TM < 256
  // rows starts inside such a block)
  const __amdgpu_buffer_rsrc_t rbias = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(a.gbias + (m0 / kTM) * ngrp * kTM + m0 % kTM), 0,
      int(ngrp * kTM - m0 % kTM) * 4, kBufferWord3);

  // per-lane load offsets (row and swizzled 16-byte unit) of the residual
  // stages; the expansion stages use the same units with their own row
  // strides; the stage's k offset is added per stage
  auto xunit = [&](int i, uint32_t stride) {
    const int off = (wid * G::NX + i) * 1024 + 16 * lane;
    const int r = off / (2 * kKS), p = (off % (2 * kKS)) / 16;
    return uint32_t(r < rows ? r : rows - 1) * stride + 16u * uint32_t(p ^ swz_x(r));
  };
  auto cunit = [&](int ci, uint32_t stride) {
    const int off = (wid * G::NC + ci) * 1024 + 16 * lane;
    const int c = off / kKS, p = (off % kKS) / 16;
    return uint32_t(c < cols ? c : cols - 1) * stride + 16u * uint32_t(p ^ swz_c(c));
  };
  uint32_t xo[G::NX];
#pragma unroll
  for (int i = 0; i < G::NX; ++i) xo[i] = xunit(i, ldx2);
  uint32_t co[G::NC];
#pragma unroll
  for (int ci = 0; ci < G::NC; ++ci) co[ci] = cunit(ci, rowbytes);
  const uint32_t ao_bias = uint32_t(wid * 64 + lane) * 4;
  const uint32_t ao_rat = uint32_t((wid & 3) * 64 + lane) * 4;

  // residual stages (an odd count is followed by one that computes nothing,
  // as the codes come for two stages), then the expansion's
  const int nres = a.d / kKS, nst = (nres + 1) & ~1, spg = a.g / kKS, ntot = nst + a.nch;
  const int st_a = nst + a.nch_u;   // first stage of the A_w part
  const int slot_a = ngrp + (a.nch_u > 0 ? 1 : 0);
  auto slot_of = [&](int s) { return s < nst ? s / spg : (s < st_a ? ngrp : slot_a); };
  auto slot_start = [&](int s) { return s < nst ? s < nres && s % spg == 0 : (s == nst || s == st_a); };
  int sg_ahead = 2 % spg, slot_ahead = 2 / spg;   // of stage s + 2 in the residual loop
  // load PART (0 .. NLX-1) of this wave's share of stage s, apart from its
  // codes, into ring slot buf: x (or t) units, then, where the stage starts a
  // slot, 64 scale ratios and (residual groups) 64 slot biases.  KIND: 1 a
  // residual stage, 2 an expansion stage, 3 either (checked).
  auto issue_part = [&](int s, int buf, int part, auto kind) {
    constexpr int KIND = decltype(kind)::value;
    lds_u8* base = L + buf * G::STAGE;
    const bool res = KIND == 1 || (KIND == 3 && s < nst);
    if (part < G::NX) {
      lds_u8* dst = base + (wid * G::NX + part) * 1024;
      if (res) dma16(rx, dst, xo[part] + uint32_t(s) * (kKS * 2));
      else dma16(rt, dst, xo[part] + uint32_t(s - nst) * 128);
    } else if (KIND == 1 ? sg_ahead == 0 : slot_start(s)) {
      const uint32_t k = uint32_t(KIND == 1 ? slot_ahead : slot_of(s)) * 1024u;
      if (part == G::NX) dma4(rrat, base + G::RAT + (wid & 3) * 256, ao_rat + k);
      else if (wid < TM / 64 && res) dma4(rbias, base + G::BIAS + wid * 256, ao_bias + k);
    }
  };
  // load CI (0 .. NC-1) of this wave's share of the codes of stages s, s + 1:
  // 64 bytes of a row (32-byte pieces, one stage's, stream the head 15% slower)
  auto issue_code = [&](int s, int ci, auto kind) {
    constexpr int KIND = decltype(kind)::value;
    lds_u8* dst = L + G::CODES + (wid * G::NC + ci) * 1024;
    if (KIND == 1 || (KIND == 3 && s < nst)) dma16(rc, dst, co[ci] + uint32_t(s) * (kKS / 2));
    else dma16(ru, dst, cunit(ci, urow) + uint32_t(s - nst) * 32);
  };
  using kMain = std::integral_constant<int, 1>;
  using kAny = std::integral_constant<int, 3>;
  auto issue = [&](int s, int buf) {
#pragma unroll
    for (int part = 0; part < G::NLX; ++part) issue_part(s, buf, part, kAny{});
  };

  // Fragment offsets within a stage.  Residual stages: half-wave h holds code
  // dwords 4h .. 4h + 3 (one 16-byte read) and takes x unit 4h + t in K-step t.
  // Expansion stages: K-step t is one part of t ([hi | mid | lo], units
  // 2t + h), against code dimensions 8h .. 8h + 7.
  const uint32_t arow = uint32_t(WM * wm + lr) * (2 * kKS);
  const uint32_t sx = uint32_t(swz_x(lr));
  uint32_t aoff[kSteps];
#pragma unroll
  for (int t = 0; t < kSteps; ++t) aoff[t] = arow + 16u * (uint32_t(4 * h + t) ^ sx);
  // codes of stage parity b: unit 2 b + h of the row's four
  const uint32_t brow = G::CODES + uint32_t(G::WN * wn + lr) * kKS;
  const uint32_t boff[2] = {brow + 16u * uint32_t(h ^ swz_c(lr)), brow + 16u * uint32_t((2 + h) ^ swz_c(lr))};

  f32x16_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[i][j][k] = 0.f;
  // the dense head's logits (fidelity pass): plain fp32 sums of bf16 products
  constexpr int MD = XE == 1 ? MI : 1;
  f32x16_t accd[MD][NI];
#pragma unroll
  for (int i = 0; i < MD; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) accd[i][j][k] = 0.f;
  // dense fragments (fidelity pass): of row WN wn + 32 ni + lr, the units
  // 4h + t of one stage; each is replaced by the next stage's right after its
  // MFMAs
  bf16x8_t dfr[XE == 1 ? NI : 1][kSteps];
  uint32_t dof[NI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) {
    const int c = G::WN * wn + 32 * ni + lr;
    dof[ni] = uint32_t(c < cols ? c : cols - 1) * dstride + 64u * uint32_t(h);
  }
  auto load_dense = [&](int s, int t) {
    if constexpr (XE == 1) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        dfr[ni][t] = __builtin_bit_cast(
            bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rd, dof[ni] + 16 * t, s * (2 * kKS), 0));
    }
  };

  // loaded before the stage loads, so it has arrived by the epilogue
  float rf[MI];   // 2^e of the lane's tokens
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) rf[mi] = a.rowexp[m0 + WM * wm + 32 * mi + lr];
  issue(0, 0);
#pragma unroll
  for (int ci = 0; ci < G::NC; ++ci) issue_code(0, ci, kAny{});
  pin_vmem_order();   // the first wait leaves the newest NX loads in flight: all of stage 1
  issue(1, 1);

  // slot start: rescale to the slot's scale and (residual groups) add its bias
  auto rescale = [&](const lds_u8* base, auto residual) {
    constexpr bool RES = decltype(residual)::value;
    float bias[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
      bias[mi] = RES ? lds_load<float>(base + G::BIAS + (WM * wm + 32 * mi + lr) * 4) : 0.f;
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f32x4_t rat = lds_load<f32x4_t>(base + G::RAT + (G::WN * wn + 32 * ni + 8 * k + 4 * h) * 4);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc[mi][ni][4 * k + i] = RES ? fmaf(acc[mi][ni][4 * k + i], rat[i], bias[mi])
                                         : acc[mi][ni][4 * k + i] * rat[i];
      }
  };

  // Stage s computes K-steps 0 .. 3.  Half way through it waits for its own
  // share of stage s + 1 and meets the other waves: stage s + 1 is then in
  // LDS, and every wave is past stage s - 1, whose ring slot takes the loads
  // of stage s + 2 (issued one at a time between the MFMAs that follow); where
  // s is even, so are the codes of stages s + 2, s + 3, in the place of those
  // of s, s + 1, which every wave has in registers by then.  The last K-step
  // reads the next stage's first fragments (and the next two stages' codes),
  // so no wave starts a stage waiting for LDS.
  bf16x8_t A[MI];
  u32x4_t braw[NI][2];
  const lds_u8* base = L;            // ring slot of the stage being computed
  int nslot_ring = 2 % kRing;        // ring slot of stage s + 2
  auto ring_next = [&](const lds_u8* p) {
    return p == L + (kRing - 1) * G::STAGE ? (const lds_u8*)L : p + G::STAGE;
  };
  auto load_codes = [&] {
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int b = 0; b < 2; ++b) braw[ni][b] = lds_load<u32x4_t>(L + boff[b] + ni * 32 * kKS);
  };
  auto load_first = [&](const lds_u8* p) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) A[mi] = lds_load<bf16x8_t>(p + aoff[0] + mi * 64 * kKS);
  };
  wait_loads_barrier<G::NX>();   // (there are two stages at least; stage 1 has at least NX loads in flight)
  load_codes();
  load_first(base);
  if constexpr (XE == 1) {
#pragma unroll
    for (int t = 0; t < kSteps; ++t) load_dense(0, t);
  }

  // issue_kind: kMain where stage s + 2 is a residual stage, else kAny (checked)
  int sg = 0;   // stage index within its scale group
  constexpr int kHalfMfma = (kSteps - kSteps / 2) * MI * NI;   // MFMA tiles after the barrier
  // loads of an even / odd stage issued after tile `tile` of them
  auto issue_after = [&](int s, int tile, auto issue_kind, auto parity) {
    constexpr int ISSUE = decltype(issue_kind)::value;
    constexpr int NCODE = decltype(parity)::value == 0 ? G::NC : 0, N = G::NLX + NCODE;
    constexpr int kPer = kHalfMfma / N > 0 ? kHalfMfma / N : 1;   // tiles between two loads
    constexpr int kBatch = (N + kHalfMfma - 1) / kHalfMfma;       // loads at a time
    if (tile % kPer) return;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int part = tile / kPer * kBatch + k;   // the codes first: they come from furthest
      if (part >= N) continue;
      auto one = [&](auto kind) {
        if (part < NCODE) issue_code(s + 2, part, kind);
        else issue_part(s + 2, nslot_ring, part - NCODE, kind);
      };
      if constexpr (ISSUE == 1) one(kMain{});
      if constexpr (ISSUE == 3) if (s + 2 < ntot) one(kAny{});
    }
  };
  auto ring_step = [&] {
    base = ring_next(base);
    nslot_ring = nslot_ring == kRing - 1 ? 0 : nslot_ring + 1;
  };
  auto main_stage = [&](int s, auto issue_kind, auto parity) {
    constexpr int PAR = decltype(parity)::value;
    const lds_u8* nbase = ring_next(base);
    // the wait below counts the dense loads of K-steps 0 and 1 as the newest
    // ones: none may be moved ahead of the loads to LDS of the stage before
    if constexpr (XE == 1) pin_vmem_order();
    if (sg == 0) rescale(base, std::true_type{});
#pragma unroll
    for (int t = 0; t < kSteps; ++t) {
      // (the fidelity pass has issued NI dense loads in each K-step so far,
      // after all of stage s + 1's)
      if (t == kSteps / 2) wait_loads_barrier<XE == 1 ? kSteps / 2 * NI : 0>();
      bf16x8_t B[NI];
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) B[ni] = unpack8_sub<XE != 0>(braw[ni][PAR][t]);
      bf16x8_t An[MI];
      if (t + 1 < kSteps) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) An[mi] = lds_load<bf16x8_t>(base + aoff[t + 1] + mi * 64 * kKS);
      } else {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) An[mi] = lds_load<bf16x8_t>(nbase + aoff[0] + mi * 64 * kKS);
      }
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(B[ni], A[mi], acc[mi][ni], 0, 0, 0);
          if constexpr (XE == 1)
            accd[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dfr[ni][t], A[mi], accd[mi][ni], 0, 0, 0);
          if (t >= kSteps / 2) issue_after(s, ((t - kSteps / 2) * MI + mi) * NI + ni, issue_kind, parity);
        }
      // (B holds this K-step's codes; the next stages' take their place)
      if (PAR == 1 && t == kSteps - 1) load_codes();
      load_dense(s + 1 < nres ? s + 1 : s, t);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) A[mi] = An[mi];
    }
    sg = sg == spg - 1 ? 0 : sg + 1;
    if (++sg_ahead == spg) {
      sg_ahead = 0;
      ++slot_ahead;
    }
    ring_step();
  };
  // the stage after an odd number of residual stages: only its share of the
  // loads, and the meeting
  auto empty_stage = [&](int s) {
    wait_loads_barrier<0>();
#pragma unroll
    for (int part = 0; part < G::NLX; ++part)
      if (s + 2 < ntot) issue_part(s + 2, nslot_ring, part, kAny{});
    load_codes();
    ring_step();
  };
  auto exp_stage = [&](int s, auto issue_kind, auto parity) {
    constexpr int PAR = decltype(parity)::value;
    if (s == nst || s == st_a) rescale(base, std::false_type{});
    bf16x8_t B[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
      // half h takes the copy in unit 2 PAR + h, dimensions 8 h .. 8 h + 7
      const u32x4_t c = braw[ni][PAR];
      B[ni] = int8x8_to_bf16(h ? c[2] : c[0], h ? c[3] : c[1]);
    }
#pragma unroll
    for (int t = 0; t < kExpParts; ++t) {
      if (t == kExpParts - 2) wait_loads_barrier<0>();
      const uint32_t eoff = arow + 16u * (uint32_t(2 * t + h) ^ sx);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        const bf16x8_t Ae = lds_load<bf16x8_t>(base + eoff + mi * 64 * kKS);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(B[ni], Ae, acc[mi][ni], 0, 0, 0);
          if (t >= kExpParts - 2)
            issue_after(s, ((t - kExpParts + 2) * MI + mi) * NI + ni, issue_kind, parity);
        }
      }
    }
    if (PAR == 1) load_codes();
    ring_step();
  };
  using Even = std::integral_constant<int, 0>;
  using Odd = std::integral_constant<int, 1>;
  int s = 0;
#pragma unroll 1
  for (; s + 3 < nres; s += 2) {
    main_stage(s, kMain{}, Even{});
    main_stage(s + 1, kMain{}, Odd{});
  }
#pragma unroll 1
  for (; s < nst; s += 2) {
    main_stage(s, kAny{}, Even{});
    if (s + 1 < nres) main_stage(s + 1, kAny{}, Odd{});
    else empty_stage(s + 1);
  }
#pragma unroll 1
  for (; s < ntot; s += 2) {
    exp_stage(s, kAny{}, Even{});
    if (s + 1 < ntot) exp_stage(s + 1, kAny{}, Odd{});
  }

  // the last slot's scales and the token's power of two (fidelity and rank:
  // the scales hold 2^-kXExp; dense sums: without the scale, and 2^-kXExpFid
  // apart, as 2^(e - kXExpFid) may be below fp32's range)
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      f32x4_t fin = *reinterpret_cast<const f32x4_t*>(a.fin + vt * kTN + G::WN * wn + 32 * ni + 8 * k + 4 * h);
      if constexpr (XE != 0) fin *= ldexpf(1.f, kXExp - kXExpFid);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[mi][ni][4 * k + i] = acc[mi][ni][4 * k + i] * fin[i] * rf[mi];
          if constexpr (XE == 1)
            accd[mi][ni][4 * k + i] = accd[mi][ni][4 * k + i] * ldexpf(1.f, -kXExpFid) * rf[mi];
        }
    }

  // ---- epilogue: a lane holds, of token block mi, the token lr and the tile
  // columns col0(ni, i) + 4 h; rising with (ni, i)
  auto col_of = [&](int ni, int i) { return G::WN * wn + 32 * ni + 8 * (i >> 2) + 4 * h + (i & 3); };
  auto tok_of = [&](int mi) { return WM * wm + 32 * mi + lr; };
  const bool partial = cols < kTN;
  if constexpr (XE == 1) {
    // per token of the tile: the FidTilePart of its valid columns (a the
    // dense logit, b the packed one); the two half-waves share tokens, the
    // four waves along the vocabulary merge through LDS in order
    FidTilePart* sp = reinterpret_cast<FidTilePart*>(mfma_lds);   // [4][TM]
    __syncthreads();
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      float ma = -INFINITY, mb = -INFINITY, bat = -INFINITY;
      int ia = kNoCol, ib = kNoCol;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int col = col_of(ni, i);
          if (partial && col >= cols) continue;
          const float av = accd[mi][ni][i], bv = acc[mi][ni][i];
          const bool up = av > ma;   // strict: the first maximum stays
          ma = up ? av : ma;
          ia = up ? col : ia;
          bat = up ? bv : bat;
          ib = bv > mb ? col : ib;
          mb = fmaxf(mb, bv);
        }
      const float oma = __shfl_xor(ma, 32, 64), obat = __shfl_xor(bat, 32, 64);
      const int oia = __shfl_xor(ia, 32, 64);
      const bool other = oma > ma || (oma == ma && oia < ia);
      ma = other ? oma : ma;
      bat = other ? obat : bat;
      ia = other ? oia : ia;
      const float omb = __shfl_xor(mb, 32, 64);
      const int oib = __shfl_xor(ib, 32, 64);
      ib = omb > mb ? oib : (omb == mb ? min(ib, oib) : ib);
      mb = fmaxf(mb, omb);
      // in groups of 4, of 16 and of all 32: 7 roundings (the tree of
      // tree_sum spills here)
      float sa = 0.f, sb = 0.f, t = 0.f, sq = 0.f;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
        float na = 0.f, nb = 0.f, nt = 0.f, nq = 0.f;
#pragma unroll
        for (int k = 0; k < 16; k += 4) {
          float ga = 0.f, gb = 0.f, gt = 0.f, gq = 0.f;
#pragma unroll
          for (int i = k; i < k + 4; ++i) {
            if (partial && col_of(ni, i) >= cols) continue;
            const float av = accd[mi][ni][i], bv = acc[mi][ni][i];
            const float ea = expf(av - ma), dd = av - bv;
            ga += ea;
            gb += expf(bv - mb);
            gt += ea * dd;
            gq += dd * dd;
          }
          na += ga;
          nb += gb;
          nt += gt;
          nq += gq;
        }
        sa += na;
        sb += nb;
        t += nt;
        sq += nq;
      }
      sa += __shfl_xor(sa, 32, 64);
      sb += __shfl_xor(sb, 32, 64);
      t += __shfl_xor(t, 32, 64);
      sq += __shfl_xor(sq, 32, 64);
      if (h == 0) sp[wn * TM + tok_of(mi)] = FidTilePart{ma, mb, bat, sa, sb, t, sq, ia | ib << 16};
    }
    __syncthreads();
    if (tid < rows) {
      FidTilePart r = sp[tid];   // wave 0 holds column 0, always valid
      int ia = r.iab & 0xffff, ib = r.iab >> 16;
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        const FidTilePart o = sp[w * TM + tid];
        if (o.ma > r.ma) {
          const float f = expf(r.ma - o.ma);
          r.sa = r.sa * f + o.sa;
          r.t = r.t * f + o.t;
          r.ma = o.ma;
          ia = o.iab & 0xffff;
          r.bat = o.bat;
        } else if (o.ma > -INFINITY) {   // equal maxima keep the smaller index (this wave's)
          const float f = expf(o.ma - r.ma);
          r.sa += o.sa * f;
          r.t += o.t * f;
        }
        if (o.mb > r.mb) {
          r.sb = r.sb * expf(r.mb - o.mb) + o.sb;
          r.mb = o.mb;
          ib = o.iab >> 16;
        } else if (o.mb > -INFINITY) {
          r.sb += o.sb * expf(o.mb - r.mb);
        }
        r.sq += o.sq;
      }
      r.iab = ia | ib << 16;
      reinterpret_cast<FidTilePart*>(a.fid_part)[(m0 + tid) * a.n_vt + vt] = r;
    }
    if (tid < TM / 64 && m0 + 64 * tid < a.M) a.fid_need[(m0 / 64 + tid) * a.n_vt + vt] = 0;
  } else if constexpr (XE == 2) {
    // per token: the packed logits of this tile ranked ahead of the
    // reference's top-1 (larger, or equal at a smaller index), added to rank
    int* scnt = reinterpret_cast<int*>(mfma_lds);   // [4][TM]
    __syncthreads();
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      const bool ok = tok_of(mi) < rows;
      const float br = ok ? a.bref[m0 + tok_of(mi)] : 0.f;
      const int64_t dr = ok ? a.ref_idx[m0 + tok_of(mi)] - v0 : -1;
      const int ri = dr < 0 ? -1 : (dr > kTN ? kTN : int(dr));
      int c = 0;
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int col = col_of(ni, i);
          const float bv = acc[mi][ni][i];
          c += (col < cols) & ((bv > br) | ((bv == br) & (col < ri)));
        }
      c += __shfl_xor(c, 32, 64);
      if (h == 0) scnt[wn * TM + tok_of(mi)] = c;
    }
    __syncthreads();
    if (tid < rows) {
      const int tot = scnt[tid] + scnt[TM + tid] + scnt[2 * TM + tid] + scnt[3 * TM + tid];
      if (tot) atomicAdd(reinterpret_cast<unsigned long long*>(a.rank + m0 + tid),
                         (unsigned long long)tot);
    }
  } else if constexpr (!CE) {
    // Each wave turns 32 tokens x 64 columns at a time through its own part
    // of the LDS, so 16 lanes store 64 consecutive logits of a token (a lane's
    // own four would be 16 bytes of a row each).
    __syncthreads();
    float* const buf = reinterpret_cast<float*>(mfma_lds) + wid * 32 * kOutStride;
    const int c0 = G::WN * wn;
    // four logits per lane where every row starts on a 4-element boundary of the output type
    const uintptr_t oa = reinterpret_cast<uintptr_t>(a.out);
    const bool vec = a.ldo % 4 == 0 && oa % (a.out_bf16 ? 8 : 16) == 0;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          *reinterpret_cast<f32x4_t*>(buf + lr * kOutStride + 32 * ni + 8 * k + 4 * h) =
              f32x4_t{acc[mi][ni][4 * k], acc[mi][ni][4 * k + 1], acc[mi][ni][4 * k + 2], acc[mi][ni][4 * k + 3]};
      const int r0 = WM * wm + 32 * mi;
      if (vec) {
        const int cc = 4 * (lane & 15);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int rl = 4 * j + (lane >> 4);
          const f32x4_t l = *reinterpret_cast<const f32x4_t*>(buf + rl * kOutStride + cc);
          if (r0 + rl >= rows || c0 + cc >= cols) continue;
          const int64_t o = (m0 + r0 + rl) * a.ldo + v0 + c0 + cc;
          if (c0 + cc + 4 <= cols) {
            if (a.out_bf16)
              *reinterpret_cast<u32x2_t*>(reinterpret_cast<uint16_t*>(a.out) + o) =
                  u32x2_t{uint32_t(f32_to_bf16_rne(l[0])) | uint32_t(f32_to_bf16_rne(l[1])) << 16,
                          uint32_t(f32_to_bf16_rne(l[2])) | uint32_t(f32_to_bf16_rne(l[3])) << 16};
            else
              *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(a.out) + o) = l;
          } else {
            for (int i = 0; c0 + cc + i < cols; ++i) {
              const float li = i == 0 ? l[0] : (i == 1 ? l[1] : l[2]);
              if (a.out_bf16) reinterpret_cast<uint16_t*>(a.out)[o + i] = f32_to_bf16_rne(li);
              else reinterpret_cast<float*>(a.out)[o + i] = li;
            }
          }
        }
      } else {
#pragma unroll 8
        for (int rl = 0; rl < 32; ++rl) {
          const float l = buf[rl * kOutStride + lane];
          if (r0 + rl >= rows || c0 + lane >= cols) continue;
          const int64_t o = (m0 + r0 + rl) * a.ldo + v0 + c0 + lane;
          if (a.out_bf16) reinterpret_cast<uint16_t*>(a.out)[o] = f32_to_bf16_rne(l);
          else reinterpret_cast<float*>(a.out)[o] = l;
        }
      }
    }
  } else {
    // per token: (max, sum exp) over this tile's valid columns; the two
    // half-waves share tokens, the four waves along the vocabulary are merged
    // through LDS in a fixed order.
    float2* sred = reinterpret_cast<float2*>(mfma_lds);               // [4][TM]
    int* sidx = reinterpret_cast<int*>(mfma_lds + 4 * TM * sizeof(float2));   // [4][TM] argmax
    __syncthreads();
    if (partial) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int mi = 0; mi < MI; ++mi)
            if (col_of(ni, i) >= cols) acc[mi][ni][i] = -INFINITY;
    }
    // IDX: also the smallest tile column at each token's maximum (argmax
    // partials); compiled apart so the CE-only pass pays nothing for it
    auto rows_pass = [&](auto IDX) {
      constexpr bool kIdx = decltype(IDX)::value;
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        float mx = -INFINITY;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[mi][ni][i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float ref = mx == -INFINITY ? 0.f : mx;   // no valid column: a sum of zeros
        float se = tree_sum<0, 16 * NI>([&](auto c) {
          return fast_exp(acc[mi][decltype(c)::value / 16][decltype(c)::value % 16] - ref);
        });
        int ai = kNoIdx;
        if constexpr (kIdx) {
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (acc[mi][ni][i] == mx && col_of(ni, i) < cols) ai = min(ai, col_of(ni, i));
        }
        se += __shfl_xor(se, 32, 64);
        if constexpr (kIdx) ai = min(ai, __shfl_xor(ai, 32, 64));
        if (h == 0) {
          sred[wn * TM + tok_of(mi)] = make_float2(mx, se);
          if constexpr (kIdx) sidx[wn * TM + tok_of(mi)] = ai;
        }
      }
    };
    if (a.part_idx)
      rows_pass(std::true_type{});
    else
      rows_pass(std::false_type{});
    // the target's logit, by the lane that holds it (few waves hold any)
    if (a.tgt) {
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        const int64_t m = m0 + tok_of(mi);
        int64_t y = -1;
        if (tok_of(mi) < rows)
          y = a.tgt64 ? reinterpret_cast<const int64_t*>(a.tgt)[m]
                      : int64_t(reinterpret_cast<const int32_t*>(a.tgt)[m]);
        const int yl = y >= v0 + G::WN * wn && y < v0 + cols && y < v0 + G::WN * (wn + 1) ? int(y - v0) : -1;
        if (__ballot(yl >= 0)) {
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (col_of(ni, i) == yl) a.tgt_logit[m] = acc[mi][ni][i];
        }
      }
    }
    __syncthreads();
    if (tid < rows) {
      float m_ = sred[tid].x, s_ = sred[tid].y;
#pragma unroll
      for (int w = 1; w < 4; ++w) lse_merge(m_, s_, sred[w * TM + tid].x, sred[w * TM + tid].y);
      a.part[(m0 + tid) * a.n_vt + vt] = make_float2(m_, s_);
      if (a.part_idx) {
        int ai = kNoIdx;
#pragma unroll
        for (int w = 0; w < 4; ++w)
          if (sred[w * TM + tid].x == m_) ai = min(ai, sidx[w * TM + tid]);
        a.part_idx[(m0 + tid) * a.n_vt + vt] = ai == kNoIdx ? kNoIdx : int(v0) + ai;
      }
    }
  }
}

// ---------------------------------------------------- MFMA path: prologue
// Per call, before stage 1, or once per head: (a) per vocabulary tile and
// column the scale ratios of the accumulator's scale slots (residual groups
// 0 .. d/g-1, then s_U if r_c > 0, then s_A if r_r > 0): ratio[vt][k][c] =
// s'_{k-1} / s'_k (0 for k = 0) and fin[vt][c] = s' of the last slot times
// 2^-(kXExp + kCodeExp), where s' is the fp16 scale with zero replaced by
// kZeroScale; columns past V repeat row V-1;
// (b) the codes of U_c and A_w side by side per vocabulary
// row, each part zero-padded to a multiple of 16 dimensions, each block of 16
// stored twice.
struct PrepArgs {
  const uint16_t* rs;
  const uint16_t* rrs;   // row scales of 8-bit group scale codes, or null (fp16 scales)
  const uint16_t* su;
  const uint16_t* sa;
  int64_t V;
  int ngrp, nslot;
  int64_t n_vt;
  float* ratio;
  float* fin;
  int rc, rr, d;
  const int8_t* cu;
  const int8_t* ca;
  int urow, rc_pad;      // bytes per ucodes row; padded dimensions of the U part
  int8_t* ucodes;
  int cu_row;            // bytes per row of U_c (r_c int8 codes, or ARCHEAD_I5 words)
  int u5;                // U_c codes are ARCHEAD_I5 words
  int blocks;            // k_stage1m: leading workgroups that build the tables
};

__device__ __forceinline__ float nz_scale(uint16_t h) {
  const float s = f16_to_f32(h);
  return s == 0.f ? kZeroScale : s;
}

// ---------------------------------------------------- MFMA path: stage 1
// Two launches.  k_stage1m: t[m, k] = sum over factor groups of s[k, grp] *
// (sum over the group of c[k, i] x[m, i]) for the R factor rows (V_c then
// B_w) as ksplit fp32 partials, and the sums of x over the residual groups;
// a workgroup takes 16 tokens, up to 64 factor rows and 1 / ksplit of d; its
// eight waves split d by residual groups and each holds 16 x 64 outputs as
// four 16x16 MFMA tiles, loading the next K-chunk's fragments before the
// current chunk's MFMAs; an extra MFMA against a column of ones gives the
// sums of x; the eight partial results are summed in LDS in a fixed order.
// The launch's further workgroups each scale one token's x for the tiled
// kernel: xs = x 2^(kXExp - e), e the exponent of the row's largest magnitude
// (rowexp = 2^e), and another 2^-4 at elements 2, 3, 6, 7 of every 8 (the odd
// code pairs; exact); for the passes that read a dense head (`even`) xs = x
// 2^(kXExpFid - e).  k_stage1m_fin: with that scale and the codes' 2^kCodeExp, t as three bf16 parts hi, mid, lo, laid out per block
// of 16 rank dimensions as [hi | mid | lo | 0], the U_c part's blocks first,
// each part zero-padded to whole blocks, and the slot biases -8 * (sum of x).
struct Stage1MArgs {
  const uint16_t* x;
  int64_t ldx, M;
  int d, g;
  const int8_t* cv;        // [rc][d] V_c codes
  const int8_t* cb;        // [rr][d] B_w codes
  const uint16_t* sv;
  int gv, rc;
  const uint16_t* sb;
  int gb, rr;
  uint16_t* tsplit;        // [M] rows of ldxs: [nch][4][16] (hi, mid, lo, 0)
  int nch, nch_u;
  float* gbias;            // [n_mt][d / g][kTM]
  float* gsum;             // [d / g][M] sums of x over the residual groups
  int ksplit;              // workgroups along d
  float* tpart;            // [ksplit][M][R]
  uint16_t* xs;            // [M][ldxs] scaled x, followed in each row by t's parts
  int ldxs;
  float* rowexp;           // [n_mt][kTM] 2^e
  int even;
  int mblocks, rblocks;    // stage-1 workgroups: mblocks * rblocks * ksplit, then M for xs
};

constexpr int kS1MTok = 16, kS1MCols = 64, kS1MBlock = 512, kS1MWaves = kS1MBlock / 64;
// Workgroups of the two launches along x; more go on along y (2^22 of
// kS1MBlock threads stay below the 2^32 of a launch's dimension).
constexpr int64_t kGridX = int64_t(1) << 22;
// (a launch with rows along y has kGridX along x: no read of the grid's size)
__device__ __forceinline__ int64_t stage1_block() { return int64_t(blockIdx.y) * kGridX + blockIdx.x; }

}  // namespace
