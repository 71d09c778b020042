// Small-batch (decode) expert FFN over packed experts: gate/up + SwiGLU
// (body in decode_dev.h) and the down projection with the weighted combine.
//
// With one to a few tokens per expert the step is bound by streaming the
// packed int8 bytes from HBM.  Both kernels feed those bytes unchanged to the
// int8 matrix cores (v_mfma_i32_16x16x64_i8): the activation side is written
// as a fixed-point integer split into signed base-256 digits, each digit one
// int8 operand column, so the products and sums are exact int32 and the only
// rounding is the fixed-point step and the final fp32 arithmetic.  x has three
// digits (2^-22 of the token's maximum); H' three (2^-22 of its 64-row block
// maximum) when the call has at most 5 tokens, else two (2^-14).  A one-token
// call instead gives every 16-row tile of H' its own exponent (three digits):
// its gate/up splits the tiles evenly over the CUs, and its down kernel gives
// each (tile, digit) pair of a k-step its own operand column.  Since the
// shared scale sigma_r factors out (section IV-B), y = Qd H' with
// H' = sigma (.) silu(G) (.) U.
#include "decode_dev.h"
#include "route_dev.h"

namespace mira {

// ---------------------------------------------------------------------------
// Gate/up + SwiGLU of calls with several tokens.  Workgroup = (non-empty
// expert a, block of 64 rows of R); the digits of x come from the workspace
// (xdig[(t*3 + d)*C + c], written by the decode preparation kernel).
// ---------------------------------------------------------------------------
// With XL (INT4, one token group, C <= kXlMaxC) the workgroup first copies
// the digit rows of its tokens into LDS (row stride C + 16 bytes, so the 16
// rows a read phase touches fall in distinct banks) and the loop reads them
// from there.
constexpr int kXlMaxC = 4096;
inline uint32_t xl_bytes(int C) { return 3 * kTokPerGroup * (C + 16); }
// k-steps per weight batch: with the digits in LDS, 8 steps let three waves
// share a SIMD; fine-grained layer, 4 / 16 tokens: 50.0 / 96.0 us per call
// against 50.8 / 99.7 with 16 steps (and 50.0 / 95.4 with 6, which costs the
// Mixtral shape 2%)
constexpr int kXlUnroll = 8;
// the same for an INT8 expert of one token group in a call of several: the
// body shares its registers with the wider ones.  us per call with 4 / 8 / 16
// steps: Mixtral shape, 13 tokens 242.0 / 238.0 / 237.4; fine-grained layer, 9
// tokens 59.3 / 57.9 / 57.4; but 16 steps do not fit three workgroups per CU
// (kThreePerCuMaxC), where they spill: C 1024, R 4096, 6 tokens 41.5 / 41.6 / 61.9
constexpr int kOneGroupUnroll = 8;
// k-steps per weight batch of the one-token INT4 tile kernel (6 KB per wave):
// a wave holds one tile and cannot issue its next loads while it unpacks and
// scales a batch, and shorter batches measured faster than 4, 8 or 16 steps
constexpr int kTileI4Unroll = 6;

// One (expert, row block) of a gate/up call for an expert of at most NG token
// groups (wk, resolved slot), H' in HD digits.
template <int NG, int NGMAX, int HD, bool I4, bool XL>
__device__ __forceinline__ void decode_gateup_body(int C, int R, int rb, int slot,
                                                   const ExpertPool& ep, const DecodeWork& wk,
                                                   const int8_t* __restrict__ xdig,
                                                   int8_t* __restrict__ hdig,
                                                   int32_t* __restrict__ hexp,
                                                   float (*bmax)[kDecodeMaxGroups * kTokPerGroup]) {
  const int n = wk.n;
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, kg = lane >> 4;
  const int m = r16 / 3, d = r16 - 3 * m;
  const int8_t* bp[NG];
  bool bv[NG];
  int xev[NG];
#pragma unroll
  for (int cg = 0; cg < NG; ++cg) {
    const int i = cg * kTokPerGroup + m;
    bv[cg] = r16 < 3 * kTokPerGroup && i < n;
    const int tok = bv[cg] ? wk.tok[i] : 0;
    xev[cg] = bv[cg] ? wk.xe[i] : 0;
    bp[cg] = xdig + ((size_t)tok * kDigits + d) * C + kg * 16;
  }
  if constexpr (XL) {
    static_assert(NG == 1, "one token group in LDS");
    extern __shared__ __attribute__((aligned(16))) int8_t xl[];  // xl_bytes(C)
    const int ld = C + 16;
    const int chunks = C / 16;
    // only the digit rows of the group's tokens are staged; lanes of the
    // other columns take a zero operand without reading LDS
    const int rows = 3 * min(n, kTokPerGroup);
    for (int i = threadIdx.x; i < rows * chunks; i += 256) {
      const int row = i / chunks, c16 = i - row * chunks;
      const int cg = row >> 4, col = row & 15;
      const int mm = col / 3, dd = col - 3 * mm, ti = cg * kTokPerGroup + mm;
      v4i v = zero16();
      if (col < 3 * kTokPerGroup && ti < n)
        v = ld16(xdig + ((size_t)wk.tok[ti] * kDigits + dd) * C + c16 * 16);
      *(v4i*)(xl + (size_t)row * ld + c16 * 16) = v;
    }
    __syncthreads();
    const int8_t* xr[NG];
#pragma unroll
    for (int cg = 0; cg < NG; ++cg) xr[cg] = xl + (size_t)(cg * 16 + r16) * ld + kg * 16;
    const auto load_x = [&](int cg, int ks) { return bv[cg] ? *(const v4i*)(xr[cg] + ks * 64) : zero16(); };
    gateup_block_i4<NG, HD, kXlUnroll, true>(C, R, rb, (const uint8_t*)ep.pool + (size_t)slot * ep.stride,
                                             wk.off, bv, xev, load_x, hdig, hexp, bmax);
    return;
  }
  const auto load_b = [&](int cg, int ks) { return ld16(bp[cg] + ks * 64); };
  if constexpr (I4)
    gateup_block_i4<NG, HD, dec_unroll(NG), false>(C, R, rb,
                                                   (const uint8_t*)ep.pool + (size_t)slot * ep.stride,
                                                   wk.off, bv, xev, load_b, hdig, hexp, bmax);
  else
    gateup_block<NG, HD, (NGMAX > 1 && NG == 1) ? kOneGroupUnroll : dec_unroll(NG)>(
        C, R, rb, ep.pool + (size_t)slot * ep.stride, wk.off, bv, xev, load_b, hdig, hexp, bmax);
}

// Workgroup = (non-empty expert, 64-row block) of a call that NGMAX token
// groups cover; the expert's own token count chooses the body (most experts
// of a call hold a few of its tokens, and a body for fewer groups spends
// fewer matrix-core steps and holds longer weight batches).  INT4, whose loop
// is not a pure stream, gains most: Mixtral shape, 12 / 16 tokens, 199 / 238
// -> 184 / 210 us per call.  INT8 is bound by the stream: 8 / 12 tokens
// 194.7 / 244.7 -> 192.6 / 238.7 us, and at four groups the narrow bodies are
// no faster (262.5 / 263.4) and the fine-grained layer 2% slower, so that call
// keeps one body.
template <int NGMAX, bool I4, bool XL>
__device__ __forceinline__ void decode_gateup_groups(int C, int R, const ExpertPool& ep,
                                                     DecodeWork* __restrict__ work,
                                                     const int8_t* __restrict__ xdig,
                                                     int8_t* __restrict__ hdig,
                                                     int32_t* __restrict__ hexp) {
  constexpr int HD = h_digits(NGMAX);
  __shared__ float bmax[4][kDecodeMaxGroups * kTokPerGroup];
  const int nrb = R / kBlk;
  const int a = blockIdx.x / nrb, rb = blockIdx.x - a * nrb;
  const DecodeWork& wk = work[a];
  const int g = wk.group;
  if (g < 0) return;
  const int slot = ep.slot_table[g];  // read now: the table may change after routing
  const bool ok = slot >= 0 && slot < ep.n_slots;
  // block 0 of the expert keeps the resolved slot for the down kernel
  if (rb == 0 && threadIdx.x == 0) work[a].slot = ok ? slot : -1;
  if (!ok) {
    if (threadIdx.x == 0 && ep.status) atomicOr(ep.status, slot < 0 ? 1 : 2);
    return;
  }
  const int n = wk.n;
  constexpr bool by_count = NGMAX > 1 && (I4 || NGMAX < 4);
  if (NGMAX == 1 || (by_count && n <= kTokPerGroup))
    decode_gateup_body<1, NGMAX, HD, I4, XL>(C, R, rb, slot, ep, wk, xdig, hdig, hexp, bmax);
  else if (NGMAX == 2 || (by_count && n <= 2 * kTokPerGroup))
    decode_gateup_body<NGMAX < 2 ? NGMAX : 2, NGMAX, HD, I4, false>(C, R, rb, slot, ep, wk, xdig, hdig, hexp, bmax);
  else
    decode_gateup_body<NGMAX, NGMAX, HD, I4, false>(C, R, rb, slot, ep, wk, xdig, hdig, hexp, bmax);
}

// WG workgroups per CU (waves per SIMD) at least.
template <int NGMAX, bool I4, int WG>
__global__ __launch_bounds__(256, WG) void decode_gateup_kernel(int C, int R, ExpertPool ep,
                                                                DecodeWork* __restrict__ work,
                                                                const int8_t* __restrict__ xdig,
                                                                int8_t* __restrict__ hdig,
                                                                int32_t* __restrict__ hexp) {
  decode_gateup_groups<NGMAX, I4, false>(C, R, ep, work, xdig, hdig, hexp);
}

// The INT4 variant with the digits of one-group experts in LDS: at most
// 62 KB (C = 4096), so that two or more workgroups share a CU.
template <int NGMAX>
__global__ __launch_bounds__(256, 2) void decode_gateup_xl_kernel(int C, int R, ExpertPool ep,
                                                                 DecodeWork* __restrict__ work,
                                                                 const int8_t* __restrict__ xdig,
                                                                 int8_t* __restrict__ hdig,
                                                                 int32_t* __restrict__ hexp) {
  decode_gateup_groups<NGMAX, true, true>(C, R, ep, work, xdig, hdig, hexp);
}

// One-token calls: every wave streams one 16-row tile of the concatenated
// rows of the active experts (tile t = expert a, rows 16*(t mod R/16) ..)
// and writes that tile's H' with its own exponent (h_tile_1tok), so no wave
// waits for another and the host splits the tiles evenly over the CUs (W
// waves per workgroup, about one workgroup per CU).  The wave of tile 0 of
// each expert also stores the slot it resolved from the table in the
// expert's descriptor (-1 if invalid), for the down kernel.
//
// With SEL (the whole layer in one call, E <= 64) no selection kernel runs
// between the router logits and this one: every wave selects from the logits
// itself (one expert per lane, as decode_work_one_token), the waves of tile 0
// write the descriptors and the last wave of the grid, which a ragged split
// leaves idle, the optional outputs.  The selection replaces the load of a
// descriptor and costs this kernel 0.3 us (8 experts) to 1.5 us (64 experts
// top-6), a selection kernel 5.5 us and a boundary: 31.4 -> 27.1 us per call of
// the fine-grained layer, 64.9 -> 64.8 us of Mixtral's (whose preparation was
// one launch already).
constexpr int kTileMaxWaves = 8;

// What a SEL kernel selects from, and the optional outputs.
struct OneTokenSel {
  const float* logits;  // [E]
  const int32_t* xe;    // the token's fixed-point exponent
  int E, k, S, softmax_all;
  PermOut o;
};

// The expert and slot of a wave's tile.
struct TileExpert {
  int slot;    // -1 if invalid
  int off, xe; // permuted position; fixed-point exponent
  bool any;    // the expert has the token
};

template <bool SEL>
__device__ __forceinline__ bool tile_expert(int a, bool first, bool outputs, const ExpertPool& ep,
                                            DecodeWork* __restrict__ work, const OneTokenSel& q,
                                            TileExpert& te) {
  const int lane = threadIdx.x & 63;
  if constexpr (!SEL) {
    const DecodeWork& wk = work[a];
    const int g = wk.group;
    if (g < 0) return false;
    const int slot = ep.slot_table[g];  // read now: the table may change after routing
    const bool ok = slot >= 0 && slot < ep.n_slots;
    if (first && lane == 0) work[a].slot = ok ? slot : -1;
    if (!ok) {
      if (lane == 0 && ep.status) atomicOr(ep.status, slot < 0 ? 1 : 2);
      return false;
    }
    te = TileExpert{slot, wk.off, wk.xe[0], wk.n > 0};
    return true;
  } else {
    const int E = q.E, k = q.k, S = q.S;
    const int slot_r = lane < E ? ep.slot_table[lane] : 0;
    const int slot_s = lane < S ? ep.slot_table[E + lane] : 0;
    const int xe = *q.xe;
    bool sel;
    int rank;
    float w;
    topk_lane64(q.logits, E, k, q.softmax_all, sel, rank, w);
    const uint64_t mask = __ballot(sel);
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int at = __popcll(mask & lt);  // position among the selected experts
    if (outputs) {
      const PermOut& o = q.o;
      if (sel) {
        if (o.idx_out) o.idx_out[rank] = lane;
        if (o.w_out) o.w_out[rank] = w;
        if (o.order_out) o.order_out[at] = rank;
      }
      if (lane < E) {
        if (o.counts_out) o.counts_out[lane] = sel ? 1 : 0;
        if (o.offsets_out) o.offsets_out[lane] = at;
      }
      if (lane < S) {
        if (o.order_out) o.order_out[k + lane] = k + lane;
        if (o.counts_out) o.counts_out[E + lane] = 1;
        if (o.offsets_out) o.offsets_out[E + lane] = k + lane;
      }
      if (lane == 0 && o.offsets_out) o.offsets_out[E + S] = k + S;
      const bool lo = (sel && slot_r < 0) || (lane < S && slot_s < 0);
      const bool hi = (sel && slot_r >= ep.n_slots) || (lane < S && slot_s >= ep.n_slots);
      const int st = (__ballot(lo) ? 1 : 0) | (__ballot(hi) ? 2 : 0);
      if (lane == 0 && ep.status) *ep.status = st;
    }
    if (a < 0) return false;
    // group a: the a-th selected expert, then the shared ones
    int g, slot;
    float wa = 1.f;
    if (a < k) {
      g = __builtin_ctzll(__ballot(sel && at == a));
      slot = __builtin_amdgcn_readlane(slot_r, g);
      wa = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), g));
    } else {
      g = E + a - k;
      slot = __builtin_amdgcn_readlane(slot_s, a - k);
    }
    const bool ok = slot >= 0 && slot < ep.n_slots;
    if (first && lane == 0) {
      DecodeWork* wk = work + a;
      wk->group = g;
      wk->slot = ok ? slot : -1;
      wk->off = a;
      wk->n = 1;
      wk->tok[0] = 0;
      wk->xe[0] = xe;
      wk->w[0] = wa;
    }
    te = TileExpert{slot, a, xe, true};
    return ok;
  }
}

template <bool SEL>
__global__ __launch_bounds__(64 * kTileMaxWaves) void decode_gateup_tile_kernel(
    int C, int R, int W, int ntiles, ExpertPool ep, DecodeWork* __restrict__ work, OneTokenSel q,
    const int8_t* __restrict__ xdig, int8_t* __restrict__ hdig, int32_t* __restrict__ hexp) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = blockIdx.x * W + wave;
  const bool outputs = SEL && blockIdx.x == gridDim.x - 1 && wave == W - 1;
  if (wave >= W || (t >= ntiles && !outputs)) return;
  const int tpe = R / 16;
  const int a = t < ntiles ? t / tpe : -1, rt = t - a * tpe;
  TileExpert te;
  if (!tile_expert<SEL>(a, rt == 0, outputs, ep, work, q, te)) return;
  const int r16 = lane & 15, kg = lane >> 4;
  const bool bv = r16 < 3 && te.any;
  // a one-token call's only token is token 0
  const int8_t* bp = xdig + (size_t)(bv ? r16 : 0) * C + kg * 16;
  const auto load_b = [&](int, int ks) { return ld16(bp + ks * 64); };
  // seven 16-row tiles per CU at Mixtral's shape: one wave per tile beat two
  // waves per tile (gate and up streamed apart, up sums handed over in LDS)
  // by 0.45 us per call
  v4i accg[1], accu[1];
  float sg[4];
  const bool bva[1] = {bv};
  gateup_tile_stream<1, dec_unroll(1)>(C, R, rt, ep.pool + (size_t)te.slot * ep.stride, bva, load_b, accg,
                                       accu, sg);
  h_tile_1tok(R, rt, te.off, bv, te.xe, accg[0], accu[0], sg, hdig, hexp);
}

// One-token INT4 calls (C <= kXlMaxC): the same tile split, with the
// token's three digit rows copied into LDS once per workgroup (row stride
// C + 16 bytes), so a wave's batches hold only weight registers.  A one-token
// call's only token is token 0, whatever expert a tile belongs to.
template <bool SEL>
__global__ __launch_bounds__(64 * kTileMaxWaves) void decode_gateup_tile_i4_kernel(
    int C, int R, int W, int ntiles, ExpertPool ep, DecodeWork* __restrict__ work, OneTokenSel q,
    const int8_t* __restrict__ xdig, int8_t* __restrict__ hdig, int32_t* __restrict__ hexp) {
  __shared__ __attribute__((aligned(16))) int8_t xl[kDigits * (kXlMaxC + 16)];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ld = C + 16, chunks = C / 16;
  for (int i = threadIdx.x; i < kDigits * chunks; i += blockDim.x) {
    const int row = i / chunks, c16 = i - row * chunks;
    *(v4i*)(xl + (size_t)row * ld + c16 * 16) = ld16(xdig + (size_t)row * C + c16 * 16);
  }
  __syncthreads();
  const int t = blockIdx.x * W + wave;
  const bool outputs = SEL && blockIdx.x == gridDim.x - 1 && wave == W - 1;
  if (wave >= W || (t >= ntiles && !outputs)) return;
  const int tpe = R / 16;
  const int a = t < ntiles ? t / tpe : -1, rt = t - a * tpe;
  TileExpert te;
  if (!tile_expert<SEL>(a, rt == 0, outputs, ep, work, q, te)) return;
  const int r16 = lane & 15, kg = lane >> 4;
  const bool bv = r16 < 3 && te.any;
  const int xe = te.xe;
  const int8_t* xr = xl + (size_t)(bv ? r16 : 0) * ld + kg * 16;
  const auto load_x = [&](int, int ks) { return bv ? *(const v4i*)(xr + ks * 64) : zero16(); };
  float accg[1][4], accu[1][4];
  const bool bva[1] = {bv};
  gateup_tile_stream_i4<1, kTileI4Unroll, true>(C, R, rt, (const uint8_t*)ep.pool + (size_t)te.slot * ep.stride,
                                                bva, load_x, accg, accu);
  // 2^-E of the token's fixed point, and 1/16 for the nibble operand (16*q)
  const bool lead = bv && r16 == 0;
  const float xs = bv ? ldexpf(1.f, -xe - 4) : 0.f;
  float hv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float gv = combine_digits_f(accg[0][i]) * xs;
    const float uv = combine_digits_f(accu[0][i]) * xs;
    const float h = gv / (1.f + expf(-gv)) * uv;
    hv[i] = lead ? h : 0.f;
  }
  write_h_tile_1tok(R, rt, te.off, lead, hv, hdig, hexp);
}

// ---------------------------------------------------------------------------
// Down projection + weighted combine.  Workgroup = 16 output rows c, or an
// equal part of their k-steps (64 entries of R each): the KS waves of the one to
// four workgroups of a row tile split the k-steps of the non-empty experts.
// For every expert, y = Qd H' with per-64-row exponents of H', multiplied by
// the combine weight of each (token, expert) pair and summed per token in a
// fixed order (expert list order inside a wave, then wave order, then the
// partial outputs of the workgroups in order, by decode_add_kernel), so the
// result is deterministic.  H' has HD digits per entry (h_digits): an operand
// of 16 columns holds 5 tokens of three digits or 8 of two (column r16 = token
// r16/HD of the group, digit r16%HD), and NG groups cover that many tokens.
// ---------------------------------------------------------------------------
// One wave's k-steps [ks_beg, ks_end) of one expert (slot; positions off ..
// off+n-1, descriptor wk), added into part[token][row] of the wave.
template <int NG, bool I4, int HD, bool TE>
__device__ __forceinline__ void down_steps(int C, int R, const ExpertPool& ep,
                                           const DecodeWork& wk, int slot, int off, int n,
                                           int ks_beg, int ks_end,
                                           const int8_t* __restrict__ hdig,
                                           const int32_t* __restrict__ hexp, float (*part)[16]) {
  constexpr int TPG = h_tok_per_group(HD);
  static_assert(!TE || (NG == 1 && HD == 3), "per-tile exponents: one token, three digits");
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, kg = lane >> 4;
  // TE: column r16 < 12 is digit d of the k-step's tile j = r16/3 (k group
  // j), so each tile's digits carry their own exponent; otherwise column
  // r16 is digit d of token m
  const int m = r16 / HD, d = r16 - HD * m;
  const int nks = R / 64;
  // tile row c0/16 of the down matrix: INT8 tiles of 1 KB (lane l at 16*l),
  // or INT4 nibble tiles of two groups (lane l at 16*l) and the tile-row's
  // 32-byte scale blocks (lane l at 8*l of a 16-group run)
  const int8_t* base = ep.pool + (size_t)slot * ep.stride;
  const int8_t* dp = I4 ? base + 2 * i4_matrix_bytes(R, C) + (size_t)blockIdx.x * (nks / 2) * kI4PairTile +
                              lane * 16
                        : base + (size_t)2 * R * C + (size_t)blockIdx.x * nks * 1024 + lane * 16;
  const int8_t* sp = base + 2 * i4_matrix_bytes(R, C) + i4_nib_bytes(C, R) +
                     (size_t)blockIdx.x * nks * 32 + lane * 8;
  const int8_t* bp[NG];
  const int32_t* hx[NG];
  bool bv[NG];
#pragma unroll
  for (int cg = 0; cg < NG; ++cg) {
    const int i = TE ? 0 : cg * TPG + m;
    bv[cg] = (TE ? r16 < 12 : r16 < HD * TPG) && i < n;
    const size_t pos = (size_t)off + (bv[cg] ? i : 0);
    bp[cg] = hdig + (pos * HD + d) * R + kg * 16;
    hx[cg] = TE ? hexp + pos * (R / 16) + m : hexp + pos * nks;
  }
  // TE: only the lanes of k group j load their tile's digits
  const bool bload = !TE || kg == m;
  // the combine's token and weight, loaded ahead of the stream so that
  // they return with the first batch
  int ctok[NG];
  float cwgt[NG];
#pragma unroll
  for (int cg = 0; cg < NG; ++cg) {
    const bool lead = (TE ? r16 == 0 : d == 0) && bv[cg];
    const int ti = TE ? 0 : cg * TPG + m;
    ctok[cg] = lead ? wk.tok[ti] : 0;
    cwgt[cg] = lead ? wk.w[ti] : 0.f;
  }
  float facc[NG][4];
#pragma unroll
  for (int cg = 0; cg < NG; ++cg)
#pragma unroll
    for (int i = 0; i < 4; ++i) facc[cg][i] = 0.f;

  // k-steps per batch: with 14 or 16 waves (up to four per SIMD, at most
  // 128 registers each) half the batch of the 8-wave layout
  constexpr int kDecUnroll = dec_unroll(NG) / 2;
  static_assert(kDecUnroll % 2 == 0 && kDecUnroll <= 16, "INT4 batches cover whole tiles");
  struct Batch {
    v4i a[I4 ? kDecUnroll / 2 : kDecUnroll], b[kDecUnroll][NG];
    uint2 s4;  // INT4: lane l holds group ks0 + l/4, rows 4*(l%4) .. +3
    int he[kDecUnroll][NG];
  };
  auto issue = [&](Batch& bt, int ks0) {
    if constexpr (I4) {
#pragma unroll
      for (int p = 0; p < kDecUnroll / 2; ++p) {
        const bool in = ks0 + 2 * p < ks_end;
        bt.a[p] = in ? ld16_stream(dp + (size_t)(ks0 / 2 + p) * kI4PairTile) : zero16();
      }
      const bool sin = (lane >> 2) < kDecUnroll && ks0 + (lane >> 2) < ks_end;
      bt.s4 = sin ? ld8_stream(sp + (size_t)ks0 * 32) : uint2{0, 0};
    }
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      const int ks = ks0 + u;
      const bool in = ks < ks_end;
      if constexpr (!I4) bt.a[u] = in ? ld16_stream(dp + ks * 1024) : zero16();
#pragma unroll
      for (int cg = 0; cg < NG; ++cg) {
        bt.b[u][cg] = (in && bv[cg] && bload) ? ld16(bp[cg] + ks * 64) : zero16();
        bt.he[u][cg] = (in && bv[cg]) ? hx[cg][TE ? 4 * ks : ks] : 0;
      }
    }
  };
  auto consume = [&](const Batch& bt) {
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      v4i a;
      float s4[4] = {1.f, 1.f, 1.f, 1.f};
      if constexpr (I4) {
        const v4i q2 = bt.a[u / 2];
        a = (u & 1) ? i4_operand(uint2{(uint32_t)q2[2], (uint32_t)q2[3]})
                    : i4_operand(uint2{(uint32_t)q2[0], (uint32_t)q2[1]});
        i4_scales(uint2{(uint32_t)__shfl((int)bt.s4.x, 4 * u + kg, 64),
                        (uint32_t)__shfl((int)bt.s4.y, 4 * u + kg, 64)}, s4);
      } else {
        a = bt.a[u];
      }
#pragma unroll
      for (int cg = 0; cg < NG; ++cg) {
        const v4i sres = mfma_i8(a, bt.b[u][cg], zero16());
        // digit weight and H' exponent; INT4 adds the row scales and 1/16
        const float sc = bv[cg] ? ldexpf(1.f, 8 * d - bt.he[u][cg] - (I4 ? 4 : 0)) : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) facc[cg][i] = fmaf((float)sres[i], sc * s4[i], facc[cg][i]);
      }
    }
  };
  // one batch per iteration (see the gate/up body)
  for (int ks = ks_beg; ks < ks_end; ks += kDecUnroll) {
    Batch bt;
    issue(bt, ks);
    consume(bt);
  }
#pragma unroll
  for (int cg = 0; cg < NG; ++cg) {
    const bool lead = (TE ? r16 == 0 : d == 0) && bv[cg];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v;
      if constexpr (TE) {
        // the twelve (tile, digit) columns of the row (lanes 12-15 hold 0)
        v = facc[cg][i];
        v += __shfl_xor(v, 1, 64);
        v += __shfl_xor(v, 2, 64);
        v += __shfl_xor(v, 4, 64);
        v += __shfl_xor(v, 8, 64);
      } else {
        v = facc[cg][i] + __shfl_down(facc[cg][i], 1, 64);
        if constexpr (HD == 3) v += __shfl_down(facc[cg][i], 2, 64);
      }
      if (lead) part[ctok[cg]][kg * 4 + i] += cwgt[cg] * v;
    }
  }
}

// NGMAX token groups cover the call.  An expert of at most one group of
// tokens runs the one-group body (batches twice as long) even if the call
// needs two.  The waves split either every expert's k-steps (each wave a range
// of each expert), or with FLAT the concatenated k-steps of all experts, so
// that a wave streams long runs of one to a few experts (kDownFlatSteps); then
// the waves of all gridDim.y workgroups of a row tile do, and out holds a
// partial output per blockIdx.y.
template <int NGMAX, int KS, bool I4, int HD, bool TE, bool FLAT>
__global__ __launch_bounds__(64 * KS) void decode_down_kernel(
    int C, int R, int T, int max_active, ExpertPool ep, const DecodeWork* __restrict__ work,
    const int8_t* __restrict__ hdig, const int32_t* __restrict__ hexp, float* __restrict__ out) {
  __shared__ float part[KS][MIRA_DECODE_MAX_TOKENS][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // each wave adds only into its own slice, so it clears only that slice and
  // nothing waits before the stream starts
  for (int i = lane; i < MIRA_DECODE_MAX_TOKENS * 16; i += 64) (&part[wave][0][0])[i] = 0.f;
  static_assert(KS > 8, "the batch size assumes more than 8 waves");

  const int nks = R / 64;
  auto steps = [&](const DecodeWork& wk, int slot, int off, int n, int ks_beg, int ks_end) {
    if (NGMAX == 1 || n <= h_tok_per_group(HD))
      down_steps<1, I4, HD, TE>(C, R, ep, wk, slot, off, n, ks_beg, ks_end, hdig, hexp, part[wave]);
    else
      down_steps<NGMAX, I4, HD, TE>(C, R, ep, wk, slot, off, n, ks_beg, ks_end, hdig, hexp, part[wave]);
  };
  if constexpr (FLAT) {
    // non-empty experts: every descriptor up to max_active is written, the
    // unused ones with group -1
    int n_act = 0;
    for (int b = 0; b < max_active; b += 64) {
      const int a = b + lane;
      n_act += __popcll(__ballot(a < max_active && work[a < max_active ? a : 0].group >= 0));
    }
    const int total = n_act * nks;
    // the waves of all gridDim.y workgroups of this row tile; even for INT4,
    // whose loads cover two k-steps (nks is even there)
    const int nw = KS * gridDim.y;
    const int per = I4 ? (((total + nw - 1) / nw + 1) & ~1) : (total + nw - 1) / nw;
    const int u0 = (blockIdx.y * KS + wave) * per, u1 = min(total, u0 + per);
    if (u0 < u1) {
      int a = u0 / nks;
      int slot = work[a].slot, off = work[a].off, n = work[a].n;
      for (int u = u0; u < u1;) {
        const int ks_beg = u - a * nks, ks_end = min(nks, u1 - a * nks);
        // the next expert's header loads while this one streams
        const int an = min(a + 1, n_act - 1);
        const int slot_n = work[an].slot, off_n = work[an].off, n_n = work[an].n;
        if (slot >= 0 && slot < ep.n_slots) steps(work[a], slot, off, n, ks_beg, ks_end);
        u = a * nks + ks_end;
        ++a;
        slot = slot_n;
        off = off_n;
        n = n_n;
      }
    }
  } else {
    // k-steps per wave; even for INT4, whose loads cover two k-steps
    const int spw = I4 ? (((nks + KS - 1) / KS + 1) & ~1) : (nks + KS - 1) / KS;
    const int ks_beg = wave * spw, ks_end = min(nks, ks_beg + spw);
    for (int a = 0; a < max_active; ++a) {
      const DecodeWork& wk = work[a];
      if (wk.group < 0) break;
      // the slot the gate/up kernel resolved from the table (-1 if invalid)
      const int slot = wk.slot;
      if (slot < 0 || slot >= ep.n_slots) continue;
      steps(wk, slot, wk.off, wk.n, ks_beg, ks_end);
    }
  }
  __syncthreads();
  for (int i = tid; i < T * 16; i += 64 * KS) {
    const int t = i >> 4, r = i & 15;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < KS; ++w) s += part[w][t][r];
    out[((size_t)blockIdx.y * T + t) * C + blockIdx.x * 16 + r] = s;
  }
}

// out = sum over p < parts of part[p], in order; n floats each, n a multiple of 4
// (out is 16-byte aligned, as every entry point requires)
__global__ __launch_bounds__(256) void decode_add_kernel(const float* __restrict__ part, int parts,
                                                         float* __restrict__ out, int n) {
  const int i = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  v4f s = *(const v4f*)(part + i);
  for (int p = 1; p < parts; ++p) s += *(const v4f*)(part + (size_t)p * n + i);
  *(v4f*)(out + i) = s;
}

// Waves per workgroup: 16 for INT8 (twice the loads in flight per CU of 8
// waves with batches of half the size); 14 for INT4, whose 16-byte loads
// cover two k-steps: R/64 = 224 k-steps then split into 16 per wave and
// expert, two whole batches (Mixtral INT4 decode 0.9 us faster per call; the
// INT8 kernel is 0.4-0.5 us slower with 14)
template <bool I4>
constexpr int down_waves() { return I4 ? 14 : 16; }

// Most k-steps per expert (R/64) for which the waves split the concatenated
// k-steps of all experts (FLAT) instead of each expert's.  Splitting each
// expert leaves a wave one to two k-steps of it at R = 1408 and one memory
// round trip per expert, up to T*k + S in a row; with FLAT a wave streams a
// few long runs.  The fine-grained layer (C 2048, R 1408, 64 experts top-6, 2
// shared), us per call with split experts / FLAT: 1 token 44.4 / 36.0, 8
// tokens 81.9 / 67.7, 16 tokens INT4 131 / 99.  FLAT is even with or ahead of
// split experts by up to 2% up to R = 5632 (88 k-steps); at R = 8192 it is
// 1% ahead with 8 tokens and 2% behind with 16, and at 14336, where a split
// expert fills two batches of a wave, 1% behind with one token.
constexpr int kDownFlatSteps = 96;

// How many workgroups share each 16-row tile, an equal part of the
// concatenated k-steps each: as many (up to 4) as the CUs that the C/16 tiles
// leave idle allow, with at least kDownPartSteps steps (of the experts the call
// can reach) a part, so that they outlast the launch that adds the partial
// outputs (some 4 us).  Those lie in the prefill path's partials, which decode
// calls do not use.  us per call with 1 / 2 workgroups a tile: C 2048, R 1408,
// 64 experts top-6, 2 shared: 2 tokens (308 steps) 34.7 / 33.8, 8 tokens 57.8 /
// 53.4, 16 tokens 89.5 / 82.4 (INT4 33.4 / 33.3, 50.3 / 47.7, 75.5 / 71.2); with 1 / 2 / 4: C
// 512, R 2816, 64 experts top-4: 2 tokens 30.6 / 29.0 / - , 8 tokens 43.0 /
// 38.0 / 33.8, 16 tokens 66.3 / 56.9 / 49.6.  Below 300 steps it is even.
constexpr int kDownPartSteps = 150, kDownMaxParts = 4;
static int down_parts(const Layout& L) {
  if (L.T == 1 || L.R / 64 > kDownFlatSteps) return 1;
  int parts = std::min(kDownMaxParts, device_cu_count() / (L.C / 16));
  parts = std::min(parts, decode_max_active(L) * (L.R / 64) / kDownPartSteps);
  parts = std::min(parts, L.ksplit * L.P / L.T);
  return std::max(parts, 1);
}

template <int NG, bool I4, int HD, bool TE = false>
static void launch_decode_down_ng(const Layout& L, const WsPtr& w, const ExpertPool& ep,
                                  float* out, hipStream_t st) {
  constexpr int KS = down_waves<I4>();
  const int parts = down_parts(L);
  if (parts > 1) {
    launch_timed("decode_down", (decode_down_kernel<NG, KS, I4, HD, TE, true>), dim3(L.C / 16, parts),
                 dim3(64 * KS), 0, st, L.C, L.R, L.T, decode_max_active(L), ep, w.dwork, w.hdig, w.hexp, w.ybuf);
    const int n = L.T * L.C;
    launch_timed("decode_add", decode_add_kernel, dim3((n / 4 + 255) / 256), dim3(256), 0, st,
                 (const float*)w.ybuf, parts, out, n);
    return;
  }
  const auto kern = L.R / 64 <= kDownFlatSteps ? decode_down_kernel<NG, KS, I4, HD, TE, true>
                                               : decode_down_kernel<NG, KS, I4, HD, TE, false>;
  launch_timed("decode_down", kern, dim3(L.C / 16), dim3(64 * KS), 0, st, L.C, L.R, L.T,
               decode_max_active(L), ep, w.dwork, w.hdig, w.hexp, out);
}

// Largest hidden size for which the INT8 gate/up kernels of two and three token
// groups keep three workgroups on a CU.  The bodies by token count take a few
// registers more than the 168 that allow it.  Up to 1024 (16 k-steps) a
// workgroup is over after two weight batches, and a third one hides the start
// of the next; with longer rows two workgroups of looser schedule are even or
// ahead.  us per call with two / three: C 512, R 8192, 8 experts top-2, 8 tokens
// 56.4 / 54.9; C 768, R 13952, 8 experts top-5 and one shared, 8 tokens 141.7 /
// 138.1; C 1024, R 4096, 16 experts top-4 and one shared, 6 tokens 44.1 / 41.5; C
// 1536, R 2048, 13 tokens 53.7 / 55.4; C 2048, R 1408, 64 experts top-6, 2 shared,
// 15 tokens 72.1 / 74.9; Mixtral shape, 8 tokens 215.9 / 216.7.
constexpr int kThreePerCuMaxC = 1024;

template <int NG, bool I4>
static void launch_decode_gateup(const Layout& L, const WsPtr& w, const ExpertPool& ep,
                                 hipStream_t st) {
  const int nrb = L.R / kBlk;
  const int max_active = decode_max_active(L);
  if constexpr (I4) {
    if (L.C <= kXlMaxC) {
      launch_timed("decode_gateup", decode_gateup_xl_kernel<NG>, dim3(max_active * nrb), dim3(256),
                   xl_bytes(L.C), st,
                   L.C, L.R, ep, w.dwork, w.xdig, w.hdig, w.hexp);
      return;
    }
  }
  auto kern = decode_gateup_kernel<NG, I4, 1>;
  if constexpr (!I4 && (NG == 2 || NG == 3)) {
    if (L.C <= kThreePerCuMaxC) kern = decode_gateup_kernel<NG, I4, 3>;
  }
  launch_timed("decode_gateup", kern, dim3(max_active * nrb), dim3(256), 0, st, L.C, L.R, ep,
               w.dwork, w.xdig, w.hdig, w.hexp);
}

// One token: the 16-row tiles of all active experts split evenly over the
// CUs (W waves per workgroup, about one workgroup per CU), and the down
// kernel reads per-tile exponents.  q: the selection, if gate/up makes it.
template <bool I4>
static void launch_decode_ffn_1tok(const Layout& L, const WsPtr& w, const ExpertPool& ep,
                                   const OneTokenSel* q, float* out, hipStream_t st) {
  const int ntiles = decode_max_active(L) * (L.R / 16);
  const int cus = device_cu_count();
  const int W = std::min(kTileMaxWaves, (ntiles + cus - 1) / cus);
  const int nwg = (ntiles + W - 1) / W;
  const auto kern = I4 ? (q ? decode_gateup_tile_i4_kernel<true> : decode_gateup_tile_i4_kernel<false>)
                       : (q ? decode_gateup_tile_kernel<true> : decode_gateup_tile_kernel<false>);
  launch_timed("decode_gateup", kern, dim3(nwg), dim3(64 * W), 0, st, L.C, L.R, W, ntiles, ep,
               w.dwork, q ? *q : OneTokenSel{}, w.xdig, w.hdig, w.hexp);
  launch_decode_down_ng<1, I4, 3, true>(L, w, ep, out, st);
}

template <bool I4>
static void launch_decode_ffn(const Layout& L, const WsPtr& w, const ExpertPool& ep, float* out,
                              hipStream_t st) {
  if (L.T == 1 && (!I4 || L.C <= kXlMaxC)) {
    launch_decode_ffn_1tok<I4>(L, w, ep, nullptr, out, st);
    return;
  }
  // token groups of an expert (each holds at most T tokens): 5 tokens per x
  // operand; H' in three digits for one x group (5 tokens per operand),
  // else in two (8 tokens per operand)
  const int ng = (L.T + kTokPerGroup - 1) / kTokPerGroup;
  switch (ng) {
    case 1: launch_decode_gateup<1, I4>(L, w, ep, st); break;
    case 2: launch_decode_gateup<2, I4>(L, w, ep, st); break;
    case 3: launch_decode_gateup<3, I4>(L, w, ep, st); break;
    default: launch_decode_gateup<4, I4>(L, w, ep, st); break;
  }
  static_assert(MIRA_DECODE_MAX_TOKENS <= 2 * h_tok_per_group(2), "two H' groups cover a decode call");
  if (ng == 1)
    launch_decode_down_ng<1, I4, 3>(L, w, ep, out, st);
  else if (L.T <= h_tok_per_group(2))
    launch_decode_down_ng<1, I4, 2>(L, w, ep, out, st);
  else
    launch_decode_down_ng<2, I4, 2>(L, w, ep, out, st);
}

hipError_t launch_decode(const mira_shape& s, const Layout& L, const WsPtr& w, const void* x,
                         const ExpertPool& ep, float* out, hipStream_t st) {
  (void)x;  // x enters through the fixed-point digits written by decode_prep_kernel
  const int T = L.T;
  if (T == 0) return hipSuccess;
  if (s.flags & MIRA_FLAG_INT4)
    launch_decode_ffn<true>(L, w, ep, out, st);
  else
    launch_decode_ffn<false>(L, w, ep, out, st);
  return hipGetLastError();
}

// Tiles per CU up to which a call of at most 16 experts selects inside gate/up.
// Eight waves fill a CU, and every further round of workgroups selects anew
// before it streams, where a router of one expert tile costs the preparation
// kernel little.  us per call, selection inside / in the preparation kernel: 8
// tiles per CU (16 experts top-8, R 4096), C 512 64.6 / 65.6 (two layers), C 4096
// 77.6 / 78.1; 12 (10 experts top-4, 2 shared), C 768, R 8192 99.3 / 99.4 (two);
// 16 (16 experts top-8, R 8192), C 768 121.2 / 120.4 (two), C 2048 90.1 / 90.0; 22, C
// 512, R 11456 148.6 / 145.2 (two); 28, C 1024, R 14336 109.2 / 106.2, INT4 85.8 /
// 83.6.  With more experts the preparation kernel costs more, and selecting inside
// is ahead at any count (64 experts top-6, 2 shared, C 512, R 11456, 22 tiles: 73.5 /
// 76.3).
constexpr int kFusedTilesPerCu = 12;

bool one_token_fused(const mira_shape& s, const Layout& L) {
  return L.T == 1 && L.E <= 64 && L.k + L.S <= 64 && (!(s.flags & MIRA_FLAG_INT4) || L.C <= kXlMaxC) &&
         (L.E > 16 || decode_max_active(L) * (L.R / 16) <= kFusedTilesPerCu * device_cu_count());
}

hipError_t launch_one_token(const mira_shape& s, const Layout& L, const WsPtr& w, const void* x,
                            const void* wr, const float* bias, float* logits_out,
                            const ExpertPool& ep, int32_t* counts_out, int32_t* idx_out,
                            float* wts_out, int32_t* offsets_out, int32_t* order_out, float* out,
                            hipStream_t st) {
  launch_decode_logits(s, L, w, x, wr, bias, logits_out, st);
  const OneTokenSel q{w.logits, decode_xe(w), L.E, L.k, L.S, (s.flags & MIRA_FLAG_SOFTMAX_ALL) ? 1 : 0,
                      perm_out(w, counts_out, idx_out, wts_out, offsets_out, order_out)};
  if (s.flags & MIRA_FLAG_INT4)
    launch_decode_ffn_1tok<true>(L, w, ep, &q, out, st);
  else
    launch_decode_ffn_1tok<false>(L, w, ep, &q, out, st);
  return hipGetLastError();
}

}  // namespace mira
